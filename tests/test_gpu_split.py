"""How a run is split into calls does not show in its populations: one call, single steps, a
restart at an odd step and a corrected run that corrects nothing give the same bits, on lattices
of every kernel that takes several steps in one pass (FP64 and FP32; strips of rows, tiles of
both widths, 3D columns) and of the in-place sweeps beside them (rows the workgroups tile, with
and without the exchange between lanes, and flat ones)."""
import numpy as np
import pytest

import synth
from test_gpu_parity import _euler, boosted, gpu_params, vb  # noqa: F401
from test_gpu_rows import _case

pytestmark = pytest.mark.gpu


def _state(model, shape, dim):
    if dim == 2:
        return _case(model, shape)
    if model == "navier_cauchy":
        return synth.workload_elastic(dim=3, shape=shape), synth.elastic_state(shape, seed=3)
    w = synth.workload_slab_3d()
    w["shape"] = shape
    Q0 = np.ascontiguousarray(boosted(synth.planar_discontinuity_3d(seed=5, shape=shape[::-1])[0], (0.3, -0.2, 0.25)))
    return (_euler(w), synth.without_field(Q0)) if model == "euler" else (w, Q0)


# strips of rows from 9.4e6 cells x variables in FP32, their last strip a quarter empty and the
# last share of rows short
ROWS = [("ideal", (2670, 450, 1)), ("euler", (9000, 17, 14)), ("navier_cauchy", (1100, 1063, 1))]
# tiles: one 16 x 16, both widths with a cell past the last whole tile, a batch
TILES = [("ideal", (31, 9, 2)), ("ideal", (261, 301, 1)), ("euler", (261, 301, 1)), ("euler", (100, 97, 4)),
         ("navier_cauchy", (261, 301, 1)), ("navier_cauchy", (79, 71, 1)), ("resistive_2d", (79, 71, 1)),
         ("resistive_2d", (287, 301, 1))]
# columns: rows the workgroups tile (64, 192) and flat rows, one to four strips
COLS = [("ideal", (64, 65, 66)), ("ideal", (63, 89, 48)), ("ideal", (190, 29, 49)), ("euler", (192, 29, 49)),
        ("euler", (119, 47, 49)), ("navier_cauchy", (119, 47, 49))]
CASES = ([(m, s, 2, st, c) for m, s in ROWS for st in ("f32",) for c in ("bgk", "trt", "mrt")]
         + [(m, s, 2, st, c) for m, s in TILES for st in ("f64", "f32") for c in ("bgk", "trt")]
         + [(m, s, 3, "f32", "bgk") for m, s in COLS]
         + [("euler", s, 3, "f32", c) for s in ((63, 89, 48), (190, 29, 49)) for c in ("trt", "mrt")])


@pytest.mark.parametrize("model,shape,dim,storage,collision", CASES)
def test_split_of_a_run(vb, model, shape, dim, storage, collision):  # noqa: F811
    """23 steps: at once; one by one; and 11, a restart of another context from its
    populations, and 12 -- bit for bit."""
    w, Q0 = _state(model, shape, dim)
    print("case split", model, shape, storage, collision, flush=True)
    p = gpu_params(vb, w, storage)
    p.collision = {"bgk": 0, "trt": 1, "mrt": 3}[collision]
    p.trt_magic, p.mrt_tau_e, p.mrt_tau_d = 0.2, 0.9, 1.1
    sims = [vb.Vlbm(p) for _ in range(2)]
    for sim in sims:
        sim.vlbm_init_fields(Q0)
    sims[0].vlbm_step(23)
    for _ in range(23):
        sims[1].vlbm_step(1)
    want, par, step = sims[1].vlbm_get_populations()
    assert (par, step) == (1, 23) and np.isfinite(want.view(np.float64 if storage == "f64" else np.float32)).all()
    assert np.array_equal(sims[0].vlbm_get_populations()[0], want)
    sims[0].vlbm_init_fields(Q0)
    sims[0].vlbm_step(11)
    saved = sims[0].vlbm_get_populations()
    sims[0].vlbm_destroy()
    sims[1].vlbm_set_populations(*saved)
    sims[1].vlbm_step(12)
    assert np.array_equal(sims[1].vlbm_get_populations()[0], want)


@pytest.mark.parametrize("shape,dim", [((64, 64, 64), 3), ((80, 64, 64), 3), ((2672, 448, 1), 2)])
def test_zero_network_on_lattices_of_passes(vb, shape, dim):  # noqa: F811
    """A corrected run whose network is zero (every step accepted) and one whose bound is zero
    (every step rejected) are bitwise the plain run, whose steps go in passes."""
    import torch
    from paper_2606_00641_amd import nn
    w, Q0 = _state("ideal", shape, dim)
    print("case zero network", shape, flush=True)
    plain, zero, held = (vb.Vlbm(gpu_params(vb, w, "f32")) for _ in range(3))
    for sim in (plain, zero, held):
        sim.vlbm_init_fields(Q0)
    net = nn.Net(8, 32, 3, stream=torch.cuda.current_stream().cuda_stream, dim=dim)
    assert nn.vlbm_step_corrected(zero, net, 10, np.full(8, 1e30), 0.1) == 0
    rng = np.random.default_rng(3)
    net.vlbm_nn_set_weights((0.1 * rng.standard_normal(net.vlbm_nn_num_params())).astype(np.float32))
    assert nn.vlbm_step_corrected(held, net, 10, np.zeros(8), 0.1) == 10
    plain.vlbm_step(10)
    want = plain.vlbm_get_populations()[0]
    assert np.array_equal(zero.vlbm_get_populations()[0], want)
    assert np.array_equal(held.vlbm_get_populations()[0], want)


@pytest.mark.parametrize("storage", ["f16", "bf16"])
@pytest.mark.parametrize("shape,dim", [((48, 32, 16), 3), ((80, 64, 32), 3), ((208, 32, 48), 3), ((80, 48, 1), 2),
                                       ((144, 96, 3), 2)])
def test_zero_network_on_flat_rows_16_bit(vb, shape, dim, storage):  # noqa: F811
    """The same in FP16 and BF16 storage on rows the workgroups do not tile: the plain sweep takes
    them flat, one and (the two large 3D lattices) two cells a lane, the injecting sweep by rows."""
    import torch
    from paper_2606_00641_amd import nn
    w, Q0 = _state("ideal", shape, dim)
    print("case zero network 16 bit", shape, storage, flush=True)
    plain, zero = (vb.Vlbm(gpu_params(vb, w, storage)) for _ in range(2))
    for sim in (plain, zero):
        sim.vlbm_init_fields(Q0)
    net = nn.Net(8, 32, 3, stream=torch.cuda.current_stream().cuda_stream, dim=dim)
    assert nn.vlbm_step_corrected(zero, net, 40, np.full(8, 1e30), 0.1) == 0
    plain.vlbm_step(40)
    assert np.array_equal(zero.vlbm_get_populations()[0], plain.vlbm_get_populations()[0])
