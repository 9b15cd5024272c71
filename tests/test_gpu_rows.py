"""Several steps of a lattice in one pass over memory: against the same number of single
steps, which sweep in place, and against the oracle.  Lattices one strip and one row past
the passes' tilings, narrower than a strip, flatter than the rows a pass adds, batches."""
import numpy as np
import pytest

import oracle
import synth
from fieldcheck import rel_l2
from test_gpu_parity import _euler, boosted, gpu_params, oracle_params, vb  # noqa: F401

pytestmark = pytest.mark.gpu


def _case(model, shape):
    nx, ny, nb = shape
    if model == "resistive_2d":
        w = synth.workload_resistive_2d(n=nx, ny=ny)
        Q0 = np.concatenate([synth.resistive_2d_state((ny, nx), seed=3 + b, tau_M=w["tau_M"], tau_H=w["tau_H"],
                                                      mu=w["mu"]) for b in range(nb)], axis=1)
    elif model == "navier_cauchy":
        w = synth.workload_elastic(dim=2, shape=shape)
        Q0 = np.concatenate([synth.elastic_state((nx, ny, 1), seed=3 + b) for b in range(nb)], axis=1)
    else:
        w = synth.workload_fourier_2d()
        rng = np.random.default_rng(5)
        u = 0.05 * rng.standard_normal((3, nb, ny, nx))
        B = 0.1 + 0.05 * rng.standard_normal((3, nb, ny, nx))
        Q0 = synth.conserved_from_primitive(1.0 + 0.05 * rng.standard_normal((nb, ny, nx)), u, 0.6, B, 5.0 / 3.0)
        if model == "euler":
            w, Q0 = _euler(w), synth.without_field(Q0)
    w["shape"] = shape
    return w, np.ascontiguousarray(Q0)


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("model,shape", [("ideal", (601, 450, 1)), ("ideal", (100, 2700, 1)), ("ideal", (140000, 2, 1)),
                                         ("ideal", (232, 130, 9)), ("euler", (583, 451, 1)),
                                         ("navier_cauchy", (583, 451, 1)), ("resistive_2d", (583, 451, 1))])
def test_passes_equal_single_steps(vb, model, shape, storage):  # noqa: F811
    """15 steps at once (in FP32 one pair of 4-step passes, one of 2-step passes and three
    sweeps) and one by one.  Both within the parity gate of the oracle: FP64 1e-10; FP32
    1e-5, or for the small transported fields, whose FP32 rounding exceeds it, twice the
    single steps' own distance (the same arithmetic per cell, rounded differently), and
    then no further from one another than the two distances together."""
    w, Q0 = _case(model, shape)
    K = Q0.shape[0]
    print("case passes", model, shape, storage, flush=True)
    sims = [vb.Vlbm(gpu_params(vb, w, storage)) for _ in range(2)]
    for sim in sims:
        sim.vlbm_init_fields(Q0)
    sims[0].vlbm_step(15)
    for _ in range(15):
        sims[1].vlbm_step(1)
    assert sims[0].vlbm_get_step() == sims[1].vlbm_get_step() == 15
    Qa, Qb = (sim.vlbm_moments()[0] for sim in sims)
    op = oracle_params(w)
    f = oracle.init(op, Q0)
    oracle.run(op, f, 15)
    Qo = oracle.moments(op, f)[0]
    gate = 1e-10 if storage == "f64" else 1e-5
    own, far, apart = rel_l2(Qb, Qo, K), rel_l2(Qa, Qo, K), rel_l2(Qa, Qb, K)
    for name in own:
        assert far[name] <= max(gate, 2.0 * own[name]), (name, far[name], own[name])
        assert apart[name] <= max(gate, 3.0 * own[name]), (name, apart[name], own[name])
    # populations of single cells after more passes from an odd step on (natural layout)
    sims[0].vlbm_step(9)
    for _ in range(9):
        sims[1].vlbm_step(1)
    cells = np.array([0, 1, shape[0] - 1, shape[0], 57, 58, 63, shape[0] * shape[1] - 1])
    a, b = (sim.vlbm_gather_cells(cells) for sim in sims)
    assert np.abs(a - b).max() <= gate * np.abs(b).max()


# 3D passes: one strip, exactly full and narrowest; two strips one column past one; four of 48
# columns and a part; rows and planes that leave the last tile and share part empty
@pytest.mark.parametrize("collision", ["bgk", "trt"])
@pytest.mark.parametrize("model,shape", [("ideal", (62, 65, 66)), ("ideal", (63, 89, 48)), ("ideal", (190, 29, 49)),
                                         ("ideal", (56, 17, 276)), ("euler", (119, 47, 49)),
                                         ("navier_cauchy", (119, 47, 49))])
def test_passes_equal_single_steps_3d(vb, model, shape, collision):  # noqa: F811
    """15 steps at once (three pairs of 2-step passes and three sweeps) and one by one, FP32;
    the gates of the 2D test, and the populations after more passes from an odd step on."""
    if model == "navier_cauchy":
        w = synth.workload_elastic(dim=3, shape=shape)
        Q0 = synth.elastic_state(shape, seed=3)
    else:
        w = synth.workload_slab_3d()
        w["shape"] = shape
        Q0 = np.ascontiguousarray(boosted(synth.planar_discontinuity_3d(seed=5, shape=shape[::-1])[0], (0.3, -0.2, 0.25)))
        if model == "euler":
            w, Q0 = _euler(w), synth.without_field(Q0)
    K = Q0.shape[0]
    print("case passes 3d", model, shape, collision, flush=True)
    p = gpu_params(vb, w, "f32")
    op = oracle_params(w)
    if collision == "trt":
        p.collision, p.trt_magic = 1, 0.25
        op.collision, op.trt_magic = 1, 0.25
    sims = [vb.Vlbm(p) for _ in range(2)]
    for sim in sims:
        sim.vlbm_init_fields(Q0)
    sims[0].vlbm_step(15)
    for _ in range(15):
        sims[1].vlbm_step(1)
    assert sims[0].vlbm_get_step() == sims[1].vlbm_get_step() == 15
    Qa, Qb = (sim.vlbm_moments()[0] for sim in sims)
    f = oracle.init(op, Q0)
    oracle.run(op, f, 15)
    Qo = oracle.moments(op, f)[0]
    own, far, apart = rel_l2(Qb, Qo, K), rel_l2(Qa, Qo, K), rel_l2(Qa, Qb, K)
    for name in own:
        assert far[name] <= max(1e-5, 2.0 * own[name]), (name, far[name], own[name])
        assert apart[name] <= max(1e-5, 3.0 * own[name]), (name, apart[name], own[name])
    sims[0].vlbm_step(9)
    for _ in range(9):
        sims[1].vlbm_step(1)
    n = int(np.prod(shape))
    cells = np.unique(np.concatenate([[0, shape[0] - 1, shape[0], n - 1], np.random.default_rng(1).integers(0, n, 4000)]))
    a, b = (sim.vlbm_gather_cells(cells) for sim in sims)
    assert np.abs(a - b).max() <= 1e-5 * np.abs(b).max()


# 2D tiles: a lattice inside one tile, one cell past the 10 x 10 and 26 x 10 results, thin ones,
# batches, one row of tiles; FP64 and 13 variables at a size of 32 x 16 tiles; large FP32 lattices
# by rows, the last strip a quarter empty and the rows fewer than one share
@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("model,shape", [("ideal", (1, 1, 1)), ("ideal", (11, 21, 3)), ("ideal", (2, 31, 1)),
                                         ("ideal", (131, 141, 2)), ("euler", (261, 301, 1)), ("navier_cauchy", (79, 71, 1)),
                                         ("resistive_2d", (287, 301, 1)), ("resistive_2d", (64, 21, 1)),
                                         ("ideal", (2670, 450, 1)), ("euler", (9000, 17, 14))])
def test_tiles_equal_single_steps(vb, model, shape, storage):  # noqa: F811
    """13 steps at once (a pair of 4-step passes, one of 2-step passes, one sweep) and one by
    one: to 1e-12 (FP64), 1e-5 (FP32) of each variable's largest population, small variables a
    tenth of the largest (a step rounds to some 1e-7 of the fluxes that enter it)."""
    w, Q0 = _case(model, shape)
    print("case tiles", model, shape, storage, flush=True)
    sims = [vb.Vlbm(gpu_params(vb, w, storage)) for _ in range(2)]
    for sim in sims:
        sim.vlbm_init_fields(Q0)
    sims[0].vlbm_step(13)
    for _ in range(13):
        sims[1].vlbm_step(1)
    n = int(np.prod(shape))
    cells = np.arange(n) if n < 200000 else np.unique(np.random.default_rng(1).integers(0, n, 200000))
    a, b = (sim.vlbm_gather_cells(cells) for sim in sims)
    scale = np.abs(b).max(axis=(0, 2), keepdims=True)
    assert np.all(np.abs(a - b) <= (1e-12 if storage == "f64" else 1e-5) * np.maximum(scale, 0.1 * np.abs(b).max()))


@pytest.mark.parametrize("model,shape,dim", [("ideal", (131, 47, 1), 2), ("ideal", (63, 89, 48), 3)])
def test_passes_under_capture(vb, model, shape, dim):  # noqa: F811
    """A captured vlbm_step(8) replayed three times, with eager work between the replays, is the
    same 24 steps taken eagerly, bit for bit (the passes are launches and nothing else)."""
    import torch
    print("case capture", model, shape, flush=True)
    if dim == 2:
        w, Q0 = _case(model, shape)
    else:
        w = synth.workload_slab_3d()
        w["shape"] = shape
        Q0 = np.ascontiguousarray(boosted(synth.planar_discontinuity_3d(seed=5, shape=shape[::-1])[0], (0.3, -0.2, 0.25)))
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        sims = [vb.Vlbm(gpu_params(vb, w, "f32")) for _ in range(2)]
        for sim in sims:
            sim.vlbm_init_fields(Q0)
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            sims[0].vlbm_step(8)
        cells = np.unique(np.random.default_rng(2).integers(0, int(np.prod(shape)), 3000))
        for _ in range(3):
            graph.replay()
            torch.zeros(1000, device="cuda").add_(1.0)
            side.synchronize()
            sims[1].vlbm_step(8)
            a, b = (sim.vlbm_gather_cells(cells) for sim in sims)
            assert np.array_equal(a, b)
