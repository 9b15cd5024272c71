"""Sweeps whose workgroups take consecutive cells of the whole lattice (x rows that no
workgroup width tiles): rows shorter and longer than a wavefront, one cell past a
workgroup, odd rows, lattices whose last workgroup is partly empty."""
import numpy as np
import pytest

import oracle
import synth
from fieldcheck import oracle_one_step, rel_l2
from test_gpu_parity import boosted, gpu_params, oracle_params, vb  # noqa: F401

pytestmark = pytest.mark.gpu


def _ideal(shape, seed=5):
    w = synth.workload_slab_3d()
    w["shape"] = shape
    Q0, _ = synth.planar_discontinuity_3d(seed=seed, shape=shape[::-1])
    return w, np.ascontiguousarray(boosted(Q0, (0.3, -0.2, 0.25)))


@pytest.mark.parametrize("steps", [5, 6])
@pytest.mark.parametrize("shape", [(1, 3, 2), (2, 3, 5), (63, 3, 2), (65, 2, 3), (129, 5, 4), (190, 7, 3), (257, 3, 2)])
def test_flat_sweep_fp64(vb, shape, steps):  # noqa: F811
    """FP64 against the oracle, both parities: the method's parity gate of 1e-10."""
    w, Q0 = _ideal(shape)
    print("case flat sweep", shape, steps, flush=True)
    sim = vb.Vlbm(gpu_params(vb, w, "f64"))
    sim.vlbm_init_fields(Q0)
    sim.vlbm_step(steps)
    Q, _ = sim.vlbm_moments()
    op = oracle_params(w)
    f = oracle.init(op, Q0)
    oracle.run(op, f, steps)
    assert max(rel_l2(Q, oracle.moments(op, f)[0], 8).values()) <= 1e-10


@pytest.mark.parametrize("storage,ulp", [("f16", 2.0 ** -11), ("bf16", 2.0 ** -8)])
@pytest.mark.parametrize("parity", [0, 1])
@pytest.mark.parametrize("shape", [(130, 41, 25), (131, 33, 33), (66, 9, 7), (21, 13, 5)])
def test_flat_sweep_low_precision_one_step(vb, shape, storage, ulp, parity):  # noqa: F811
    """FP16/BF16: two cells per lane (the two large lattices; an odd one at parity 0) and
    one.  One step from the GPU's own populations against the oracle's collision of every
    cell, up to one rounding of the stored deviation (plus FP32 arithmetic)."""
    w, Q0 = _ideal(shape)
    print("case flat pair", shape, storage, parity, flush=True)
    sim = vb.Vlbm(gpu_params(vb, w, storage))
    sim.vlbm_init_fields(Q0)
    sim.vlbm_step(2 + parity)
    cells = np.arange(int(np.prod(shape)))
    op = oracle_params(w)
    want = oracle_one_step(oracle, op, sim.vlbm_gather_cells, cells, shape, 3)
    sim.vlbm_step(1)
    got = sim.vlbm_gather_cells(cells)
    rest_Q, sigma = sim.vlbm_get_codec()
    sc = sigma[:, None] * np.array([0.25] + [0.125] * 6)[None, :]
    h_want = np.abs(want - oracle.equilibrium(op, rest_Q)[None]) / sc[None]
    bound = sc[None] * (2.0 * ulp * h_want + 2.0 ** -24) + 4e-6 * (1.0 + np.abs(want))
    err = np.abs(got - want)
    assert np.all(err <= bound), float((err / bound).max())
    # the padding of the planes stays as the context made it
    buf = sim.vlbm_get_populations()[0].view(np.uint16).reshape(56, -1)
    assert not buf[:, len(cells):].any()
