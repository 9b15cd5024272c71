"""vlbm_pass_bytes (no GPU): the lattices whose steps can go in passes, and what buffer they take."""
import ctypes

import pytest

BODY = dict(c0=[40, 40, 40], v=[0, 0, 0], R0=2.0, a=[0] * 4, d=[[1, 0, 0]] * 4, b=[0] * 4, e=[[1, 0, 0]] * 4, m=[0, 0, 0],
            mode=2)
RES = dict(dt=1e-3, tau_M=0.01, tau_H=0.01)


@pytest.mark.parametrize("takes,kw", [
    (True, dict()),
    (True, dict(storage="f64", collision="trt")),
    (True, dict(model="resistive_2d", **RES)),
    (True, dict(lattice="D3Q7", shape=(64, 64, 64))),
    (True, dict(lattice="D3Q7", shape=(64, 64, 64), model="euler", collision="mrt")),
    (True, dict(shape=(4096, 4096, 1), model="resistive_2d", **RES)),  # 4.4 GB, below 4.5 GiB
    (False, dict(storage="f16")),
    (False, dict(source="guo", storage="f64")),
    (False, dict(shape=(1400, 2, 40000))),  # 16 GB, above 4.5 GiB
    (False, dict(lattice="D3Q7", shape=(64, 64, 64), storage="f64")),
    (False, dict(lattice="D3Q7", shape=(64, 64, 64), collision="trt")),
    (False, dict(lattice="D3Q7", shape=(64, 64, 63))),  # fewer than 2^18 cells
    (False, dict(lattice="D3Q7", shape=(64, 64, 64), model="resistive", **RES)),
    (False, dict(lattice="D3Q7", shape=(64, 64, 64), bc=(0, 0, 2, 2, 0, 0), inflow_Q=[1, 0, 0, 0, 1, 0, 0, 0])),
    (False, dict(lattice="D3Q7", shape=(64, 64, 64), body=BODY, inflow_Q=[1, 0, 0, 0, 1, 0, 0, 0])),
])
def test_pass_bytes(takes, kw):
    from paper_2606_00641_amd import vlbm as vb
    p = vb.make_params(**kw)
    n, m = ctypes.c_size_t(), ctypes.c_size_t()
    assert vb.lib().vlbm_population_bytes(ctypes.byref(p), ctypes.byref(n)) == 0
    assert vb.lib().vlbm_pass_bytes(ctypes.byref(p), ctypes.byref(m)) == 0
    assert m.value == (n.value if takes else 0)
    assert vb.lib().vlbm_pass_bytes(ctypes.byref(p), None) == vb.VLBM_ERR_ARG
    assert vb.lib().vlbm_set_passes(None, 1) == vb.VLBM_ERR_ARG
