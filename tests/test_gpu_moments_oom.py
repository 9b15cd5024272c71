"""Moments to an FP32 host array need an FP64 host array on their way: where it cannot be had, the
call returns VLBM_ERR_OOM and the context goes on working."""
import ctypes
import resource

import numpy as np
import pytest

import synth
from test_gpu_parity import gpu_params, vb  # noqa: F401

pytestmark = pytest.mark.gpu


def test_no_host_memory_for_the_moments(vb):  # noqa: F811
    w = synth.workload_slab_3d()
    w["shape"] = (192, 192, 192)
    sim = vb.Vlbm(gpu_params(vb, w, "f32"))
    Q0 = np.zeros((8, sim.N), np.float32)
    Q0[0], Q0[4] = 1.0, 1.0
    sim.vlbm_init_fields(Q0)
    want, got = (np.empty((8, sim.N), np.float32) for _ in range(2))
    tot = (ctypes.c_double * 13)()

    def moments(Q):
        return vb.lib().vlbm_moments(sim.ctx, Q.ctypes.data_as(ctypes.c_void_p), 0, 1, tot)

    assert moments(want) == 0  # the device's scratch is taken
    print("case no host memory", flush=True)
    with open("/proc/self/statm") as fh:
        used = int(fh.read().split()[0]) * resource.getpagesize()
    soft, hard = resource.getrlimit(resource.RLIMIT_AS)
    resource.setrlimit(resource.RLIMIT_AS, (used + (128 << 20), hard))  # 453 MB are needed
    try:
        st = moments(got)
    finally:
        resource.setrlimit(resource.RLIMIT_AS, (soft, hard))
    assert st == vb.VLBM_ERR_OOM
    assert b"host" in vb.lib().vlbm_last_error(sim.ctx)
    assert moments(got) == 0 and np.array_equal(got, want)
