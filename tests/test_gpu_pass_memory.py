"""The second population buffer of the passes of several steps: taken by the first step that
uses it and by nothing else, given back on request, never beside an adopted buffer unasked;
the populations do not depend on it."""
import numpy as np
import pytest

import synth
from test_gpu_parity import gpu_params, vb  # noqa: F401
from test_gpu_rows import _case

pytestmark = pytest.mark.gpu

SHAPE = (1536, 1536, 1)  # 8 variables in FP32: 378 MB of populations


def _free():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.fixture(scope="module")
def case(vb):  # noqa: F811
    w, Q0 = _case("ideal", SHAPE)
    import torch
    Q = torch.from_numpy(Q0).cuda()
    sim = vb.Vlbm(gpu_params(vb, w, "f32"))  # the library's kernels are loaded
    sim.vlbm_init_fields(Q)
    sim.vlbm_step(1)
    sim.vlbm_destroy()
    return w, Q


def test_only_passes_take_the_buffer(vb, case):  # noqa: F811
    """Creation, initialisation, calls of fewer steps and corrected steps take at most a tenth
    of a second buffer beyond the first, whatever the lattice could use."""
    import torch
    from paper_2606_00641_amd import nn
    w, Q = case
    print("case buffer of passes", flush=True)
    net = nn.Net(8, 32, 3, stream=torch.cuda.current_stream().cuda_stream)
    warm = vb.Vlbm(gpu_params(vb, w, "f32"))  # the network's own workspace
    warm.vlbm_init_fields(Q)
    nn.vlbm_step_corrected(warm, net, 1, np.full(8, 1e30), 0.1)
    warm.vlbm_destroy()
    before = _free()
    sim = vb.Vlbm(gpu_params(vb, w, "f32"))
    one = sim.population_bytes()
    sim.vlbm_init_fields(Q)
    sim.vlbm_step(3)
    nn.vlbm_step_corrected(sim, net, 5, np.full(8, 1e30), 0.1)
    assert before - _free() < 1.1 * one
    sim.vlbm_step(4)
    assert before - _free() > 1.9 * one
    sim.vlbm_destroy()
    assert before - _free() < 0.1 * one


def test_buffer_is_given_back_and_taken_again(vb, case):  # noqa: F811
    """vlbm_set_passes(0) frees it and steps in place, 1 lets the next call take it again; the
    populations are those of a context left alone, bit for bit."""
    w, Q = case
    print("case buffer given back", flush=True)
    sims = [vb.Vlbm(gpu_params(vb, w, "f32")) for _ in range(2)]
    one = sims[0].population_bytes()
    assert sims[0].pass_bytes() == one
    for sim in sims:
        sim.vlbm_init_fields(Q)
        sim.vlbm_step(8)
    before = _free()
    sims[0].vlbm_set_passes(False)
    assert _free() - before > 0.9 * one
    sims[0].vlbm_step(8)
    assert _free() - before > 0.9 * one
    sims[0].vlbm_set_passes(True)
    sims[0].vlbm_step(8)
    assert _free() - before < 0.1 * one
    sims[1].vlbm_step(16)
    assert np.array_equal(sims[0].vlbm_get_populations()[0], sims[1].vlbm_get_populations()[0])
    with pytest.raises(vb.VlbmError):
        vb._check(vb.lib().vlbm_set_passes(sims[0].ctx, 2), sims[0].ctx)


def test_adopted_buffer_stays_alone(vb, case):  # noqa: F811
    """A context on the caller's buffer steps in place until the caller turns passes on."""
    import torch
    w, Q = case
    print("case adopted buffer", flush=True)
    own = vb.Vlbm(gpu_params(vb, w, "f32"))
    one = own.population_bytes()
    pop = torch.empty(one, dtype=torch.uint8, device="cuda")
    sim = vb.Vlbm(gpu_params(vb, w, "f32"), pop_tensor=pop)
    before = _free()
    sim.vlbm_init_fields(Q)
    sim.vlbm_step(8)
    assert before - _free() < 0.1 * one
    sim.vlbm_set_passes(True)
    sim.vlbm_step(8)
    assert before - _free() > 0.9 * one
    own.vlbm_init_fields(Q)
    own.vlbm_step(16)
    assert np.array_equal(sim.vlbm_get_populations()[0], own.vlbm_get_populations()[0])
