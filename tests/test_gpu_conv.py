"""The convolution kernels at the edges of how they share out work."""
import numpy as np
import pytest

from oracle import conv_ref as C
from test_gpu_nn import bm, cm, env, make_net, rand_params, rel_l2  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nz", [1, 2, 3, 5, 9])
@pytest.mark.parametrize("nx,ny", [(16, 16), (48, 32)])
def test_forward_3d_z_shares(env, nx, ny, nz):  # noqa: F811
    """3x3x3 layers walk up each tile column in shares of at least four slices: depths of one
    to three slices (every neighbour wraps), one past a share and two past two shares, against
    the oracle at the BF16 tolerance of the other forward tests."""
    torch = env[0]
    rng = np.random.default_rng(7 + nz)
    params = rand_params(rng, 3, dim=3)
    X = rng.normal(size=(1, 8, nz, ny, nx))
    net = make_net(env, 3, params, dim=3)
    print('case z shares', nx, ny, nz, flush=True)
    x = cm(torch, X)
    out = torch.full_like(x, 1e30)
    net.vlbm_nn_forward(x, out)
    want = C.Net(params, layers=3, quantize=True, dim=3).forward(X)
    assert rel_l2(bm(out), want) <= 1e-2
