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


@pytest.mark.parametrize("layers", [3, 4])
@pytest.mark.parametrize("B,ny,nx", [(257, 16, 16), (43, 32, 48), (2, 192, 192)])
def test_whole_network_equals_layers(env, layers, B, ny, nx):  # noqa: F811
    """Lattices of at most 256 tiles run the whole network in one launch, larger ones (here
    the batch) a launch per layer: the same products in the same order, so the same bits."""
    torch, _, nn = env
    print("case whole network", layers, B, ny, nx, flush=True)
    net = nn.Net(8, 32, layers, stream=torch.cuda.current_stream().cuda_stream)
    rng = np.random.default_rng(layers)
    net.vlbm_nn_set_weights((0.15 * rng.standard_normal(net.vlbm_nn_num_params())).astype(np.float32))
    net.vlbm_nn_set_norm(rng.standard_normal(8), 0.5 + rng.random(8), rng.standard_normal(8), 0.5 + rng.random(8))
    X = torch.from_numpy(rng.standard_normal((8, B, ny, nx)).astype(np.float32)).cuda()
    whole = torch.empty_like(X)
    net.vlbm_nn_forward(X, whole)
    for b in range(0, B, max(1, B // 3)):
        x = X[:, b:b + 1].contiguous()
        y = torch.empty_like(x)
        net.vlbm_nn_forward(x, y)
        assert torch.equal(y, whole[:, b:b + 1]), b
