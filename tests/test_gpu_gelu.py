"""The network's GELU: the activations are those of the exact form z / 2 (1 + erf(z / sqrt 2))
in FP32, rounded to BF16, for every z -- finite, infinite and not a number."""
import numpy as np
import pytest

import oracle.conv_ref as C
from test_gpu_nn import env, flat  # noqa: F401

pytestmark = pytest.mark.gpu

# 3x3 networks of 2 layers run a launch per layer, of 3 and 4 layers all in one; 3x3x3
NETS = [(2, 2), (2, 3), (2, 4), (3, 2)]


@pytest.mark.parametrize("dim,layers", NETS)
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_infinite_activation(env, dim, layers, value):  # noqa: F811
    """Positive weights and an input of one infinite value: GELU(+inf) = +inf passes on through
    every layer; GELU(-inf) = -inf x 0 and that of a NaN are NaN.  The cells within reach of
    the input, one further per layer, hold the value, all others finite ones."""
    torch, _, nn = env
    net = nn.Net(8, 32, layers, stream=torch.cuda.current_stream().cuda_stream, dim=dim)
    net.vlbm_nn_set_weights(np.full(net.vlbm_nn_num_params(), 0.01, np.float32))
    shape = (16, 32, 32) if dim == 3 else (32, 32)
    X = torch.ones((8, 1) + shape, dtype=torch.float32, device="cuda")
    at = tuple(n // 2 for n in shape)
    X[(3, 0) + at] = value
    Y = torch.zeros_like(X)
    print("case infinite activation", dim, layers, value, flush=True)
    net.vlbm_nn_forward(X, Y)
    got = Y.cpu().numpy()[:, 0]
    near = np.max([np.abs(g - c) for g, c in zip(np.indices(shape), at)], axis=0) <= layers
    near = np.broadcast_to(near, got.shape)
    assert np.isfinite(got[~near]).all()
    assert (got[near] == np.inf).all() if value == np.inf else np.isnan(got[near]).all()


@pytest.mark.parametrize("field", ["normal", "patterns"])
def test_activation_equals_the_exact_form(env, field):  # noqa: F811
    """Two layers that pass single hidden channels through: the first makes z = w x + b of one
    input (w x exact in FP32, one rounding), the second hands eight of the 32 activations on.
    x: normally distributed, and every BF16 pattern up to 2^60.  Two million z each."""
    torch, _, nn = env
    rng = np.random.default_rng(5)
    n = 256
    if field == "normal":
        x = C.bf16_round(2.0 * rng.standard_normal((n, n))).astype(np.float32)
    else:
        x = (np.arange(n * n, dtype=np.uint32) << 16).view(np.float32).reshape(n, n).copy()
        x[~(np.abs(x) <= 2.0 ** 60)] = 0.0
    X = torch.zeros((8, 1, n, n), dtype=torch.float32, device="cuda")
    X[0, 0] = torch.from_numpy(x).cuda()
    w = C.bf16_round(rng.uniform(0.5, 2.0, 32)).astype(np.float32)
    b = (0.3 * rng.standard_normal(32)).astype(np.float32)
    print("case activation", field, flush=True)
    for part in range(4):
        (W1, b1), (W2, b2) = [(np.zeros(Ws), np.zeros(bs)) for Ws, bs in C.Net.shapes(8, 32, 2)]
        W1[:, 0, 1, 1], b1[:] = w, b
        for o in range(8):
            W2[o, 8 * part + o, 1, 1] = 1.0
        net = nn.Net(8, 32, 2, stream=torch.cuda.current_stream().cuda_stream)
        net.vlbm_nn_set_weights(flat([(W1, b1), (W2, b2)]))
        Y = torch.empty_like(X)
        net.vlbm_nn_forward(X, Y)
        for o in range(8):
            z = X[0, 0] * float(w[8 * part + o]) + float(b[8 * part + o])
            want = (0.5 * z * (1.0 + torch.erf(z * 0.70710678118654752))).bfloat16().float()
            bad = Y[o, 0] != want
            assert not bool(bad.any()), (int(bad.sum()), z[bad][:4].tolist(), Y[o, 0][bad][:4].tolist(), want[bad][:4].tolist())
