"""The polynomials of the network's GELU and of its derivative, read from the kernel source and
evaluated in FP32 (fused steps, the exponential correctly rounded), against FP64."""
import os
import re

import numpy as np
import pytest
from scipy.special import ndtr

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_00641_amd", "csrc",
                   "vlbm_nn.hip")


def coefficients(function):
    body = open(SRC).read().split(function + "(", 1)[1].split("\n}\n", 1)[0]
    first = re.search(r"float p = ([-+0-9.e]+)f;", body).group(1)
    return [np.float32(c) for c in [first] + re.findall(r"p = fmaf\(p, a, ([-+0-9.e]+)f\);", body)]


def upper_tail(function, a):
    """2^P(a) in FP32: the polynomial's fused steps round once each."""
    c = coefficients(function)
    assert len(c) == {"gelu_grad": 11, "gelu_bf16": 9}[function]
    p = np.full(a.shape, c[0], np.float32)
    for k in c[1:]:
        p = (p.astype(np.float64) * a.astype(np.float64) + float(k)).astype(np.float32)
    return np.exp2(p.astype(np.float64)).astype(np.float32)


def grid():
    rng = np.random.default_rng(0)
    z = np.concatenate([np.linspace(-8.0, 8.0, 400001), rng.standard_normal(400000), rng.uniform(-100.0, 100.0, 50000),
                        [0.0, -0.0, 1e-30, -1e-30]])
    return z.astype(np.float32)


def test_activation_within_its_guard():
    """The value's distance from the exact GELU is below the 1.77e-7 |z| it is stated to keep from
    the erff form, plus that form's own error (erff to an ulp of 1, 1.2e-7 |z| / 2, its argument
    and three products, 6e-8 |z| in all)."""
    z = grid()
    a = np.abs(z)
    v = (np.maximum(z, np.float32(0)).astype(np.float64) - a.astype(np.float64) * upper_tail("gelu_bf16", a)).astype(np.float32)
    exact = z.astype(np.float64) * ndtr(z.astype(np.float64))
    assert np.all(np.abs(v - exact) <= (1.77e-7 + 0.6e-7 + 0.6e-7) * a)


def test_derivative_error():
    """Phi(z) + z phi(z): 1.3e-7 at most on [-8, 8], as stated, and beyond."""
    z = grid()
    a = np.abs(z)
    h = upper_tail("gelu_grad", a)
    cdf = np.where(z < 0, h, np.float32(1) - h)
    phi = (np.float32(0.39894228040143268) * np.exp2((z * z * np.float32(-0.72134752044448170)).astype(np.float64))).astype(np.float32)
    got = (z.astype(np.float64) * phi + cdf).astype(np.float32)
    zz = z.astype(np.float64)
    exact = ndtr(zz) + zz * np.exp(-0.5 * zz * zz) / np.sqrt(2.0 * np.pi)
    assert np.abs(got - exact).max() <= 1.35e-7


@pytest.mark.parametrize("function", ["gelu_grad", "gelu_bf16"])
def test_tail_falls_beyond_the_fit(function):
    a = np.geomspace(5.0, 3e38, 200000).astype(np.float32)
    with np.errstate(over="ignore"):
        h = upper_tail(function, a)
    assert np.all(np.diff(h) <= 0.0) and h[a > 20.0].max() == 0.0
