"""The erf approximation of the GELU epilogue (paper_2301_10936_amd/csrc/pit_gemm_dev.hpp, gelu_erf_fast), evaluated
here in numpy float32 with the constants of the kernel, against scipy's erf: the bound the kernel's comment states.  The kernel
evaluates x / 2 + |x| (1/2 - 2^-q / 2) with q as a polynomial in |x|; the first test pins q itself."""
import numpy as np
import pytest
from scipy.special import erf, erfc

C = np.array([1.6278890371, 0.9185093641, 0.1486656219, -0.02959003858, 0.00294415676], dtype=np.float32)


def gelu_kernel_formula(x):
    x = x.astype(np.float32)
    z = np.abs(x) * np.float32(0.70710678118654752)
    with np.errstate(over="ignore", invalid="ignore"):
        acc = np.full_like(z, C[4])
        for k in (3, 2, 1, 0):
            acc = acc * z + C[k]
        q = acc * z
        p = np.exp2(-q.astype(np.float64))
    p[p < 2.0 ** -126] = 0.0                    # the hardware exp2 flushes denormal results to zero
    e = np.float32(1) - p.astype(np.float32)
    return e, np.float32(0.5) * x * (np.float32(1) + np.copysign(e, x))


def test_erf_error_bound_and_tails():
    x = np.linspace(-40.0, 40.0, 2000001)
    e, g = gelu_kernel_formula(x)
    exact_erf = erf(np.abs(x) / np.sqrt(2.0))
    assert np.abs(e - exact_erf).max() <= 7e-7
    exact = 0.5 * x * (1.0 + erf(x / np.sqrt(2.0)))
    assert np.abs(g - exact).max() <= 3e-6
    # far tails: exactly x for large positive, exactly (minus) zero for large negative arguments
    _, t = gelu_kernel_formula(np.array([1e3, 1e6, -9.0, -50.0, -1e4, -1e30]))
    assert t[0] == np.float32(1e3) and t[1] == np.float32(1e6) and np.all(t[2:] == 0.0)
    _, n = gelu_kernel_formula(np.array([np.nan]))
    assert np.isnan(n[0])


D = np.array([1.151091337, 0.4592546821, 0.05256123468, -0.007397509646, 0.0005204583285], dtype=np.float32)


def _fma(a, b, c):
    return (np.float64(a) * np.float64(b) + np.float64(c)).astype(np.float32)


def gelu_kernel(x):
    x = x.astype(np.float32)
    with np.errstate(over="ignore", invalid="ignore", under="ignore"):
        a = np.abs(x)
        p = np.full_like(a, D[4])
        for c in (D[3], D[2], D[1], D[0]):
            p = _fma(p, a, c)
        e = np.exp2(-(a * p).astype(np.float64)).astype(np.float32)
        e[e < 2.0 ** -126] = 0.0
        return _fma(a, _fma(np.float32(-0.5), e, np.float32(0.5)), np.float32(0.5) * x)


def test_gelu_in_the_form_of_the_kernel():
    assert np.allclose(D, C.astype(np.float64) * 0.5 ** (np.arange(1, 6) / 2.0), rtol=1e-7)
    g = np.random.default_rng(1)
    for scale in (0.3, 1.0, 3.0, 10.0):
        x = (g.standard_normal(1 << 18) * scale).astype(np.float32)
        exact = 0.5 * x.astype(np.float64) * (1.0 + erf(x.astype(np.float64) / np.sqrt(2.0)))
        now, before = gelu_kernel(x) - exact, gelu_kernel_formula(x)[1] - exact
        assert np.abs(now).max() <= 3e-6
        assert np.linalg.norm(now) <= np.linalg.norm(before)          # no larger than in the form it replaces
    t = gelu_kernel(np.array([1e3, 1e6, np.inf, -9.0, -50.0, -1e4, -1e30, 0.0, -0.0]))
    assert t[0] == np.float32(1e3) and t[1] == np.float32(1e6) and t[2] == np.inf and np.all(t[3:] == 0.0)
    assert np.all(np.isnan(gelu_kernel(np.array([np.nan, -np.inf]))))  # (-inf: -inf * 0, as in x (1 + erf))


@pytest.mark.parametrize("lo,hi", [(-8, -4), (-4, -1), (-1, -0.1), (-0.1, -1e-3), (-1e-3, -1e-6), (1e-6, 1e-3), (1e-3, 0.1), (0.1, 1), (1, 4), (4, 8)])
def test_no_range_of_arguments_lost_precision(lo, hi):
    """Range by range against x (1 + erf) / 2: near zero and for small negative x too, where a norm over a normal distribution
    sees nothing.  (0.5 %: the coefficients are rounded once more, and a root mean square of 2^18 draws is good to 0.2 %.)"""
    x = (np.random.default_rng(2).random(1 << 18) * (hi - lo) + lo).astype(np.float32)
    d = x.astype(np.float64)
    exact = np.where(d < 0, 0.5 * d * erfc(-d / np.sqrt(2.0)), 0.5 * d * (1.0 + erf(d / np.sqrt(2.0))))
    now, before = gelu_kernel(x) - exact, gelu_kernel_formula(x)[1] - exact
    assert np.linalg.norm(now) <= 1.005 * np.linalg.norm(before)
    assert np.abs(now).max() <= 1.005 * np.abs(before).max()
