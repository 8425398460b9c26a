"""The admissibility screen of a generic gamma (host build): a state that it
certifies lies inside the admissible set by at least eight times the error of
its single-precision logarithms.

With l = log2 w - (gamma+1) log2 rho, Phi >= 0 <=> l >= 0.  Rounding w and rho
to single precision moves each log2 by 2^-24 / ln 2 = 8.6e-8, the one of rho
gamma + 1 <= 8/3 times: 3.2e-7 together; the logarithms themselves add an ulp
of their values, 1.2e-7 |.|.  So a certified state needs l >= 8 (3.2e-7 + 1.2e-7
(|log2 w| + |(gamma+1) log2 rho|)) less the error itself."""
import ctypes

import numpy as np
import pytest

import host_math

DRIVER = r"""
extern "C" void screen(double g, const double* r, long n, int* o) {
  for (long i = 0; i < n; ++i, r += 10) o[i] = surely_admissible<2, 0>(r[8], r, r + 4, phys(g).gsure / r[9], phys(g));
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return host_math.build(str(tmp_path_factory.mktemp("screen")), ["ipow_c", "surely_admissible"], DRIVER)


@pytest.mark.parametrize("scale", [1.0, 1e-3, 1e4])
@pytest.mark.parametrize("gamma", [1.2, 1.3, 1.6])
def test_margin(lib, gamma, scale):
    rng = np.random.default_rng(5)
    n = 400000
    rho, p = scale * rng.uniform(0.7, 1.4, n), 10 ** rng.uniform(-1, 1, n)
    q = rng.uniform(0, 2, n) * np.sqrt(gamma * p / rho)
    th = rng.uniform(0, 2 * np.pi, n)
    u = np.stack([rho, rho * q * np.cos(th), rho * q * np.sin(th), p / (gamma - 1) + 0.5 * rho * q * q], 1)
    # K_min around the state's own K: just admissible, just not
    d = rng.choice([-1, 1], n) * 10 ** rng.uniform(-8, -2.5, n)
    km = p * rho ** -gamma * (1 - d)
    r = np.ascontiguousarray(np.concatenate([u, np.zeros((n, 4)), np.ones((n, 1)), km[:, None]], 1))
    o = np.empty(n, np.int32)
    lib.screen(ctypes.c_double(gamma), host_math.ptr(r), ctypes.c_long(n), host_math.ptr(o))
    L = np.longdouble
    w = (L(1) * r[:, 3] * r[:, 0] - (L(1) * r[:, 1] ** 2 + L(1) * r[:, 2] ** 2) / 2) * (L(gamma) - 1) / r[:, 9]
    a, b = np.log2(w), (L(gamma) + 1) * np.log2(L(1) * r[:, 0])
    err = 3.2e-7 + 1.2e-7 * (np.abs(a) + np.abs(b))
    ok = o == 1
    assert ok.sum() > n // 20 and not ok.all()
    worst = ((a - b)[ok] / err[ok]).min()
    print("gamma %.1f scale %g: least margin of a certified state %.2f errors" % (gamma, scale, worst))
    assert worst >= 7.0
    # and the screen still settles what lies well inside
    assert o[(a - b) > 40 * err].all()
