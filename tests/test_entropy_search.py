"""The entropy search of a subcell face (host build of the kernel's
functions) against the supremum in long double: sup { t in [0, U] :
u^L + t P has Phi >= 0 }.

What the kernel promises is a computed-admissible point within tol =
1e-14 max|u^L| / max|P| below the supremum.  Phi is evaluated in doubles, as
the difference of terms no larger than max|u^L| = E with at most 16 roundings
between them, so a computed root may lie off by delta = 16 eps E / |Phi'|:
the bounds below are t* - tol - delta <= t <= t* + delta."""
import numpy as np
import pytest

import host_math

DRIVER = r"""
template <int GN> static void faces(double g, const double* r, long n, double* t) {
  for (long i = 0; i < n; ++i, r += 10) t[i] = entropy_root_face<2, GN>(r, r + 4, r[8], r[9], 0.0, phys(g));
}
extern "C" void search(int gn, double g, const double* r, long n, double* t) {
  if (gn == 5) faces<5>(g, r, n, t);
  else if (gn == 3) faces<3>(g, r, n, t);
  else faces<0>(g, r, n, t);
}
"""
NAMES = ["ipow_c", "root_step", "inv_root", "rcp_nr", "pow_pos", "PhiVal", "phi_at", "admissible",
         "entropy_root_face"]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return host_math.build(str(tmp_path_factory.mktemp("search")), NAMES, DRIVER)


def segments(rng, n, gamma, size):
    """Records (u^L, P, U = 1, K_min) with u^L admissible: random states at
    rest to Mach 3, K_min below their own K by a relative 1e-6 to 0.5, and
    corrections of relative size `size`."""
    rho, p = 10 ** rng.uniform(-1, 1, n), 10 ** rng.uniform(-1, 1, n)
    mach, th = rng.uniform(0, 3, n), rng.uniform(0, 2 * np.pi, n)
    q = mach * np.sqrt(gamma * p / rho)
    u = np.stack([rho, rho * q * np.cos(th), rho * q * np.sin(th), p / (gamma - 1) + 0.5 * rho * q * q], 1)
    P = rng.standard_normal((n, 4)) * size * np.abs(u).max(1)[:, None]
    km = p * rho ** -gamma * (1 - 10 ** rng.uniform(-6, -0.3, n))
    return np.concatenate([u, P, np.ones((n, 1)), km[:, None]], 1)


def phi(r, t, gamma):
    """Phi and its t-derivative along the records, in long double."""
    r, t, g = r.astype(np.longdouble), t.astype(np.longdouble), np.longdouble(gamma)
    v, P = r[:, :4] + t[:, None] * r[:, 4:8], r[:, 4:8]
    rho = np.where(v[:, 0] > 0, v[:, 0], np.longdouble(1))
    ke = (v[:, 1] ** 2 + v[:, 2] ** 2) / (2 * rho)
    kr = r[:, 9] / (g - 1) * rho ** g
    f = np.where(v[:, 0] > 0, v[:, 3] - ke - kr, -np.longdouble(np.inf))
    df = P[:, 3] - (v[:, 1] * P[:, 1] + v[:, 2] * P[:, 2]) / rho + (ke - g * kr) / rho * P[:, 0]
    return f, df


@pytest.mark.parametrize("gn,gamma", [(5, 1.4), (3, 5.0 / 3.0), (0, 1.3)], ids=["7/5", "5/3", "1.3"])
@pytest.mark.parametrize("size", [1.0, 1e-3, 1e-6])
def test_within_the_tolerance(lib, gn, gamma, size):
    rng = np.random.default_rng(11)
    r = segments(rng, 60000, gamma, size)
    f1, _ = phi(r, r[:, 8], gamma)
    r = np.ascontiguousarray(r[f1 < 0])
    t = np.empty(len(r))
    lib.search(gn, host_math.ctypes.c_double(gamma), host_math.ptr(r), host_math.ctypes.c_long(len(r)), host_math.ptr(t))
    lo, hi = np.zeros(len(r), np.longdouble), r[:, 8].astype(np.longdouble)
    for _ in range(64):
        m = (lo + hi) / 2
        ok = phi(r, m, gamma)[0] >= 0
        lo, hi = np.where(ok, m, lo), np.where(ok, hi, m)
    us = np.abs(r[:, :4]).max(1)
    tol = np.maximum(1e-15, 1e-14 * us / np.abs(r[:, 4:8]).max(1))
    slope = np.abs(phi(r, lo, gamma)[1]).astype(float)
    delta = 16 * 2.0 ** -53 * us / np.maximum(slope, 1e-300)
    well = delta < 0.5 * tol   # elsewhere rounding, not the search, decides
    e = (t - lo).astype(float)
    assert well.sum() > 0.2 * len(r) > 400
    worst = (np.abs(e[well]) / (tol + delta)[well]).max()
    print("gamma %.3f size %g: %d faces, worst |t - t*| / (tol + delta) = %.3f" % (gamma, size, well.sum(), worst))
    assert np.all(e[well] <= delta[well]) and np.all(e[well] >= -(tol + delta)[well])
