"""Pointwise Euler physics at the edges of its arguments (host build of the
kernel's functions): zero, infinite, negative and NaN densities and pressures
give what IEEE square roots, divisions and powers give, so that a bad state
reaches its neighbours in one way only.  The integer-gamma roots are NaN
outside (0, inf).  A NaN never enters a minimum or maximum, so a side of a
face whose wave speed is NaN does not count.

Finite values: X and K are products of at most eight factors within 2 ulps
each, so 16 eps relative; lambda loses at most as much again in each of its
three stages (x3 p*, the root, the sum), 64 eps of the larger terms."""
import ctypes
import itertools
import math

import numpy as np
import pytest

import host_math

DRIVER = r"""
template <int GN, bool WK> static void aux(double g, const double* U, long n, double* o) {
  for (long i = 0; i < n; ++i, U += 3, o += 6) {
    bool bad;
    double K = -7.0, p;
    euler_aux<1, GN, WK>(U, phys(g), o, K, p, bad);
    o[4] = K;
    o[5] = p;
  }
}
extern "C" void aux_(int gn, int wk, double g, const double* U, long n, double* o) {
  if (gn == 5) wk ? aux<5, true>(g, U, n, o) : aux<5, false>(g, U, n, o);
  else wk ? aux<0, true>(g, U, n, o) : aux<0, false>(g, U, n, o);
}
extern "C" void lambda_(int gn, double g, const double* a, long n, double* o) {
  for (long i = 0; i < n; ++i, a += 7)
    o[i] = gn == 5 ? euler_lambda<5>(a[0], a[1], a[2], a[3], a[4], a[5], a[6], phys(g))
                   : euler_lambda<0>(a[0], a[1], a[2], a[3], a[4], a[5], a[6], phys(g));
}
extern "C" void pow_(const double* x, const double* y, long n, double* o) {
  for (long i = 0; i < n; ++i) o[i] = pow_pos(x[i], y[i]);
}
"""
NAMES = ["ipow_c", "root_step", "inv_root", "sqrt_nr", "sqrt_ge1", "rcp_nr", "sqrt_any", "rcp_any", "pow_pos",
         "euler_aux", "euler_lambda"]
INF, NAN, EPS = math.inf, math.nan, 2.0 ** -53


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return host_math.build(str(tmp_path_factory.mktemp("special")), NAMES, DRIVER)


def call(f, *args):
    f(*[host_math.ptr(a) if isinstance(a, np.ndarray) else a for a in args])


def same(got, want, tol, what):
    for g, w, k in zip(got.ravel(), np.asarray(want, float).ravel(), what):
        ok = (math.isnan(g) and math.isnan(w)) or g == w or (math.isfinite(w) and abs(g - w) <= tol * abs(w))
        assert ok, (k, g, w)


def ieee(f, *a):
    with np.errstate(all="ignore"):
        return float(f(*[np.float64(v) for v in a]))


def div(a, b):
    return ieee(np.divide, a, b)


def power(x, y):
    return ieee(np.power, x, y)


def root(x, n, k):
    """x^(-k/n), NaN outside (0, inf)."""
    return float(np.longdouble(x) ** (np.longdouble(-k) / n)) if 0.0 < x < INF else NAN


def test_powers(lib):
    xs = [0.0, 5e-324, 1e-310, 1e-300, 1e-3, 1.0, 7.0, 1e300, INF, -1e-300, -1.0, -INF, NAN]
    ys = (-1.3, -0.115, 0.115, 1.3, 8.67)
    # finite arguments with results of normal magnitude, and every other argument
    c = [(x, y) for x in xs for y in ys if not 0.0 < x < INF or 1e-300 < power(x, y) < 1e300]
    x, y = np.array([a for a, _ in c]), np.array([b for _, b in c])
    o = np.empty(len(c))
    call(lib.pow_, x, y, ctypes.c_long(len(c)), o)
    same(o, [power(a, b) if 0.0 < a < INF else NAN for a, b in c], 4 * EPS, c)


@pytest.mark.parametrize("with_k", [0, 1])
@pytest.mark.parametrize("gn,gamma", [(5, 1.4), (0, 1.3)])
def test_node_state(lib, gn, gamma, with_k):
    # densities and energies whose pressure is exactly zero, negative, infinite or ordinary
    c = list(itertools.product([0.0, 1.0, 3.0, -2.0, 1e-200, 1e200, INF, NAN], [0.0, 2.0, -3.0],
                               [0.0, 0.5, 2.0, 1e3, -1.5, INF, NAN]))
    U = np.array(c)
    o = np.empty((len(c), 6))
    call(lib.aux_, gn, with_k, ctypes.c_double(gamma), U, ctypes.c_long(len(c)), o)
    ex = (gamma - 1) / (2 * gamma)
    want = []
    for rho, m, E in c:
        ri = root(rho, 5, 5) if gn and with_k else div(1.0, rho)
        with np.errstate(all="ignore"):
            p = float(np.float64(gamma - 1) * (np.float64(E) - np.float64(0.5 * m * m) * np.float64(ri)))
            s = ieee(np.sqrt, gamma * p * ri)
            x3 = root(p, 7, 1) if gn else power(p, -ex)
            ip = root(p, 7, 7) if gn else div(1.0, p)
            K = -7.0 if not with_k else p * root(rho, 5, 7) if gn else float(np.float64(p) * power(rho, -gamma))
        if not gn and (p == 0.0 or math.isinf(p)):
            ip = NAN   # in no wave speed: the other factors of such a face are NaN
        want.append([ri, s, s * x3, (gamma + 1) / (2 * gamma) * ip, K, p])
    want = np.array(want)
    for q in range(6):
        same(o[:, q], want[:, q], 16 * EPS, [(q,) + k for k in c])


@pytest.mark.parametrize("gn,gamma", [(5, 1.4), (0, 1.3)])
def test_wave_speed_bound(lib, gn, gamma):
    ex, fac = (gamma - 1) / (2 * gamma), (gamma + 1) / (2 * gamma)
    c = []
    for vl, vr in ((0.0, 0.0), (1.0, 1.0), (-2.0, 3.0), (3.0, -2.0)):
        for (cl, xl, zl), (cr, xr, zr) in itertools.product(
                [(1.0, 0.9, 0.8), (0.0, NAN, NAN), (1e-150, 1e-130, 1e300), (INF, NAN, NAN), (NAN, NAN, NAN)], repeat=2):
            c.append((vl, vr, cl, cr, xl + xr, zl, zr))
        c.append((vl, vr, 1e40, 1e40, 1e-5, 1e290, 1.0))   # p*/p past the largest double
    a = np.array(c)
    o = np.empty(len(c))
    call(lib.lambda_, gn, ctypes.c_double(gamma), a, ctypes.c_long(len(c)), o)

    def mx(x, y):   # the other one for a NaN
        return y if math.isnan(x) else x if math.isnan(y) else max(x, y)

    want = []
    for vl, vr, cl, cr, x2, zl, zr in c:
        num = mx(cl + cr - 0.5 * (gamma - 1) * (vr - vl), 0.0)
        base = num / x2 if 0.0 < x2 < INF and num < INF else NAN
        ps = power(base, 7.0 if gn else 1.0 / ex)
        tl, tr = (ieee(np.sqrt, mx(ieee(np.multiply, ps, z) + 1.0 - fac, 1.0)) for z in (zl, zr))
        want.append(mx(mx(mx(-vl + ieee(np.multiply, cl, tl), vr + ieee(np.multiply, cr, tr)), 0.0), 0.0))
    assert any(w == INF for w in want) and any(w == 1.0 for w in want)
    same(o, want, 64 * EPS, c)


def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2004_08503_amd import idp_dg, workloads as W
    return torch, idp_dg, W


@pytest.mark.gpu
@pytest.mark.parametrize("gamma", [1.4, 5.0 / 3.0, 1.3])
def test_pressureless_flow_has_its_velocity_as_wave_speed(gamma):
    torch, idp_dg, W = _gpu()
    prob = W.Problem(dim=1, nx=6, ny=1, p=3, eq=W.EULER, gamma=gamma)
    u = torch.tensor([1.0, 1.0, 0.5], dtype=torch.float64, device="cuda")[:, None].repeat(1, prob.num_nodes)
    sv = idp_dg.Solver(prob)
    w0 = 1.0 / 12.0   # end weight of the four-point rule on [0, 1]
    assert sv.max_dt(u.contiguous()) == pytest.approx(0.5 * w0 / 6, rel=1e-14)
    sv.close()


@pytest.mark.gpu
@pytest.mark.parametrize("gamma", [1.4, 5.0 / 3.0, 1.3])
def test_a_bad_node_bounds_no_neighbour(gamma):
    """A node of negative density has no K; its neighbours' K_min is theirs
    (the formula p rho^-gamma to 32 roundings, as in the parity tests)."""
    torch, idp_dg, W = _gpu()
    prob = W.Problem(dim=1, nx=6, ny=1, p=3, eq=W.EULER, gamma=gamma)
    rng = np.random.default_rng(3)
    n = prob.num_nodes
    rho, v, p = rng.uniform(0.5, 2.0, n), rng.uniform(-1, 1, n), rng.uniform(0.5, 2.0, n)
    K = p * rho ** -gamma
    u = np.stack([rho, rho * v, p / (gamma - 1) + 0.5 * rho * v * v])
    bad = 9
    u[0, bad], K[bad] = -1.0, INF
    want = np.minimum(K, np.minimum(np.roll(K, 1), np.roll(K, -1)))
    sv = idp_dg.Solver(prob)
    ut = torch.from_numpy(u).cuda()
    tr = sv.stage_trace(None, ut, sv.empty(), 1e-3, 0).cpu().numpy()
    ok = np.arange(n) != bad
    assert np.allclose(tr[2][ok], want[ok], rtol=32 * EPS, atol=0)
    assert sv.diagnostics()["bad_input"]
    sv.close()


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny", [(8, 8), (9, 8)])
def test_bound_of_a_nan_state(nx, ny):
    """No node with a wave speed: the bound is +infinity, on a mesh of one
    full tile (whose minimum no second kernel folds) as on one of two."""
    torch, idp_dg, W = _gpu()
    prob = W.Problem(dim=2, nx=nx, ny=ny, p=1, eq=W.BURGERS)
    sv = idp_dg.Solver(prob)
    assert sv.tile_dims == (8, 8)
    u = torch.full((1, prob.num_nodes), NAN, dtype=torch.float64, device="cuda")
    d = torch.zeros(1, dtype=torch.float64, device="cuda")
    sv.max_dt_async(u, d)
    assert sv.max_dt(u) == INF and float(d) == INF
    sv.close()
