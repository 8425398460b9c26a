"""The high-order metric terms of a curved mesh (host) against the derivative
of the same interpolant in extended precision.

Every term is a derivative along a node line, sum_c D(a, c) (x_c - x_a): the
difference of two coordinates, the entry D(a, c), the product and the sum are
rounded once each, so a term is off by at most (p + 5) eps sum_c |D(a, c)|
|x_c - x_a|, whatever the mesh's distance from the origin."""
import numpy as np
import pytest

from paper_2004_08503_amd import idp_dg, workloads as W

L = np.longdouble


def derivative_matrix(p):
    """Gauss-Lobatto derivative matrix on [0, 1] in extended precision."""
    x = np.array([-np.cos(np.pi * k / p) for k in range(p + 1)], dtype=L)

    def leg(n):
        a, b = np.ones_like(x), x
        for k in range(2, n + 1):
            a, b = b, ((2 * k - 1) * x * b - (k - 1) * a) / k
        return (a, b) if n else (0 * x, a)

    for _ in range(20):   # roots of P_{p+1} - P_{p-1} inside, whose derivative is (2p+1) P_p
        pm1 = leg(p - 1)[1] if p > 1 else np.ones_like(x)
        pp, pp1 = leg(p + 1)
        x[1:-1] -= ((pp1 - pm1) / ((2 * p + 1) * pp))[1:-1]
    x[0], x[-1] = -1, 1
    xi = (x + 1) / 2
    bw = np.array([1 / np.prod([xi[j] - xi[m] for m in range(p + 1) if m != j]) for j in range(p + 1)], dtype=L)
    D = np.array([[bw[j] / bw[i] / (xi[i] - xi[j]) if i != j else L(0) for j in range(p + 1)] for i in range(p + 1)])
    return D   # without its diagonal: used on differences


@pytest.mark.parametrize("shift", [0.0, 100.0])
@pytest.mark.parametrize("p,n", [(1, 20), (2, 30), (3, 80), (4, 40), (7, 40), (8, 36)])
def test_derivatives(p, n, shift):
    prob = W.Problem(dim=2, nx=n, ny=n, p=p, eq=W.EULER)
    xy = np.ascontiguousarray(W.perturbed_coords(prob) + shift)
    met = idp_dg.mesh_metric(prob, xy)
    n1 = p + 1
    D = derivative_matrix(p)
    c = xy.reshape(2, n * n, n1, n1).astype(L)
    dxi = c[:, :, :, None, :] - c[:, :, :, :, None]               # [.., b, a, c] = x(c, b) - x(a, b)
    deta = c.transpose(0, 1, 3, 2)[:, :, :, None, :] - c.transpose(0, 1, 3, 2)[:, :, :, :, None]   # [.., a, b, c]
    xi, exi = (D * dxi).sum(-1), (abs(D) * abs(dxi)).sum(-1)
    eta, eeta = (D * deta).sum(-1).swapaxes(-1, -2), (abs(D) * abs(deta)).sum(-1).swapaxes(-1, -2)
    want = np.stack([eta[1], -eta[0], -xi[1], xi[0]]).reshape(4, -1)
    size = np.stack([eeta[1], eeta[0], exi[1], exi[0]]).reshape(4, -1)
    bound = (p + 5) * 2.0 ** -53 * size
    err = abs(met[:4] - want)
    print("p %d, %d^2 elements, shift %g: worst %.1e of the largest term, %.2f of the bound" % (
        p, n, shift, float(err.max() / abs(want).max()), float((err / np.maximum(bound, L(1e-300))).max())))
    assert (err <= bound).all()
