"""Linear advection: the low-order state stays between its bar states (the
node's own value and its upwind neighbours') to rounding of those values, not
of a larger downwind neighbour's: the low-order flux is the upwind flux.  Every
node's value is drawn over sixty decades.  A face flux, the node's update and
the bounds are six roundings, each of at most the larger bound."""
import numpy as np
import pytest

from paper_2004_08503_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
EPS = 2.0 ** -53


@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("kind", ["1-D", "2-D", "rotation"])
@pytest.mark.parametrize("p", [1, 3, 6])
def test_low_order_state_within_its_bounds(kind, p, sign):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2004_08503_amd import idp_dg
    if kind == "rotation":
        prob = W.Problem(dim=2, nx=13, ny=11, p=p, eq=W.ADVECTION_FIELD, limiter=W.LOW)
        vr, vc = W.rotation_lines(prob, omega=2.0 * sign)
        prob = prob.replace(vrows=vr, vcols=vc)
    else:
        d = int(kind[0])
        prob = W.Problem(dim=d, nx=21 if d == 1 else 9, ny=1 if d == 1 else 7, p=p, eq=W.ADVECTION,
                         vel=(0.7 * sign, -0.3 * sign), limiter=W.LOW)
    rng = np.random.default_rng(8)
    u = torch.from_numpy(10.0 ** rng.uniform(-60, 0, (1, prob.num_nodes))).cuda()
    sv = idp_dg.Solver(prob)
    out = sv.empty()
    tr = sv.stage_trace(None, u, out, 0.9 * sv.max_dt(u), 0)
    lo, hi = tr[0], tr[1]
    assert bool((out[0] >= lo - 6 * EPS * hi).all()) and bool((out[0] <= hi * (1 + 6 * EPS)).all())
    assert not sv.diagnostics()["low_order_violation"]
    sv.close()


@pytest.mark.parametrize("p,n,vel", [(1, 12, (1.0, 0.5)), (3, 9, (0.7, -0.3)), (3, 9, (1.0, 0.0)), (6, 7, (-0.7, 0.3))])
def test_low_order_state_within_its_bounds_curved(p, n, vel):
    """On a curved mesh the two sides of a subcell face may have different
    coefficients, so both states count; the downwind one by lambda minus its
    coefficient, which is exactly 0 on element faces and never negative.  A
    positive state stays positive, and no node leaves its bounds by the 1e-12
    of the larger one that the violation flag allows."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2004_08503_amd import idp_dg
    prob = W.Problem(dim=2, nx=n, ny=n, p=p, eq=W.ADVECTION, limiter=W.LOW, vel=vel)
    prob = prob.replace(coords=W.perturbed_coords(prob))
    rng = np.random.default_rng(8)
    u = torch.from_numpy(10.0 ** rng.uniform(-60, 0, (1, prob.num_nodes))).cuda()
    sv = idp_dg.Solver(prob)
    out = sv.empty()
    tr = sv.stage_trace(None, u, out, 0.9 * sv.max_dt(u), 0)
    room = torch.minimum(tr[1] - out[0], out[0] - tr[0])
    off = int((room < -1e-12 * torch.maximum(tr[0].abs(), tr[1].abs())).sum())
    assert off == 0 and bool((out >= 0.0).all())
    assert not sv.diagnostics()["low_order_violation"]
    sv.close()


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("a,b", [(0, 0), (3, 3), (0, 2), (1, 2)])
@pytest.mark.parametrize("kind", ["1-D", "2-D", "rotation"])
def test_a_non_finite_node_reaches_its_neighbours(kind, a, b, value):
    """A NaN or infinite node spoils the lines of its element (whose
    high-order fluxes hold it) and the nodes beyond its element's faces,
    upwind and downwind alike, as the flux 1/2 (F_L + F_R) - lambda/2 (u_R -
    u_L) does; every other node stays finite."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2004_08503_amd import idp_dg
    p, nx, ny = 3, 13, 1 if kind == "1-D" else 11
    if kind == "rotation":
        prob = W.Problem(dim=2, nx=nx, ny=ny, p=p, eq=W.ADVECTION_FIELD)
        vr, vc = W.rotation_lines(prob, omega=2.0)
        prob = prob.replace(vrows=vr, vcols=vc)
    else:
        prob = W.Problem(dim=int(kind[0]), nx=nx, ny=ny, p=p, eq=W.ADVECTION, vel=(0.7, -0.3))
    n1, d, ex, ey = p + 1, prob.dim, 4, 0 if kind == "1-D" else 3
    b = b if d == 2 else 0

    def node(ex, ey, a, b):
        return (ey * nx + ex) * n1 ** d + b * n1 + a

    want = {node(ex, ey, c, b) for c in range(n1)}
    if a in (0, p):
        want.add(node(ex + (1 if a else -1), ey, p - a, b))
    if d == 2:
        want |= {node(ex, ey, a, c) for c in range(n1)}
        if b in (0, p):
            want.add(node(ex, ey + (1 if b else -1), a, p - b))
    u = torch.from_numpy(np.random.default_rng(1).uniform(0, 1, (1, prob.num_nodes))).cuda()
    u[0, node(ex, ey, a, b)] = value
    sv = idp_dg.Solver(prob)
    out = sv.empty()
    sv.stage(None, u, out, 1e-3, 0)
    assert set(torch.nonzero(~torch.isfinite(out[0])).flatten().tolist()) == want
    sv.close()
