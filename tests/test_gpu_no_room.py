"""A node without room for its corrections has the limiter coefficient 0,
not a tiny one: Zalesak's ratio of the room to the sum of the corrections is
0, or at least a rounding of the state over that sum, and 1 without
corrections.  (A coefficient of 1e-308 puts subnormal values where the state is
zero.)  Data of zeros and ones: what a stage leaves that is not zero is a
rounding, 1e-17, or more, and Burgers' flux squares it at most once in each of
the two stages that follow, 1e-68."""
import numpy as np
import pytest

from paper_2004_08503_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def problem(kind, lim):
    if kind == "1-D advection":
        prob = W.Problem(dim=1, nx=50, ny=1, p=4, eq=W.ADVECTION, vel=(1.0, 0.0), limiter=lim)
    elif kind == "Burgers":
        prob = W.Problem(dim=2, nx=17, ny=13, p=3, eq=W.BURGERS, vel=(1.0, 1.0), limiter=lim)
    else:
        prob = W.Problem(dim=2, nx=19, ny=16, p=3, eq=W.ADVECTION_FIELD, limiter=lim)
        vr, vc = W.rotation_lines(prob)
        prob = prob.replace(vrows=vr, vcols=vc)
    n1 = prob.p + 1
    u = np.zeros((prob.ny, prob.nx) + ((n1, n1) if prob.dim == 2 else (n1,)))
    u[prob.ny // 4:prob.ny // 2 + 1, prob.nx // 4:prob.nx // 2] = 1.0   # a block of elements, its edge on element faces
    return prob.replace(gmin=0.0, gmax=1.0), u.reshape(1, -1)


@pytest.mark.parametrize("lim", [W.SUBCELL, W.SUBCELL_SI, W.ELEMENTWISE], ids=["subcell", "si", "elementwise"])
@pytest.mark.parametrize("kind", ["1-D advection", "Burgers", "rotation"])
def test_coefficients_are_zero_or_real(kind, lim):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2004_08503_amd import idp_dg
    prob, u0 = problem(kind, lim)
    sv = idp_dg.Solver(prob)
    u = torch.from_numpy(u0).cuda()
    dt = 0.2 * sv.max_dt(u)
    tr = sv.stage_trace(None, u, sv.empty(), dt, 0)
    az, al = tr[3], tr[4]
    assert not bool(((az > 0) & (az < 1e-200)).any()) and not bool(((al > 0) & (al < 1e-200)).any())
    assert float(az.min()) >= 0 and float(az.max()) <= 1
    sv.step(u, dt)
    a = u.abs()
    assert not bool(((a > 0) & (a < 1e-200)).any()), float(a[a > 0].min())
    assert bool((az == 1).any()) and bool((u == 0).any())
    sv.close()
