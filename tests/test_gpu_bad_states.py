"""What a bad node (flagged as bad input) does to the coefficients around it:
the limiter stays on the safe side.  One node of an otherwise ordinary random
state has a negative energy, or is infinite or NaN."""
import numpy as np
import pytest

import oracle
from paper_2004_08503_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
NAN, INF = float("nan"), float("inf")


def solver(prob):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2004_08503_amd import idp_dg
    return idp_dg.Solver(prob)


def euler_state(prob):
    rng = np.random.default_rng(5)
    n = prob.num_nodes
    rho, p, v = rng.uniform(0.5, 2, n), rng.uniform(0.5, 2, n), rng.uniform(-0.5, 0.5, (prob.dim, n))
    return np.concatenate([rho[None], rho * v, (p / (prob.gamma - 1) + 0.5 * rho * (v * v).sum(0))[None]])


def problem(dim, eq=W.EULER, **kw):
    return W.Problem(dim=dim, nx=7, ny=1 if dim == 1 else 6, p=3, eq=eq, gmin=0.5, gmax=2.0, **kw)


def first_node(prob):
    """of an element with neighbours on all sides"""
    return 3 * 4 if prob.dim == 1 else (2 * prob.nx + 3) * 16


@pytest.mark.parametrize("lim", [W.SUBCELL, W.SUBCELL_SI, W.ELEMENTWISE], ids=["subcell", "si", "elementwise"])
@pytest.mark.parametrize("gamma", [1.4, 5.0 / 3.0, 1.3])
@pytest.mark.parametrize("dim", [1, 2])
def test_negative_energy(dim, gamma, lim):
    """K of the node is negative, and so is rho times its internal energy:
    their ratio is positive and says nothing.  A correction that, taken as far
    as the density allows, leaves Phi below zero by more than the rounding of
    its terms lowers the node's coefficient there too (u^L and the corrections
    are the oracle's)."""
    prob = problem(dim, gamma=gamma, limiter=lim)
    dt, n1, seen = 1e-4, prob.p + 1, 0
    _, w = oracle.gl(prob.p)
    mass = np.tile(w / prob.nx, prob.nx) if dim == 1 else np.tile(np.outer(w, w).ravel() / (prob.nx * prob.ny), prob.nx * prob.ny)
    for pos in ((0, 2) if dim == 1 else (0, 5, 15)):
        u = euler_state(prob)
        bad = first_node(prob) + pos
        u[dim + 1, bad] = -1.0
        sv = solver(prob)
        tr = sv.stage_trace(None, torch.from_numpy(u).cuda(), sv.empty(), dt, 0).cpu().numpy()
        assert sv.diagnostics()["bad_input"]
        sv.close()
        ref = oracle.fe(prob, u, dt, trace=True)[1]
        if lim == W.ELEMENTWISE:
            P = [ref["uH"] - ref["uL"]]
        else:
            P = []
            for k in range(dim):
                c = 2 * dim * dt / mass * ref["rbar"][k]     # to the node's right (above it); 0 on element faces
                step, at = n1 ** k, (np.arange(u.shape[1]) // n1 ** k) % n1
                P += [c, np.where(at > 0, -np.roll(2 * dim * dt * ref["rbar"][k], step, axis=1) / mass, 0.0)]
        for p in P:
            v = ref["uL"] + tr[3] * p
            kin = 0.5 * (v[1:-1] ** 2).sum(0) / v[0]
            kr = tr[2] * v[0] ** gamma / (gamma - 1)
            off = v[-1] - kin - kr < -1e-11 * (abs(v[-1]) + kin + abs(kr))
            seen += int(off[bad])
            assert (tr[4] < tr[3])[off].all(), np.nonzero(off & ~(tr[4] < tr[3]))
    assert seen or dim == 1


@pytest.mark.parametrize("gamma", [1.4, 5.0 / 3.0, 1.3])
def test_nan_corrections_take_nothing(gamma):
    """A NaN momentum makes the corrections of its element line NaN: the
    line's nodes have no admissible part of them, the coefficient 0."""
    prob = problem(2, gamma=gamma)
    u = euler_state(prob)
    n0 = first_node(prob)
    u[1, n0] = NAN
    sv = solver(prob)
    tr = sv.stage_trace(None, torch.from_numpy(u).cuda(), sv.empty(), 1e-4, 0)
    line = tr[4][[n0 + 2, n0 + 3, n0 + 8, n0 + 12]]   # of its row and of its column, past its neighbours
    assert bool((line == 0.0).all()), line
    sv.close()


@pytest.mark.parametrize("curved", [False, True])
@pytest.mark.parametrize("eq", [W.ADVECTION, W.BURGERS])
def test_infinite_corrections_take_nothing(eq, curved):
    """The room over an infinite sum of corrections is 0 (at most the state's
    over the largest double)."""
    prob = problem(2, eq=eq, vel=(0.7, -0.3))
    if curved:
        prob = prob.replace(coords=W.perturbed_coords(prob))
    u = np.random.default_rng(5).uniform(0.1, 1, (1, prob.num_nodes))
    n0 = first_node(prob)
    u[0, n0 + 15] = INF
    sv = solver(prob)
    tr = sv.stage_trace(None, torch.from_numpy(u).cuda(), sv.empty(), 1e-4, 0)
    line = tr[4][[n0 + 13, n0 + 7]]   # a = 1 of its row, b = 1 of its column: finite themselves
    assert bool((line <= 1e-300).all()), line
    sv.close()


@pytest.mark.parametrize("value", [INF, 1e200])
@pytest.mark.parametrize("dim", [1, 2])
def test_energy_past_the_doubles_is_not_smooth(dim, value):
    """The fraction of an infinite energy is not a number, and neither are the
    relaxed bounds: no node of the element takes a correction that is a number."""
    prob = problem(dim, eq=W.ADVECTION, vel=(0.7, -0.3), limiter=W.SUBCELL_SI)
    u = np.random.default_rng(5).uniform(0.5, 2, (1, prob.num_nodes))
    n0, n1 = first_node(prob), 4 ** dim
    u[0, n0 + 1] = value
    sv = solver(prob)
    tr = sv.stage_trace(None, torch.from_numpy(u).cuda(), sv.empty(), 1e-4, 0)
    inside = torch.zeros(prob.num_nodes, dtype=torch.bool, device="cuda")
    inside[n0:n0 + n1] = True
    assert torch.equal(torch.isnan(tr[0]), inside) and torch.equal(torch.isnan(tr[1]), inside)
    far = tr[4][n0 + n1 - 1]   # the element's last node, whose corrections the value reaches by high-order fluxes only
    assert float(far) == 0.0
    sv.close()
