"""A state that raises a diagnostic flag in every wave (NaN everywhere) steps
about as fast as an ordinary one: a flag that is up is read, not set again.
With an atomic of every wave on the flag's address the step took more than
three times as long.  And the flag comes up again after it was read and reset."""
import pytest

from paper_2004_08503_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def step_time(sv, u, dt):
    for _ in range(20):
        sv.step(u, dt)
    times = []
    for _ in range(9):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(30):
            sv.step(u, dt)
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b))
    return sorted(times)[4]


@pytest.mark.parametrize("curved", [False, True])
def test_a_flagged_step_is_no_slower(curved):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2004_08503_amd import idp_dg
    wl = W.euler_2d(n=160, p=4)
    prob = wl.prob.replace(limiter=W.TARGET)
    if curved:
        prob = prob.replace(coords=W.perturbed_coords(prob))
    sv = idp_dg.Solver(prob)
    u = torch.from_numpy(wl.u0.copy()).cuda()
    plain = step_time(sv, u, 0.0)       # a zero step keeps the state
    assert not sv.diagnostics()["bad_input"]
    u.fill_(float("nan"))
    flagged = step_time(sv, u, 0.0)
    assert sv.diagnostics()["bad_input"]
    assert flagged < 2.0 * plain, (flagged, plain)
    assert not sv.diagnostics()["bad_input"]   # reading resets it
    sv.step(u, 0.0)
    assert sv.diagnostics()["bad_input"]
    sv.close()
