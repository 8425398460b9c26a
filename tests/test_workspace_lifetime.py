"""Memory that torch's allocator lends to a handle: its workspace and its
boundary arrays are read and written on the handle's stream (and on that of a
batch that holds it), while the allocator frees them in the order of the
stream they were allocated on.  Every other stream has to be recorded with
the allocator, or close() gives memory away that a queued step still uses."""
import types

import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2004_08503_amd import idp_dg, workloads as W  # noqa: E402


class Tensor(torch.Tensor):
    """A host tensor that passes for a device one and notes its streams."""
    @property
    def is_cuda(self):
        return True

    def record_stream(self, s):
        self.__dict__.setdefault("streams", []).append(s)


@pytest.fixture
def faked(monkeypatch):
    made = []

    def empty(n, dtype=None, device=None):
        made.append(torch.empty(n, dtype=dtype).as_subclass(Tensor))
        return made[-1]

    side, other = types.SimpleNamespace(cuda_stream=11), types.SimpleNamespace(cuda_stream=12)
    fake = types.SimpleNamespace(empty=empty, uint8=torch.uint8, int8=torch.int8, float64=torch.float64, Tensor=torch.Tensor,
                                 cuda=types.SimpleNamespace(current_stream=lambda *a: types.SimpleNamespace(cuda_stream=0)))

    class Lib:
        def __getattr__(self, name):
            return lambda *a: 4096 if name == "idp_dg_workspace_bytes" else 0

    monkeypatch.setattr(idp_dg, "_torch", lambda: fake)
    monkeypatch.setattr(idp_dg, "lib", Lib())
    return made, side, other


def used(t):
    return [s.cuda_stream for s in t.__dict__.get("streams", [])]


def test_streams_are_recorded(faked):
    made, side, other = faked
    prob = W.Problem(dim=1, nx=4, ny=1, p=3, eq=W.BURGERS, bc=(1, 0))
    sv = idp_dg.Solver(prob, stream=side, workspace=True)
    assert used(made[0]) == [11]
    t, s = (torch.zeros(1, dtype=d).as_subclass(Tensor) for d in (torch.int8, torch.float64))
    sv.set_boundary(0, t, s)
    assert used(t) == used(s) == [11]
    b = idp_dg.Batch([sv], stream=other)
    assert set(used(made[0])) == set(used(t)) == set(used(s)) == {11, 12}
    t2 = torch.zeros(1, dtype=torch.int8).as_subclass(Tensor)
    sv.set_boundary(1, t2)      # the batch reads it too
    assert set(used(t2)) == {11, 12}
    sv2 = idp_dg.Solver(prob, stream=side, workspace=True)
    b.update([sv, sv2])
    assert set(used(made[1])) == {11, 12}


@pytest.mark.gpu
def test_memory_of_a_closed_solver_waits_for_its_stream():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    prob = W.Problem(dim=2, nx=64, ny=64, p=4, eq=W.EULER)
    side = torch.cuda.Stream()
    u = torch.from_numpy(W.euler_quadrants(prob, np.random.default_rng(1))).cuda()
    torch.cuda.synchronize()
    sv = idp_dg.Solver(prob, stream=side, workspace=True)
    n, at = sv._ws.numel(), sv._ws.data_ptr()
    with torch.cuda.stream(side):
        torch.cuda._sleep(200_000_000)   # about 0.1 s ahead of the step
    sv.step_cfl(u, 0.5)
    sv.close()
    x = torch.empty(n, dtype=torch.uint8, device="cuda")
    pending = not side.query()
    assert pending and x.data_ptr() != at
    torch.cuda.synchronize()
    assert bool(torch.isfinite(u).all())
