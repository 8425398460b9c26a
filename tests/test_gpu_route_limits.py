"""Steps on either side of the limits of their routes, bitwise against the
separate entry points (the routes themselves are read on the host): the last
1-D Euler mesh of one launch and the one after it, and the last number of
tiles whose minima the first stage folds and the one after it, with the sizes
taken from the tile shape."""
import pytest

from paper_2004_08503_amd import workloads as W
from test_gpu_step_launches import _gpu, check

pytestmark = pytest.mark.gpu
pytest.importorskip("torch")


@pytest.mark.parametrize("p", [1, 4, 8])
@pytest.mark.parametrize("gamma", [1.4, 5.0 / 3.0, 1.3])
def test_one_launch_euler(gamma, p):
    idp_dg = _gpu()
    for k, nx in enumerate((510 // (p + 1), 510 // (p + 1) + 1)):
        check(idp_dg, W.Problem(dim=1, nx=nx, ny=1, p=p, eq=W.EULER, gamma=gamma, limiter=k, bc=(k, 0)), p + k)


@pytest.mark.parametrize("shape", [0, 1])
@pytest.mark.parametrize("p", [2, 6, 8])
def test_folded_minima(p, shape):
    idp_dg = _gpu()
    sv = idp_dg.Solver(W.Problem(dim=2, nx=2, ny=2, p=p, eq=W.EULER))
    sv.set_tile_shape(shape)
    tx, ty = sv.tile_dims
    sv.close()
    for nx in (32 * tx, 32 * tx + 1):   # 1024 tiles, then 33 x 32
        check(idp_dg, W.Problem(dim=2, nx=nx, ny=32 * ty, p=p, eq=W.EULER), p, shape)


@pytest.mark.parametrize("prob", [W.Problem(dim=1, nx=60, ny=1, p=3, eq=W.EULER), W.Problem(dim=2, nx=20, ny=17, p=4, eq=W.EULER),
                                  W.Problem(dim=2, nx=100, ny=100, p=4, eq=W.BURGERS)], ids=["one", "fold", "reduce"])
def test_captured_steps(prob):
    """Every route inside a caller's graph: replays, with eager work and
    synchronisation between them, equal eager steps bitwise."""
    import torch
    from test_gpu_step_launches import data
    idp_dg = _gpu()
    prob, u0 = data(prob, 5)
    s = torch.cuda.Stream()
    sv, ref = idp_dg.Solver(prob, stream=s), idp_dg.Solver(prob)
    u, v = torch.from_numpy(u0).cuda(), torch.from_numpy(u0).cuda()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        sv.step_cfl(u, 0.5)
    for k in range(4):
        with torch.cuda.stream(s):
            g.replay()
        ref.step_cfl(v, 0.5)
        if k % 2:
            with torch.cuda.stream(s):
                w = u.clone()
            sv.step(w, 1e-4)   # eager work through the same buffers
        torch.cuda.synchronize()
        assert torch.equal(u, v), k
        assert sv.last_dt() == ref.last_dt()
    sv.close()
    ref.close()
