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
