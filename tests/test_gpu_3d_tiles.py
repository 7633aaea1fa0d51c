"""The 3-D kernels at the edges of their tiles: grids smaller than a tile, one
column or plane past one, single-plane segments, every side kind on every
axis; 33 steps, so that decisions are taken in the prologues of a captured
graph and of the attempts after it.  Tolerances of test_gpu_3d.py."""
import pytest

from test_gpu_3d import _run_pair

pytestmark = pytest.mark.gpu
P, E, R = "periodic", "extrap0", "reflect"


@pytest.mark.parametrize("precision,tol", [("f64", 1e-10), ("f32", 2e-6)])
@pytest.mark.parametrize("shape,bc", [
    ((4, 4, 4), (P,) * 6),
    ((4, 5, 6), (R, E, R, E, R, E)),
    ((61, 9, 4), (E, E, P, P, E, R)),
    ((7, 61, 33), (P, P, E, R, P, P)),
    ((64, 17, 5), (R,) * 6),
    ((125, 6, 12), (E, R, E, E, P, P)),
    ((9, 8, 130), (E, E, R, R, R, E)),
])
def test_3d_tiles_vs_oracle(shape, bc, precision, tol):
    err, st, info = _run_pair(precision, 33, False, shape=shape, bc=bc, seed=sum(shape))
    assert err <= tol
    assert st["rejected"] == 0
