"""Results do not depend on where tiles begin: strong, rough and strongly damped
flow, in which a velocity that differs in its last bit at a tile's first row
reaches the stored values through the limiter, the source or the CFL maximum.
2-D: every segment height and the block tiles give the same bits.  3-D, whose
tiles follow from the grid: a periodic state moved along x2 and x3 gives the
moved result."""
import numpy as np
import pytest

from common import pulse_workload, run_gpu

pytestmark = pytest.mark.gpu
P, E = "periodic", "extrap0"
DX = 1e-4
MED = {"c0": 1500.0, "rho0": 1000.0, "beta": 3.5, "delta": 0.2 * 1500.0 * DX}   # delta / (c0 dx) = 0.2


def rough(shape, fields, seed):
    """(rho', momenta) in SI: white noise about a compressed medium (in which
    such flow stays hyperbolic)."""
    rng = np.random.default_rng(seed)
    R = rng.uniform(0.15, 0.45, shape)
    s = MED["rho0"] * MED["c0"]
    return (R * MED["rho0"],) + tuple(s * (1 + R) * rng.uniform(-0.25, 0.25, shape) for _ in range(fields - 1))


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("nx,ny,bc,geometry", [(174, 700, (P, P, P, P), "planar"), (150, 611, (E, E, "reflect", E), "planar"),
                                               (116, 640, (E, E, "reflect", E), "axisym")])
def test_heights_and_block_tiles_bitwise(nx, ny, bc, geometry, precision):
    w = pulse_workload(nx, ny, bc, geometry=geometry, medium=MED)
    w["state"] = rough((ny, nx), 3, nx + ny)
    want = None
    for tile_rows in (16, 0, 8, 13, 40, 300):
        g, st, sim = run_gpu(w, 40, precision, tile_rows=tile_rows)
        sim.fvna_destroy()
        assert st["status"] == 0 and st["steps"] == 40
        if want is None:
            want = g, st
        assert st == want[1], tile_rows
        for a, b in zip(g, want[0]):
            assert np.array_equal(a, b), tile_rows


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("shape", [(64, 60, 50), (90, 75, 64)])
def test_3d_moved_state_gives_the_moved_result_bitwise(shape, precision):
    from paper_1311_3004_amd import fvna3d as f3
    nx, ny, nz = shape
    q = rough((nz, ny, nx), 4, sum(shape))
    want = None
    for dz, dy in ((0, 0), (0, 1), (0, 3), (1, 0), (4, 2)):
        s = f3.Sim3(f3.make_params(nx, ny, nz, DX, MED, bc=(P,) * 6, precision=precision))
        s.fvna3_set_state(*[np.ascontiguousarray(np.roll(f, (dz, dy), (0, 1))) for f in q])
        s.fvna3_step(20)
        g = [np.roll(f, (-dz, -dy), (0, 1)) for f in s.fvna3_get_state()]
        st = s.fvna3_get_stats()
        s.fvna3_destroy()
        assert st["steps"] == 20
        if want is None:
            want = g, st
        assert st == want[1], (dz, dy)
        for a, b in zip(g, want[0]):
            assert np.array_equal(a, b), (dz, dy)
