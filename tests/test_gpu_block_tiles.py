"""Block tiles of the step (small grids: k_step_block) against wavefront
segments (tile_rows given: k_step) and the oracle.  The two evaluate every
cell with the same operations, so they are compared bit for bit."""
import numpy as np
import pytest

from common import max_rel, pulse_workload, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

SOURCE = {"freq": 1e6, "p_surface": 2e5, "focal_length": 6e-3, "aperture": 4e-3, "ramp_cycles": 3.0}
TAYLOR = {"amplitude_pa": 2e6, "x0_m": 2.2e-3, "angle": np.pi / 8}

# sizes: one strip and one past it, a tile's rows and one past them, a grid
# narrower than the halos of its strip, tiles of one, two and several batches
CASES = [
    (4, 4, ("periodic",) * 4, "planar"),
    (58, 8, ("extrap0",) * 4, "planar"),
    (59, 11, ("reflect",) * 4, "planar"),
    (63, 2 * 10 + 1, ("extrap0", "reflect", "periodic", "periodic"), "planar"),
    (64, 33, ("periodic", "periodic", "reflect", "extrap0"), "planar"),
    (117, 700, ("reflect", "extrap0", "extrap0", "reflect"), "planar"),
    (150, 90, ("taylor",) * 4, "planar"),
    (131, 75, ("source", "extrap0", "reflect", "extrap0"), "planar"),
    (200, 61, ("source", "extrap0", "reflect", "extrap0"), "axisym"),
    (75, 131, ("extrap0", "extrap0", "reflect", "taylor"), "axisym"),
]


def workload(nx, ny, bc, geometry):
    w = pulse_workload(nx, ny, bc, geometry=geometry, seed=nx + ny,
                       source=SOURCE if "source" in bc else None, taylor=TAYLOR if "taylor" in bc else None)
    if "source" in bc:
        w["t0"] = 2.0e-6
    return w


@pytest.mark.parametrize("precision", ["f64", "f32", "f32_f16store", "f32_bf16store"])
@pytest.mark.parametrize("nx,ny,bc,geometry", CASES)
def test_block_tiles_equal_segments_bitwise(nx, ny, bc, geometry, precision):
    w = workload(nx, ny, bc, geometry)
    over = {"store_scale": (2e-3,) * 3} if "store" in precision else {}
    a, sa, simA = run_gpu(w, 35, precision, **over)
    b, sb, simB = run_gpu(w, 35, precision, tile_rows=16, **over)
    simA.fvna_destroy()
    simB.fvna_destroy()
    assert sa == sb
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("nx,ny,bc,geometry", CASES)
def test_block_tiles_vs_oracle(orc, nx, ny, bc, geometry):
    w = workload(nx, ny, bc, geometry)
    (R, M, N), info = run_oracle(orc, w, 20)
    g, st, sim = run_gpu(w, 20, "f64")
    sim.fvna_destroy()
    assert st["steps"] == 20 and st["rejected"] == info["rejected"]
    assert max_rel(g, (R, M, N)) < 1e-10
