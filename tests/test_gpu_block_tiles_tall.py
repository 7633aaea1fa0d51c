"""Block tiles of three and more batches (what a batch keeps in LDS is read by
the one after the next, the analytic side data are in their second and later
slots, ghost and axisymmetric rows lie in other batches than the first) against
wavefront segments, bit for bit."""
import numpy as np
import pytest

from common import run_gpu
from test_gpu_block_tiles import workload

pytestmark = pytest.mark.gpu
SOURCE_SIDES = ("source", "extrap0", "reflect", "extrap0")


def batches(nx, ny, f64):
    """Batches of a block tile by the library's rule: 8 B - 6 rows in B batches,
    blocks in rounds of two per CU, two together 1.55 times as long as one."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    strips, best = -(-nx // 58), (1e30, 0)
    for b in range(1, ny):
        segs = -(-ny // (8 * b - 6))
        full, rest = divmod(strips * segs, 2 * cus)
        us = 4.5 + (2.85 if f64 else 2.0) * b * (1.55 * full + (1.55 if rest > cus else 1.0 if rest else 0.0))
        best = min(best, (us, b))
        if segs == 1:
            break
    return best[1]


@pytest.mark.parametrize("nx,ny,bc,geometry,precision,count", [
    (480, 800, SOURCE_SIDES, "axisym", "f64", 3),
    (480, 800, SOURCE_SIDES, "planar", "f64", 3),
    (1044, 503, ("taylor",) * 4, "planar", "f64", 3),
    (850, 850, ("extrap0", "reflect", "periodic", "periodic"), "planar", "f64", 4),
    (850, 850, ("extrap0", "extrap0", "reflect", "taylor"), "axisym", "f64", 4),
    (428, 2087, ("taylor", "extrap0", "taylor", "reflect"), "planar", "f64", 5),
    (428, 2087, SOURCE_SIDES, "axisym", "f64", 5),
    (480, 800, SOURCE_SIDES, "axisym", "f32", 3),
    (1044, 503, ("taylor",) * 4, "planar", "f32", 3),
    (850, 850, ("source", "taylor", "reflect", "taylor"), "axisym", "f32", 4),
    (850, 850, ("taylor",) * 4, "planar", "f32_f16store", 4),
    (850, 850, SOURCE_SIDES, "axisym", "f32_bf16store", 4),
])
def test_tall_block_tiles_equal_segments_bitwise(nx, ny, bc, geometry, precision, count):
    assert batches(nx, ny, precision == "f64") == count
    w = workload(nx, ny, bc, geometry)
    over = {"store_scale": (2e-3,) * 3} if "store" in precision else {}
    a, sa, simA = run_gpu(w, 9, precision, **over)
    b, sb, simB = run_gpu(w, 9, precision, tile_rows=16, **over)
    assert simA.fvna_get_tile_rows() == 0 and simB.fvna_get_tile_rows() == 16
    simA.fvna_destroy()
    simB.fvna_destroy()
    assert sa == sb and sa["steps"] == 9
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
