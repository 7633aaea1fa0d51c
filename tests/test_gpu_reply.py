"""Answers through pinned memory: a state or window of any size is the same
whichever way it comes (small: written by the kernel; large: in chunks by the
copy engine; between, and rows longer than a chunk: copied), bit for bit, and
two threads that ask members of one batch get each their own."""
import threading

import numpy as np
import pytest

from common import pulse_workload

pytestmark = pytest.mark.gpu
BC = ("extrap0",) * 4


# cells of a small answer: 8192; of one in chunks: 3 nx ny >= 524288, 131072 a chunk
@pytest.mark.parametrize("nx,ny", [(64, 128), (64, 129), (512, 341), (512, 342), (1000, 525), (131072, 4), (131073, 4)])
def test_state_equals_its_rows(nx, ny):
    from paper_1311_3004_amd import fvna
    w = pulse_workload(nx, ny, BC)
    s = fvna.sim_from_workload(w, precision="f64")
    s.fvna_step(3)
    state = s.fvna_get_state()
    full = s.fvna_get_window(0, 0, nx, ny)
    ni = min(nx, 2000)
    for j in sorted({0, 1, ny // 2, ny - 2, ny - 1}):
        for i0 in {0, nx - ni}:
            row = s.fvna_get_window(i0, j, ni, 1)
            for a, b, r in zip(state, full, row):
                assert np.array_equal(a[j, i0:i0 + ni], r[0]) and np.array_equal(b[j, i0:i0 + ni], r[0])
    sums = s.fvna_sums()
    s.fvna_destroy()
    for a, t in zip(state, sums):       # FP64 sums in another order: 1e-12 of the sum of magnitudes
        assert abs(a.sum() - t) <= 1e-12 * np.abs(a).sum()


@pytest.mark.parametrize("shape", [(30, 20, 10), (128, 33, 40), (257, 64, 32)])
def test_3d_state_survives_the_round_trip(shape):
    from paper_1311_3004_amd import fvna3d as f3
    from test_gpu_3d import DX, MED
    nx, ny, nz = shape
    rng = np.random.default_rng(nx)
    q = [rng.standard_normal((nz, ny, nx)) * 1e-3 for _ in range(4)]
    q[0] *= MED["rho0"]
    q[1:] = [m * MED["rho0"] * MED["c0"] for m in q[1:]]
    s = f3.Sim3(f3.make_params(nx, ny, nz, DX, MED, bc=BC + BC[:2], precision="f64"))
    s.fvna3_set_state(*q)
    g = s.fvna3_get_state()
    s.fvna3_destroy()
    for a, b in zip(g, q):              # one division and one multiplication: two roundings
        assert np.max(np.abs(a - b) / np.abs(b)) <= 2.3e-16 * 2


def test_members_of_a_batch_asked_by_two_threads():
    from paper_1311_3004_amd import fvna
    works = [pulse_workload(60 + 10 * k, 50 + k, BC, seed=k + 1) for k in range(4)]
    b = fvna.Batch([fvna.make_params(w["nx"], w["ny"], w["dx"], w["medium"], bc=w["bc"], precision="f64") for w in works])
    for k, w in enumerate(works):
        b.fvna_batch_set_state(k, *w["state"])
    b.fvna_batch_step(5)
    want = [b.fvna_batch_get_state(k) for k in range(4)]
    bad = []

    def ask(k):
        for _ in range(20):
            if not all(np.array_equal(x, y) for x, y in zip(b.fvna_batch_get_state(k), want[k])):
                bad.append(k)
            if b.fvna_batch_get_stats(k)["steps"] != 5:
                bad.append(k)
    t = [threading.Thread(target=ask, args=(k,)) for k in range(2)]
    [x.start() for x in t]
    [x.join() for x in t]
    b.fvna_batch_destroy()
    assert not bad
