"""Flows as fast as sound somewhere, so that a wave family moves against its
usual direction there (|w| >= c) and the sweeps leave the form that takes the
directions for granted: jets along each axis, each narrower than a wavefront,
beside slow flow.  Tolerances: those of the other oracle comparisons (FP64 1e-10,
FP32 2e-6), of the largest field, here a momentum; FP32 four times as much, the
slowest squared wave speed being about a quarter of the medium's."""
import numpy as np
import pytest

from common import max_rel, pulse_workload, run_gpu, run_oracle

pytestmark = pytest.mark.gpu
P, E = "periodic", "extrap0"


def jets(nx, ny, bc):
    w = pulse_workload(nx, ny, bc, seed=nx + ny)
    med = w["medium"]
    x, y = np.meshgrid(np.arange(nx) + 0.5, np.arange(ny) + 0.5)
    rho = 0.1 * np.exp(-((x - 0.3 * nx) ** 2 + (y - 0.6 * ny) ** 2) / 72.0)
    u = 0.78 * np.exp(-((y - 0.25 * ny) / 6.0) ** 2)
    v = -0.78 * np.exp(-((x - 0.8 * nx) / 6.0) ** 2)
    s = med["rho0"] * med["c0"]
    w["state"] = (med["rho0"] * rho, s * (1 + rho) * u, s * (1 + rho) * v)
    return w


def both_kinds(w):
    """Whether the state has interfaces with |w| >= c and with |w| < c along x1 and x2."""
    med = w["medium"]
    r, m, n = w["state"]
    rho, u, v = r / med["rho0"], m / (med["rho0"] * med["c0"]), n / (med["rho0"] * med["c0"])
    out = []
    for ax, q in ((1, u), (0, v)):
        z = q / (1 + rho)
        lo, hi = [slice(None)] * 2, [slice(None)] * 2
        lo[ax], hi[ax] = slice(None, -1), slice(1, None)
        sr, sn = rho[tuple(lo)] + rho[tuple(hi)], z[tuple(lo)] + z[tuple(hi)]
        ww = sn / (2 + sr)
        d = 1 + ww * (ww - sn) + (med["beta"] - 1) * sr
        fast = ww * ww >= d
        out.append(bool((d > 0).all() and fast.any() and not fast.all()))
    return all(out)


@pytest.mark.parametrize("tile_rows", [0, 12, 40])
@pytest.mark.parametrize("nx,ny,bc", [(150, 90, (E, E, E, E)), (117, 131, (P, P, E, E)), (64, 61, (P, P, P, P))])
def test_fast_flow_2d_vs_oracle(orc, nx, ny, bc, tile_rows):
    w = jets(nx, ny, bc)
    assert both_kinds(w)
    o, info = run_oracle(orc, w, 5)
    assert info["status"] == 0
    for precision, tol in (("f64", 1e-10), ("f32", 8e-6)):
        g, st, sim = run_gpu(w, 5, precision, tile_rows=tile_rows)
        sim.fvna_destroy()
        assert st["steps"] == 5
        assert max_rel(g, o, peak=max(np.max(np.abs(f)) for f in o)) < tol


@pytest.mark.parametrize("axis", [0, 1, 2])
def test_fast_flow_3d_vs_oracle(axis):
    from oracle import oracle3d as o3
    from paper_1311_3004_amd import fvna3d as f3
    from test_gpu_3d import DX, MED
    n = (70, 40, 38)
    x = np.meshgrid(*[np.arange(k) + 0.5 for k in n[::-1]], indexing="ij")[::-1]
    rho = 0.1 * np.exp(-sum((x[a] - 0.4 * n[a]) ** 2 for a in range(3)) / 50.0)
    u = 0.8 * np.exp(-sum(((x[a] - 0.5 * n[a]) / 7.0) ** 2 for a in range(3) if a != axis))
    M = [(1 + rho) * u * (1.0 if a == axis else 0.05) for a in range(3)]
    bc = (P, P) * 3
    po = o3.make_params(*n, MED["beta"], MED["delta"] / (MED["c0"] * DX), bc=bc)
    o, info = o3.run(po, [rho] + M, 6)
    assert info["status"] == 0
    for precision, tol in (("f64", 1e-10), ("f32", 8e-6)):
        s = f3.Sim3(f3.make_params(*n, DX, MED, bc=bc, precision=precision))
        s.fvna3_set_state(rho * MED["rho0"], *[m * MED["rho0"] * MED["c0"] for m in M])
        s.fvna3_step(6)
        g = s.fvna3_get_state()
        s.fvna3_destroy()
        g = (g[0] / MED["rho0"],) + tuple(m / (MED["rho0"] * MED["c0"]) for m in g[1:])
        assert max(np.max(np.abs(a - b)) for a, b in zip(g, o)) / max(np.max(np.abs(f)) for f in o) < tol
