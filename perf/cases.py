"""Timed cases of the finite-volume step: what the users of libfvna and
libfvna3d run, through the ctypes bindings, over the sizes, boundary kinds,
geometries and precisions that this repository's workloads, tests and
benchmark use.

Kinds of case (`kind`) and what each stands for in real use:

  sampled   the axis-sampling loop without a recorder: two steps, one grid row
            and the clock read back.  Latency of a call counts, not throughput.
  pulse     a planar run between two reads of the state: a Gaussian pulse with
            noise; open, closed, periodic or half periodic sides.
  focused   the same for the axisymmetric focused field, source ramping up.
  shock     the oblique Taylor shock with analytic data on all four sides.
  packet    the focused packet on the moving domain with the on-axis recorder,
            mid-flight, and the final read of the state.
  batch     many uneven simulations advanced by one launch per step.
  box       the 3-D step, the state left on the device.
  box_io    a short 3-D run with the final read of the state.
  whole     a whole short run: state in, steps, conservation sums, state out.

Outputs are whole states: the caller-owned buffer that holds the current state
(an even number of accepted steps after the state was set it is the first one;
in three dimensions, a multiple of six steps after, density and momenta are in
the second and the first), or the arrays that the read entry points return.

exact() is the method in plain torch, 64 bits, without this package.
"""
import math

import numpy as np
import torch

WATER = {"c0": 1500.0, "rho0": 1000.0, "beta": 3.5, "delta": 4.3e-6}
TISSUE = {"c0": 1540.0, "rho0": 1000.0, "beta": 4.8, "delta": 6.4117e-4}
PACKET_FREQ = 1.1e6
RISE = 2.0 * math.atanh(0.8)            # 10-90% rise of tanh in tanh units

SIDES = {"open": ("extrap0",) * 4, "closed": ("reflect",) * 4, "periodic": ("periodic",) * 4,
         "channel": ("extrap0", "extrap0", "periodic", "periodic")}
SIDES3 = {"open": ("extrap0",) * 6, "closed": ("reflect",) * 6,
          "mixed": ("periodic", "periodic", "reflect", "extrap0", "extrap0", "reflect")}
FLOPS_2D = 260.0      # two Roe solves, two limited wave sums and the source of one cell
FLOPS_3D = 540.0


def listed():
    return [
        # the smallest calls: an axis-sampling loop on a small grid
        {"name": "sampled 96x64 f64", "kind": "sampled", "nx": 96, "ny": 64, "precision": "f64", "steps": 2},
        # the paper's plain workload, 200 adaptive steps
        {"name": "channel 256x256 f64", "kind": "pulse", "sides": "channel", "nx": 256, "ny": 256,
         "precision": "f64", "steps": 200},
        # the benchmark's grid in the paper's arithmetic
        {"name": "pulse 4096x4096 f64", "kind": "pulse", "sides": "open", "nx": 4096, "ny": 4096,
         "precision": "f64", "steps": 20},
        # an ordinary ragged grid in single precision
        {"name": "pulse 1501x1099 f32", "kind": "pulse", "sides": "closed", "nx": 1501, "ny": 1099,
         "precision": "f32", "steps": 50},
        # the axisymmetric focused field of the benchmark
        {"name": "focused 8192x2048 f32", "kind": "focused", "nx": 8192, "ny": 2048, "precision": "f32",
         "steps": 32},
        # half-width storage, ragged
        {"name": "focused 2051x1027 f16", "kind": "focused", "nx": 2051, "ny": 1027,
         "precision": "f32_f16store", "steps": 40},
        # one run of the Taylor-shock study (10 cells per rise, pi/8), between two looks at its clock
        {"name": "shock 1044x503 f64", "kind": "shock", "nx": 1044, "ny": 503, "eta": 10, "angle": math.pi / 8,
         "precision": "f64", "steps": 60},
        # the focused packet on the paper's moving domain, 20 cells per wavelength
        {"name": "packet 480x800 f64", "kind": "packet", "nx": 480, "ny": 800, "eta": 20, "precision": "f64",
         "steps": 240},
        # uneven simulations in one batch
        {"name": "batch of 12 f32", "kind": "batch", "members": 12, "least": 256, "most": 1024,
         "layout": 4, "precision": "f32", "steps": 32},
        # the 3-D step of the benchmark
        {"name": "box 256^3 f32", "kind": "box", "sides": "open", "nx": 256, "ny": 256, "nz": 256,
         "precision": "f32", "steps": 12},
        # a small ragged 3-D run with its final read
        {"name": "box 90x75x64 f64", "kind": "box_io", "sides": "mixed", "nx": 90, "ny": 75, "nz": 64,
         "precision": "f64", "steps": 120},
        # a whole short run
        {"name": "whole 1024x768 f64", "kind": "whole", "sides": "periodic", "nx": 1024, "ny": 768,
         "precision": "f64", "steps": 100},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("sampled", "pulse", "pulse", "pulse", "focused", "focused", "shock", "packet", "batch",
                       "box", "box_io", "whole"))
    if kind == "sampled":
        return {"kind": kind, "nx": _log(rng, 64, 600), "ny": _log(rng, 48, 600),
                "precision": rng.choice(("f64", "f32")), "steps": 2}
    if kind == "pulse":
        nx, ny = _log(rng, 128, 4096), _log(rng, 128, 4096)
        return {"kind": kind, "sides": rng.choice(sorted(SIDES)), "nx": nx, "ny": ny,
                "precision": rng.choice(("f64", "f64", "f32", "f32_f16store", "f32_bf16store")),
                "steps": 2 * rng.randint(5, 100 if nx * ny < 1 << 18 else 30 if nx * ny < 1 << 21 else 8)}
    if kind == "focused":
        nx, ny = _log(rng, 600, 8192), _log(rng, 200, 2048)
        return {"kind": kind, "nx": nx, "ny": ny, "precision": rng.choice(("f64", "f32", "f32", "f32_f16store")),
                "steps": 2 * rng.randint(4, 24 if nx * ny < 1 << 21 else 10)}
    if kind == "shock":
        eta = rng.choice((5, 10, 20))
        return {"kind": kind, "nx": _log(rng, 20 * eta, 112 * eta), "ny": _log(rng, 20 * eta, 60 * eta),
                "eta": eta, "angle": rng.choice((math.pi / 32, math.pi / 16, math.pi / 8, math.pi / 4)),
                "precision": rng.choice(("f64", "f64", "f32")), "steps": 2 * rng.randint(5, 40)}
    if kind == "packet":
        eta = rng.choice((20, 20, 41))
        return {"kind": kind, "nx": rng.randint(18, 30) * eta, "ny": rng.randint(20, 40) * eta, "eta": eta,
                "precision": rng.choice(("f64", "f64", "f32")), "steps": rng.randint(30, 240)}
    if kind == "batch":
        return {"kind": kind, "members": rng.randint(3, 16), "least": 96, "most": rng.choice((256, 512, 1024)),
                "layout": rng.randint(1, 10 ** 6), "precision": rng.choice(("f32", "f32", "f64")),
                "steps": 2 * rng.randint(5, 24)}
    if kind in ("box", "box_io"):
        top = 224 if kind == "box" else 100
        return {"kind": kind, "sides": rng.choice(sorted(SIDES3)), "nx": _log(rng, 24, top),
                "ny": _log(rng, 20, top), "nz": _log(rng, 20, top), "precision": rng.choice(("f64", "f32")),
                "steps": 6 * rng.randint(1, 8 if kind == "box" else 20)}
    return {"kind": "whole", "sides": rng.choice(sorted(SIDES)), "nx": _log(rng, 128, 1400),
            "ny": _log(rng, 128, 1000), "precision": rng.choice(("f64", "f32")), "steps": 2 * rng.randint(10, 80)}


# ---------------------------------------------------------------------------
# Inputs, from the seed alone (SI fields and parameters).
# ---------------------------------------------------------------------------

def _gauss(n, centre, sigma):
    return np.exp(-((np.arange(n) - centre) ** 2) / (2.0 * sigma * sigma))


def _pulse_fields(nx, ny, seed, med, sigma=20.0, amplitude=2e6):
    rng = np.random.default_rng(seed)
    a = amplitude * rng.uniform(0.8, 1.2) / (med["rho0"] * med["c0"] ** 2)
    ci, cj = int(rng.integers(nx // 4, nx - nx // 4)), int(rng.integers(ny // 4, ny - ny // 4))
    s = min(sigma, min(nx, ny) / 8.0)
    R = np.outer(_gauss(ny, cj, s), a * _gauss(nx, ci, s))
    R += 0.005 * a * rng.uniform(-1.0, 1.0, R.shape)
    return med["rho0"] * R, (0.3 * med["rho0"] * med["c0"]) * R, (-0.2 * med["rho0"] * med["c0"]) * R, a


def _setup(c, seed):
    """Everything both sides need to know about one planar or axisymmetric
    simulation: grid, medium, sides, source or profile, start time, fields."""
    kind, nx, ny = c["kind"], c["nx"], c["ny"]
    w = {"nx": nx, "ny": ny, "dx": 1e-4, "medium": dict(WATER), "geometry": "planar", "t0": 0.0,
         "precision": c["precision"], "cfl_target": 0.9, "cfl_max": 1.0, "scale": 1.0}
    if kind in ("pulse", "sampled", "whole"):
        w["bc"] = SIDES[c.get("sides", "channel")]
        r, m, n, a = _pulse_fields(nx, ny, seed, w["medium"])
        w["state"] = (r, m, n)
        w["scale"] = 4.0 * a
    elif kind == "focused":
        w.update(dx=2e-5, geometry="axisym", bc=("source", "extrap0", "reflect", "extrap0"))
        w["source"] = {"freq": 1e6, "p_surface": 2e5, "focal_length": 62.6e-3, "aperture": 35e-3,
                       "ramp_cycles": 3.0}
        w["t0"] = 2.5e-6
        r, m, n, a = _pulse_fields(nx, ny, seed, w["medium"], amplitude=4e5)
        w["state"] = (r, m, np.zeros_like(n))
        w["scale"] = 32.0 * a
    elif kind == "shock":
        rng = np.random.default_rng(seed)
        amp = 1e-7 * rng.uniform(0.8, 1.25)
        med = w["medium"]
        wt = med["delta"] / (med["c0"] * med["beta"] * amp)
        w["dx"] = dx = wt * RISE / c["eta"]
        ca, sa = math.cos(c["angle"]), math.sin(c["angle"])
        x0 = rng.uniform(0.2, 0.5) * nx * dx * ca
        w["bc"] = ("taylor",) * 4
        w["taylor"] = {"amplitude_pa": amp * med["rho0"] * med["c0"] ** 2, "x0_m": x0, "angle": c["angle"]}
        x, y = (np.arange(nx) + 0.5) * dx, (np.arange(ny) + 0.5) * dx
        R = -amp * np.tanh(((x[None, :] - x0) * ca + y[:, None] * sa) / wt)
        k = med["rho0"] * med["c0"]
        w["state"] = (med["rho0"] * R, k * ca * R, k * sa * R)
    elif kind == "packet":
        rng = np.random.default_rng(seed)
        w["medium"] = med = dict(TISSUE)
        lam = med["c0"] / PACKET_FREQ
        eta = c["eta"]
        w["dx"] = lam / eta
        w["bc"] = ("source", "extrap0", "reflect", "extrap0")
        a_wl = max(4, ny // eta - 10)
        t1 = 0.5 * (nx // eta) / PACKET_FREQ
        w["source"] = {"freq": PACKET_FREQ, "p_surface": 4.217e-4 * med["rho0"] * med["c0"] ** 2,
                       "focal_length": 50.0 * lam, "aperture": a_wl * lam, "ramp_cycles": 3.0,
                       "envelope": "packet", "packet_cycles": 4.0, "stage2_time": t1}
        w["t0"] = t1
        q = max(4, int(round(eta / 4)))
        w["window"] = {"t1": t1, "check_every": q, "quantum": q}
        w["path"] = 105 * eta
        w["probe_col"] = nx // 2
        # the packet in mid-flight: a focusing carrier under its envelope
        x, y = (np.arange(nx) + 0.5) / eta, (np.arange(ny) + 0.5) / eta
        tau = 0.5 * nx / eta - x[None, :] + y[:, None] ** 2 / 100.0
        env = np.exp(-(tau / 4.0) ** 10) / (1.0 + np.exp(np.minimum(4.0 * (y[:, None] - a_wl), 60.0)))
        R = 4.217e-4 * rng.uniform(0.8, 1.2) * env * np.sin(2 * np.pi * (tau + rng.uniform(0, 1)))
        k = med["rho0"] * med["c0"]
        w["state"] = (med["rho0"] * R, k * R, -k * R * (y[:, None] / 50.0))
    return w


def _members(c, seed):
    sizes = np.random.default_rng(c["layout"])
    out = []
    for k in range(c["members"]):
        nx, ny = (int(sizes.integers(c["least"], c["most"] + 1)) for _ in range(2))
        beta, delta = float(sizes.uniform(3, 5)), float(10.0 ** sizes.uniform(-6, -5))
        w = _setup({"kind": "pulse", "sides": "open", "nx": nx, "ny": ny, "precision": c["precision"]},
                   seed * 1000 + k)
        w["medium"].update(beta=beta, delta=delta)
        out.append(w)
    return out


def _fields3(c, seed):
    rng = np.random.default_rng(seed)
    n = (c["nz"], c["ny"], c["nx"])
    a = 2e6 * rng.uniform(0.8, 1.2) / (WATER["rho0"] * WATER["c0"] ** 2)
    g = [_gauss(m, rng.uniform(0.35, 0.65) * m, min(8.0, m / 6.0)) for m in n]
    R = a * g[0][:, None, None] * g[1][None, :, None] * g[2][None, None, :]
    R += 0.005 * a * rng.uniform(-1.0, 1.0, n)
    k = WATER["rho0"] * WATER["c0"]
    return WATER["rho0"] * R, 0.3 * k * R, -0.2 * k * R, 0.1 * k * R


# ---------------------------------------------------------------------------
# The framework's side.
# ---------------------------------------------------------------------------

_TYPES = {"f64": torch.float64, "f32": torch.float32, "f32_f16store": torch.float16,
          "f32_bf16store": torch.bfloat16}


def _plane_view(buf, precision, nx, ny, fields=3):
    """A state buffer as [fields][ny][nx] (rows are padded to 256 bytes)."""
    t = _TYPES[precision]
    per = 256 // torch.empty((), dtype=t).element_size()
    pitch = -(-nx // per) * per
    n = fields * ny * pitch
    return buf.view(t)[:n].view(fields, ny, pitch)[:, :, :nx]


def _sim(w):
    from paper_1311_3004_amd import fvna
    over = {}
    if "store" in w["precision"]:
        over["store_scale"] = (w["scale"],) * 3
    return fvna.sim_from_workload(w, precision=w["precision"], **over)


def prepare(case, seed):
    from paper_1311_3004_amd import fvna
    kind = case["kind"]
    if kind == "batch":
        ws = _members(case, seed)
        b = fvna.Batch([fvna.make_params(w["nx"], w["ny"], w["dx"], w["medium"], bc=w["bc"],
                                         precision=w["precision"]) for w in ws])
        for k, w in enumerate(ws):
            b.fvna_batch_set_state(k, *w["state"])
        return {"case": case, "batch": b,
                "out": [_plane_view(b.bufs[3 * k], w["precision"], w["nx"], w["ny"]) for k, w in enumerate(ws)]}
    if kind in ("box", "box_io"):
        from paper_1311_3004_amd import fvna3d
        s = fvna3d.Sim3(fvna3d.make_params(case["nx"], case["ny"], case["nz"], 1e-4, WATER,
                                           bc=SIDES3[case["sides"]], precision=case["precision"]))
        s.fvna3_set_state(*_fields3(case, seed))
        a, b = (_plane_view(x, case["precision"], case["nx"], case["ny"] * case["nz"], 4) for x in s.bufs[:2])
        return {"case": case, "sim": s, "out": {"R": b[0], "M": a[1:]}}
    w = _setup(case, seed)
    s = _sim(w)
    st = {"case": case, "sim": s, "out": _plane_view(s.buf_a, w["precision"], w["nx"], w["ny"])}
    if kind == "whole":
        st["state"] = w["state"]
    if kind == "packet":
        dev = s.device
        st["row_max"] = torch.zeros(w["path"], dtype=torch.float64, device=dev)
        st["probe_t"] = torch.zeros(4096, dtype=torch.float64, device=dev)
        st["probe_rho"] = torch.zeros(4096, dtype=torch.float64, device=dev)
        torch.cuda.synchronize()
        s.fvna_set_recorder(0, w["probe_col"], w["path"], st["row_max"], st["probe_t"], st["probe_rho"])
        q = w["window"]
        st["window"] = fvna.fvna_window(q["t1"], q["check_every"], q["quantum"])
        st["moved"] = fvna.fvna_window_state(0, 0)
    return st


def run(state):
    case = state["case"]
    kind, steps = case["kind"], case["steps"]
    if kind == "batch":
        state["batch"].fvna_batch_step(steps)
        return state["out"]
    s = state["sim"]
    if kind == "box":
        s.fvna3_step(steps)
        return state["out"]
    if kind == "box_io":
        s.fvna3_step(steps)
        return s.fvna3_get_state()
    if kind == "sampled":
        s.fvna_step(steps)
        row = s.fvna_get_window(0, 0, case["nx"], 1)
        return {"state": state["out"], "row": row, "t": s.fvna_get_stats()["t"]}
    if kind == "whole":
        s.fvna_set_state(*state["state"])
        s.fvna_step(steps)
        return {"sums": s.fvna_sums(), "state": s.fvna_get_state()}
    if kind == "packet":
        s.fvna_step_window(state["window"], state["moved"], steps)
        return {"state": s.fvna_get_state(), "row_max": state["row_max"], "probe_t": state["probe_t"],
                "probe_rho": state["probe_rho"], "x_off": int(state["moved"].x_off)}
    s.fvna_step(steps)
    return state["out"]


def work(case):
    """One read and one write of the state per step, plus what goes to or
    comes from the host."""
    size = {"f64": 8, "f32": 4}.get(case["precision"], 2)
    if case["kind"] == "batch":
        cells = sum(w[0] * w[1] for w in _sizes(case))
    else:
        cells = case["nx"] * case["ny"] * case.get("nz", 1)
    fields, flops = (4, FLOPS_3D) if "nz" in case else (3, FLOPS_2D)
    nbytes = 2.0 * fields * size * cells * case["steps"]
    if case["kind"] in ("box_io", "packet"):
        nbytes += 8.0 * fields * cells
    if case["kind"] == "whole":
        nbytes += 16.0 * fields * cells
    return {"bytes": nbytes, "flops": flops * cells * case["steps"]}


def _sizes(c):
    sizes = np.random.default_rng(c["layout"])
    out = []
    for _ in range(c["members"]):
        out.append(tuple(int(sizes.integers(c["least"], c["most"] + 1)) for _ in range(2)))
        sizes.uniform(3, 5)
        sizes.uniform(-6, -5)
    return out


# ---------------------------------------------------------------------------
# The method in plain torch, 64 bits.
# ---------------------------------------------------------------------------

def _roe(q, d, beta):
    """Waves of the interfaces along dimension d of the cells q = [R, normal
    momentum, tangential momenta ...] (one interface fewer than cells)."""
    n = q[0].shape[d] - 1
    lo, hi = (lambda v: v.narrow(d, 0, n)), (lambda v: v.narrow(d, 1, n))
    q1 = 1.0 + q[0]
    vel = [m / q1 for m in q[1:]]
    zm = 0.5 * (lo(q[0]) + hi(q[0]))
    z1 = 1.0 + zm
    z = [0.5 * (lo(v) + hi(v)) for v in vel]
    w = z[0] / z1
    disc = w * w - 2.0 * z[0] * w + 1.0 + 2.0 * (beta - 1.0) * zm
    c = disc.sqrt()
    dq = [hi(v) - lo(v) for v in q]
    s = [w + c, w - c, w]
    a1 = (dq[1] - s[1] * dq[0]) / (2.0 * c)
    a = [a1, dq[0] - a1]
    waves = []
    for p in range(2):
        g = (s[p] - 2.0 * z[0]) / (z1 * (s[p] - w))
        waves.append([a[p], a[p] * s[p]] + [a[p] * zt * g for zt in z[1:]])
    shear = [dq[2 + k] - waves[0][2 + k] - waves[1][2 + k] for k in range(len(z) - 1)]
    return s, waves, shear, c + w.abs()


def _mc(theta):
    return torch.minimum(torch.minimum(0.5 * (1.0 + theta), torch.full_like(theta, 2.0)),
                         2.0 * theta).clamp_(min=0.0)


def _sweep(q, d, dt, beta):
    """One high-resolution sweep of cells with two ghost cells at each end of
    dimension d -> the updated interior cells and the largest speed."""
    s, waves, shear, speed = _roe(q, d, beta)
    n = q[0].shape[d] - 4
    mid = lambda v: v.narrow(d, 1, n + 1)     # noqa: E731  interfaces that border an interior cell
    up, dn = (lambda v: v.narrow(d, 0, n + 1)), (lambda v: v.narrow(d, 2, n + 1))
    low, high = [0.0] * len(q), [0.0] * len(q)       # what the cell below / above an interface receives
    fam = [(s[0], waves[0], None), (s[1], waves[1], None)] + [(s[2], [v], 2 + k) for k, v in enumerate(shear)]
    for sp, W, only in fam:
        num_lo = sum(up(v) * mid(v) for v in W)
        num_hi = sum(dn(v) * mid(v) for v in W)
        den = sum(mid(v) * mid(v) for v in W)
        sm = mid(sp)
        th = torch.where(sm < 0, num_hi, num_lo) / den
        ph = _mc(torch.where(den == 0, torch.zeros_like(th), th))
        a = sm.abs()
        f = 0.5 * a * (1.0 - dt * a) * ph
        neg, pos = sm.clamp(max=0.0) + f, sm.clamp(min=0.0) - f
        for k, v in enumerate(W):
            comp = k if only is None else only
            low[comp] = low[comp] + neg * mid(v)
            high[comp] = high[comp] + pos * mid(v)
    out = [v.narrow(d, 2, n) - dt * (lo.narrow(d, 1, n) + hi.narrow(d, 0, n)) for v, lo, hi in zip(q, low, high)]
    return out, float(mid(speed).max())


def _pad(q, d, normal, kinds, layers, given=(None, None)):
    """Cells with `layers` ghost cells at both ends of dimension d by the side
    kinds; given[side](layers) supplies (cells, rows it holds for)."""
    n = q[0].shape[d]
    out = []
    ends = []
    for side in range(2):
        kind = kinds[side]
        if given[side] is not None:
            ends.append(given[side](layers))
            continue
        if kind == "periodic":
            at = range(n - layers, n) if side == 0 else range(layers)
        elif kind == "reflect":
            at = range(layers - 1, -1, -1) if side == 0 else range(n - 1, n - 1 - layers, -1)
        else:
            at = [0 if side == 0 else n - 1] * layers
        at = torch.tensor(list(at), device=q[0].device)
        ends.append([v.index_select(d, at) * (-1.0 if kind == "reflect" and k == normal else 1.0)
                     for k, v in enumerate(q)])
    for k, v in enumerate(q):
        out.append(torch.cat([ends[0][k], v, ends[1][k]], d))
    return out


class _Plane:
    """One planar or axisymmetric run in dimensionless variables."""

    def __init__(self, w, dev):
        med, dx = w["medium"], w["dx"]
        self.w, self.dev, self.bc = w, dev, w["bc"]
        self.beta, self.delta = med["beta"], med["delta"] / (med["c0"] * dx)
        self.unit = dx / med["c0"]
        self.t = w["t0"] / self.unit
        fac = (med["rho0"], med["rho0"] * med["c0"], med["rho0"] * med["c0"])
        self.q = [torch.from_numpy(np.ascontiguousarray(a)).to(dev) / f for a, f in zip(w["state"], fac)]
        self.nx, self.ny = w["nx"], w["ny"]
        self.r = torch.arange(self.ny, device=dev, dtype=torch.float64)[:, None] + 0.5
        self.dt = 0.9 / self._dry()

    def _taylor(self, i, j):
        p, med = self.w["taylor"], self.w["medium"]
        amp = p["amplitude_pa"] / (med["rho0"] * med["c0"] ** 2)
        width = med["delta"] / (med["c0"] * med["beta"] * amp * self.w["dx"])
        ca, sa = math.cos(p["angle"]), math.sin(p["angle"])
        x = torch.as_tensor(i, device=self.dev, dtype=torch.float64)[None, :] + 0.5
        y = torch.as_tensor(j, device=self.dev, dtype=torch.float64)[:, None] + 0.5
        R = -amp * torch.tanh(((x - p["x0_m"] / self.w["dx"]) * ca + y * sa - self.t) / width)
        return [R, R * ca, R * sa]

    def _source(self, q, layers):
        p, med, dx = self.w["source"], self.w["medium"], self.w["dx"]
        edge = [v[:, :1].expand(-1, layers) for v in q]
        if self.t * self.unit >= p.get("stage2_time", math.inf):
            return edge
        f, F = p["freq"] * self.unit, p["focal_length"] / dx
        tau = self.t + self.r * self.r / (2.0 * F)
        if p.get("envelope", "ramp") == "packet":
            env = torch.exp(-(f * tau / p["packet_cycles"]) ** 10)
        else:
            rc = p["ramp_cycles"]
            env = 0.0 if self.t <= 0 else math.sin(math.pi * f * self.t / (2 * rc)) ** 2 if self.t < rc / f else 1.0
        g = p["p_surface"] / (med["rho0"] * med["c0"] ** 2) * env * torch.sin(2 * math.pi * torch.frac(f * tau))
        h = torch.sqrt(self.r * self.r + F * F)
        on = self.r <= p["aperture"] / dx
        return [torch.where(on, a, b).expand(-1, layers) if layers == 1 else
                torch.where(on, a.expand(-1, layers), b) for a, b in zip((g, g * F / h, -g * self.r / h), edge)]

    def _pad_x(self, q, layers):
        rows = range(self.ny)
        cols = lambda n, side: range(-n, 0) if side == 0 else range(self.nx, self.nx + n)   # noqa: E731
        given = []
        for side in range(2):
            if self.bc[side] == "taylor":
                given.append(lambda n, s=side: self._taylor(cols(n, s), rows))
            elif self.bc[side] == "source":
                given.append(lambda n: self._source(q, n))
            else:
                given.append(None)
        return _pad(q, 1, 1, self.bc[:2], layers, given)

    def _pad_y(self, q, layers, swept):
        given = []
        for side in range(2):
            if self.bc[2 + side] != "taylor":
                given.append(None)
                continue

            def ghost(n, s=side):
                rows = range(-n, 0) if s == 0 else range(self.ny, self.ny + n)
                if not swept:
                    return self._taylor(range(self.nx), rows)
                return _sweep(self._taylor(range(-2, self.nx + 2), rows), 1, self.dt, self.beta)[0]
            given.append(ghost)
        return _pad(q, 0, 2, self.bc[2:], layers, given)

    def _dry(self):
        x = _roe(self._pad_x(self.q, 1), 1, self.beta)[3]
        y = self._pad_y(self.q, 1, False)
        return max(float(x.max()), float(_roe([y[0], y[2], y[1]], 0, self.beta)[3].max()))

    def _geometric(self, q):
        if self.w["geometry"] != "axisym":
            return q
        h = 0.5 * self.dt
        u, v = q[1] / (1.0 + q[0]), q[2] / (1.0 + q[0])
        return [q[0] - h * q[2] / self.r, q[1] - h * u * v / self.r, q[2] - h * v * v / self.r]

    def step(self):
        dt = self.dt
        q, sx = _sweep(self._pad_x(self.q, 2), 1, dt, self.beta)
        q = self._geometric(q)
        y = self._pad_y(q, 2, True)
        q, sy = _sweep([y[0], y[2], y[1]], 0, dt, self.beta)
        q = self._geometric([q[0], q[2], q[1]])
        u = [[m / (1.0 + p[0]) for m in p[1:]] for p in (q, self._pad_x(q, 1), self._pad_y(q, 1, False))]
        new = [q[0]]
        for k in range(2):
            c, x, y = u[0][k], u[1][k], u[2][k]
            lap = x[:, :-2] + x[:, 2:] + y[:-2] + y[2:] - 4.0 * c
            if self.w["geometry"] == "axisym":
                lap = lap + 0.5 * (y[2:] - y[:-2]) / self.r
                if k == 1:
                    lap = lap - c / (self.r * self.r)
            new.append(q[1 + k] + dt * self.delta * lap)
        nu = dt * max(sx, sy)
        self.dt = dt * 0.9 / nu
        if nu > 1.0:                      # redone with the smaller step
            return self.step()
        self.q = new
        self.t += dt
        return None


def _sweep3(q, kinds, dt):
    top = 0.0
    for a, d in ((0, 2), (1, 1), (2, 0)):
        order = [0, 1 + a] + [1 + b for b in range(3) if b != a]
        p = _pad(q, d, 1 + a, kinds[2 * a:2 * a + 2], 2)
        out, s = _sweep([p[k] for k in order], d, dt, WATER["beta"])
        top = max(top, s)
        q = [None] * 4
        for k, v in zip(order, out):
            q[k] = v
    return q, top


def _box(c, seed, dev):
    rho0, k = WATER["rho0"], WATER["rho0"] * WATER["c0"]
    q = [torch.from_numpy(a).to(dev) / f for a, f in zip(_fields3(c, seed), (rho0, k, k, k))]
    kinds, delta = SIDES3[c["sides"]], WATER["delta"] / (WATER["c0"] * 1e-4)
    dt = 0.9 / _sweep3(q, kinds, 0.0)[1]
    done = 0
    while done < c["steps"]:
        p, top = _sweep3(q, kinds, dt)
        nu = dt * top
        if nu <= 1.0:
            laps = [-6.0 * m / (1.0 + p[0]) for m in p[1:]]
            for a, d in ((0, 2), (1, 1), (2, 0)):
                e = _pad(p, d, 1 + a, kinds[2 * a:2 * a + 2], 1)
                n = p[0].shape[d]
                for m in range(3):
                    v = e[1 + m] / (1.0 + e[0])
                    laps[m] += v.narrow(d, 0, n) + v.narrow(d, 2, n)
            q = [p[0]] + [m + dt * delta * lap for m, lap in zip(p[1:], laps)]
            done += 1
        dt = dt * 0.9 / nu
    return q, (rho0, k, k, k)


def _packet(p, c, w):
    """The moving domain with its recorder: the runs' rules, step by step."""
    row_max = torch.zeros(w["path"], dtype=torch.float64, device=p.dev)
    pt, pr = (torch.zeros(4096, dtype=torch.float64, device=p.dev) for _ in range(2))
    x_off, phase, rho0 = 0, 0, w["medium"]["rho0"]
    quantum, t1 = w["window"]["quantum"], w["window"]["t1"] / p.unit
    for k in range(c["steps"]):
        p.step()
        row = p.q[0][0] * rho0
        n = max(0, min(p.nx, w["path"] - x_off))
        row_max[x_off:x_off + n] = torch.maximum(row_max[x_off:x_off + n], row[:n])
        if 0 <= w["probe_col"] - x_off < p.nx:
            pt[k], pr[k] = p.t * p.unit, row[w["probe_col"] - x_off]
        phase += 1
        if phase == w["window"]["check_every"]:
            phase = 0
            target = quantum * math.floor((p.t - t1) / quantum) if p.t >= t1 else 0
            if target > x_off:
                move = target - x_off
                p.q = [torch.cat([v[:, move:], torch.zeros_like(v[:, :min(move, p.nx)])], 1) for v in p.q]
                x_off = target
    return row_max, pt, pr, x_off


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    kind = case["kind"]
    if kind in ("box", "box_io"):
        q, fac = _box(case, seed, dev)
        if kind == "box":
            n = case["ny"] * case["nz"]
            q = [v.reshape(n, case["nx"]) for v in q]
            return {"R": q[0], "M": torch.stack(q[1:])}
        return tuple((v * f).cpu().numpy() for v, f in zip(q, fac))
    if kind == "batch":
        out = []
        for w in _members(case, seed):
            p = _Plane(w, dev)
            for _ in range(case["steps"]):
                p.step()
            out.append(torch.stack(p.q))
        return out
    w = _setup(case, seed)
    p = _Plane(w, dev)
    med = w["medium"]
    fac = (med["rho0"], med["rho0"] * med["c0"], med["rho0"] * med["c0"])
    si = lambda: tuple((v * f).cpu().numpy() for v, f in zip(p.q, fac))     # noqa: E731
    if kind == "packet":
        row_max, pt, pr, _ = _packet(p, case, w)
        return {"state": si(), "row_max": row_max, "probe_t": pt, "probe_rho": pr, "x_off": None}
    for _ in range(case["steps"]):
        p.step()
    if kind == "sampled":
        return {"state": torch.stack(p.q), "row": tuple(v[:1] for v in si()), "t": p.t * p.unit}
    if kind == "whole":
        # the sums of fields that cancel have no digits to compare
        return {"sums": None, "state": si()}
    return torch.stack(p.q) / (w["scale"] if "store" in w["precision"] else 1.0)
