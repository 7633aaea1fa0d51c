"""The moving domain decided on the device (fvna_step_window) against the same
rule applied by the host with fvna_step and fvna_shift, and the recorder
against rows read back after every step: bit for bit, also when a rejected
attempt delays a check, for calls that end between checks, checks further
apart than a captured graph and the largest jump."""
import math

import numpy as np
import pytest

from common import pulse_workload

pytestmark = pytest.mark.gpu
C0, DX = 1500.0, 1e-4


def sim(precision, dt0, tile_rows, bc=("extrap0",) * 4, taylor=None):
    from paper_1311_3004_amd import fvna
    w = pulse_workload(150, 70, bc, seed=5, taylor=taylor)
    return fvna.sim_from_workload(w, precision=precision, dt0=dt0, tile_rows=tile_rows)


def host_rule(s, calls, t1, every, quantum, speed):
    """fvna_window's rule with the entry points that leave the decision to the
    host; the row and clock after every step."""
    x_off = phase = 0
    rows, ts = [], []
    for n in calls:
        for _ in range(n):
            s.fvna_step(1)
            rows.append((x_off, s.fvna_get_window(0, 9, 150, 1)[0][0]))
            ts.append(s.fvna_get_stats()["t"])
            phase += 1
            if phase < every:
                continue
            phase = 0
            t = ts[-1] * C0 / DX
            target = quantum * math.floor((t - t1) * speed / quantum) if t >= t1 else 0
            if target > x_off:
                s.fvna_shift(target - x_off)
                x_off = target
    return x_off, phase, rows, ts


@pytest.mark.parametrize("precision,tile_rows", [("f64", 0), ("f32", 0), ("f32_bf16store", 16), ("f64", 16)])
@pytest.mark.parametrize("calls,t1,every,quantum,speed,reject", [
    ([40], 4.0, 4, 3, 1.0, False),
    ([40], 4.0, 4, 3, 1.0, True),             # the first attempt is rejected: every check comes one attempt later
    ([1, 2, 7, 30], 0.0, 5, 5, 1.3, True),
    ([90], 10.0, 45, 1, 0.7, True),
    ([12], 0.0, 3, 7, 40.0, False),           # moves of more columns than the grid has
])
def test_moving_domain_on_the_device_equals_the_host_rule(precision, tile_rows, calls, t1, every, quantum, speed, reject):
    import torch
    from paper_1311_3004_amd import fvna
    dt0 = 3.0 * 0.9 * DX / C0 if reject else 0.0
    a, b = (sim(precision, dt0, tile_rows) for _ in range(2))
    steps, path, probe = sum(calls), 400, 60
    row_max = torch.full((path,), -math.inf, dtype=torch.float64, device="cuda")
    pt, pr = (torch.full((steps + 4,), math.nan, dtype=torch.float64, device="cuda") for _ in range(2))
    torch.cuda.synchronize()
    a.fvna_set_recorder(9, probe, path, row_max, pt, pr)
    # C0 / DX converts times to cells; t1 in seconds gives the same cells back
    win, state = fvna.fvna_window(t1 * DX / C0, every, quantum, speed), fvna.fvna_window_state(0, 0)
    for n in calls:
        a.fvna_step_window(win, state, n)
    x_off, phase, rows, ts = host_rule(b, calls, win.t1 * C0 / DX, every, quantum, speed)
    assert (state.x_off, state.phase) == (x_off, phase)
    sa, sb = a.fvna_get_stats(), b.fvna_get_stats()
    assert sa == sb and sa["steps"] == steps and sa["rejected"] == (1 if reject else 0)
    for x, y in zip(a.fvna_get_state(), b.fvna_get_state()):
        assert np.array_equal(x, y)
    want = np.full(path, -math.inf)
    for off, row in rows:
        n = max(0, min(150, path - off))
        want[off:off + n] = np.maximum(want[off:off + n], row[:n])
    assert np.array_equal(row_max.cpu().numpy(), want)
    got_t, got_r = pt.cpu().numpy(), pr.cpu().numpy()
    for k, (off, row) in enumerate(rows):
        if off <= probe < off + 150:
            assert got_t[k] == ts[k] and got_r[k] == row[probe - off]
        else:
            assert math.isnan(got_t[k])
    assert np.isnan(got_t[steps:]).all()
    a.fvna_destroy()
    b.fvna_destroy()


def test_moving_domain_with_steps_owed_and_with_a_latched_error():
    """Steps owed from a rejected fvna_step are completed before the rule's
    own; an error latched before the call is returned and nothing moves."""
    from paper_1311_3004_amd import fvna
    dt0 = 3.0 * 0.9 * DX / C0
    a, b = (sim("f64", dt0, 0) for _ in range(2))
    win, state = fvna.fvna_window(0.0, 3, 2, 1.0), fvna.fvna_window_state(0, 0)
    a.fvna_step(5)                             # one attempt is rejected: a step stays owed
    a.fvna_step_window(win, state, 9)
    b.fvna_step(5)
    b.fvna_sync()
    other = fvna.fvna_window_state(0, 0)
    b.fvna_step_window(win, other, 9)
    assert (state.x_off, state.phase) == (other.x_off, other.phase)
    assert a.fvna_get_stats() == b.fvna_get_stats()
    for x, y in zip(a.fvna_get_state(), b.fvna_get_state()):
        assert np.array_equal(x, y)
    bad = sim("f64", dt0, 0)
    bad.params.max_retries = 0
    c = fvna.Sim(bad.params)
    c.fvna_set_state(*pulse_workload(150, 70, ("extrap0",) * 4, seed=5)["state"])
    c.fvna_step(1)
    st = fvna.fvna_window_state(0, 0)
    with pytest.raises(fvna.FvnaError):
        c.fvna_step_window(win, st, 6)
    assert (st.x_off, st.phase) == (0, 0)
    assert c.fvna_get_stats(allow_device_errors=True)["steps"] == 0
