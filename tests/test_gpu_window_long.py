"""Long calls of fvna_step_window: the host looks at the clock in between, so
that a call whose simulation has failed ends early, and the steps and moves are
those of the rule applied by the host."""
import time

import pytest

from common import pulse_workload
from test_gpu_window_device import C0, DX, test_moving_domain_on_the_device_equals_the_host_rule as same_as_host_rule

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("calls,every,speed,reject", [
    ([2500], 5, 1.0, True),              # the attempts between two looks end inside a segment
    ([1024, 1400], 4, 1.0, False),       # and at its end
    ([1300, 1200], 1100, 0.05, True),   # segments longer than that (slow: the host rule moves nx cells at most)
])
def test_long_calls_equal_the_host_rule(calls, every, speed, reject):
    same_as_host_rule("f64", 0, calls, 4.0, every, 3, speed, reject)


def test_a_call_ends_soon_after_an_error():
    from paper_1311_3004_amd import fvna
    w = pulse_workload(150, 70, ("extrap0",) * 4, seed=5)
    s = fvna.sim_from_workload(w, precision="f64", dt0=3.0 * 0.9 * DX / C0, max_retries=0)

    def failing(n):
        st = fvna.fvna_window_state(0, 0)
        t = time.perf_counter()
        with pytest.raises(fvna.FvnaError):
            s.fvna_step_window(fvna.fvna_window(0.0, 5, 2, 1.0), st, n)
        assert (st.x_off, st.phase) == (0, 0)
        return time.perf_counter() - t
    failing(10)
    short, long = min(failing(1000) for _ in range(3)), min(failing(40000) for _ in range(3))
    assert long < 5 * short + 0.01
    assert s.fvna_get_stats(allow_device_errors=True)["steps"] == 0
    s.fvna_destroy()
