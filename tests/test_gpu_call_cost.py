"""Host time of calls of one step: the launch geometry is settled when the
handle's settings change, not per call."""
import time

import pytest

from gpu_util import say
from paper_2609_09160_amd import inputs

pytestmark = pytest.mark.gpu


def _us_per_call(shape, phase):
    import numpy as np
    from paper_2609_09160_amd import Solver
    s = Solver(shape, 0.8)
    s.set_moments(inputs.random_state(shape, seed=1))
    if phase:
        s.enable_two_phase(0.03, 4.0, 0.1)
        s.set_phase(np.full(shape[::-1], 0.5))
    s.step(10)
    s.sync()
    best = 1e9
    for _ in range(20):
        t = time.perf_counter()
        for _ in range(20):
            s.step(1)
        best = min(best, (time.perf_counter() - t) / 20)
        s.sync()
    s.close()
    return best * 1e6


@pytest.mark.parametrize("phase", [False, True])
def test_a_call_costs_the_same_on_a_long_grid(phase):
    """4 x 4 x 100000 has 600 chunk lengths to choose from, 4 x 4 x 64 a dozen:
    the choice is not in the call (where it was, 11 us against 3, with two
    components 18 against 5)."""
    short, long = _us_per_call((4, 4, 64), phase), _us_per_call((4, 4, 100000), phase)
    say(f"host us per step call, two components {phase}: {short:.2f} short, {long:.2f} long")
    assert long <= 1.5 * short + 1.0
