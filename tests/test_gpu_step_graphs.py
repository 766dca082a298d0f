"""Which graphs replay a call of fixed steps: the same bits and counters as
single steps, whichever it is."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


# 16 steps of three or more stages on their own: single steps; a second 16, one
# after a short call, 24 at once, or two stages: eight steps a graph; a new dt
# or method: anew
@pytest.mark.parametrize("n", [(33, 20, 1), (12, 10, 4)])
def test_step_graphs_equal_single_steps(lib, n):
    calls = [("heun", 5e-14, 16), ("heun", 4e-14, 17), ("rk4", 4e-14, 16), ("rk4", 4e-14, 16), ("rk4", 2e-14, 3),
             ("rk4", 2e-14, 17), ("rk3", 3e-14, 24), ("rk3", 3e-14, 9), ("euler", 1e-14, 25)]
    out = []
    for split in (False, True):
        prob, m0 = workloads.small_problem(n, seed=9, alpha=0.2, T=300.0)
        s = lib.Solver(0)
        s.set_problem(prob)
        s.set_m(m0)
        got = []
        for method, dt, k in calls:
            for _ in range(k if split else 1):
                s.step(method, dt, 1 if split else k)
            got.append(s.get_m())
        out.append((got, s.stats()))
        s.close()
    for a, b in zip(out[0][0], out[1][0]):
        assert np.array_equal(a, b)
    assert out[0][1] == out[1][1]
