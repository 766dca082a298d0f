"""Compiled variants beyond the tuners' own tests: the table's row variants in
3D, and the lengths added last."""
import numpy as np
import pytest

import workloads
from oracle import fields

pytestmark = pytest.mark.gpu


def maxrel(a, b):
    a = np.asarray(a, dtype=np.float64).reshape(3, -1)
    b = np.asarray(b, dtype=np.float64).reshape(3, -1)
    return float(np.max(np.linalg.norm(a - b, axis=0)) / np.max(np.linalg.norm(b, axis=0)))


@pytest.mark.parametrize("nx", [32, 96])
def test_3d_rows_follow_the_table(lib, default_variants, nx):
    """A 3D grid copies the row variant that a tuning call set for its length
    (the variants differ in rounding, each within the FP32 bar of the oracle)."""
    prob, m0 = workloads.small_problem((nx, 16, 4), seed=nx)
    ref = fields.heff(m0.astype(np.float64), prob)
    t = lib.Solver(0)
    t.set_geometry((nx, 32, 1))
    out = []
    for var in (0, 1):
        t.set_variants(var, 0)
        s = lib.Solver(0)
        s.set_problem(prob)
        s.set_m(m0)
        out.append(np.asarray(s.eval_heff()))
        assert maxrel(out[-1], ref) <= 1e-5
        s.close()
    t.close()
    assert not np.array_equal(out[0], out[1])
