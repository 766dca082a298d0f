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


@pytest.mark.parametrize("n", [(768, 32), (32, 768), (768, 768)])
def test_variants_of_1536_and_768(lib, default_variants, n):
    """Rows of 1536 points and columns of 768 halves in every variant, alone
    and in a batch, against the oracle."""
    prob, m0 = workloads.small_problem((n[0], n[1], 1), seed=n[0] + n[1])
    ref = fields.heff(m0.astype(np.float64), prob)
    s = lib.Solver(0)
    s.set_problem(prob)
    tried = 0
    for rv in range(2):
        for cv in range(2):
            try:
                s.set_variants(rv, cv)
            except lib.LLGError as err:
                assert err.code == lib.LLG_E_ARG and (rv, cv) != (0, 0)
                print(n, "variants", (rv, cv), "refused", flush=True)
                continue
            s.set_m(m0)
            e = maxrel(s.eval_heff(), ref)
            print(n, "variants", (rv, cv), e, flush=True)
            assert e <= 1e-5
            s.step("rk4", 1e-14, 2)
            b = lib.Batch([(prob, m0)])
            b.step("rk4", 1e-14, 2)
            assert np.array_equal(b.get_m(0), s.get_m())
            b.close()
            tried += 1
    s.close()
    assert tried >= 2
