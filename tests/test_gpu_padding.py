"""Geometries whose shortest FFT lengths have no compiled kernels run on the
next compiled lengths (zero padding beyond 2n - 1 leaves the convolution
unchanged): H_eff and steps with every term on against the FP64 oracle, and
against the runtime-length kernels at the shortest lengths
(LLG_FORCE_GENERIC).  FP32 bar: 1e-5 max-relative, as for every H_eff."""
import numpy as np
import pytest

import workloads
from oracle import fields, llg as ollg

pytestmark = pytest.mark.gpu

ALL = dict(alpha=0.3, Kc1=4e3, Kc2=2e3, c1=(1.0, 0.0, 0.0), c2=(0.0, 1.0, 0.0), j=(1e12, 2e11, 0.0), P=0.5, xi=0.05)

# smallest, odd, both sides of the 1024 / 1536 / 2048 row and 512 / 768 / 1024
# column lengths, periodic rows of compiled length
FILMS = [((1, 1), (False, False)), ((3, 2), (False, False)), ((33, 2), (False, False)), ((100, 37), (False, False)),
         ((250, 63), (False, False)), ((513, 40), (False, False)), ((767, 33), (False, False)),
         ((768, 768), (False, False)), ((600, 520), (False, False)), ((769, 35), (False, False)),
         ((40, 769), (False, False)), ((1000, 5), (False, False)), ((64, 50), (True, False)),
         ((256, 31), (True, False)),
         # periodic y, or periodic x of no compiled length: padded with the
         # kernel continued periodically
         ((50, 64), (False, True)), ((100, 37), (True, False)), ((6, 5), (True, True)), ((48, 35), (True, True)),
         ((64, 49), (True, True)), ((33, 3), (False, True)), ((70, 64), (True, True)), ((1000, 6), (True, False)),
         ((8, 1000), (True, True))]


# 3D: the planes of the register z pass (2 ... 8) and beyond, both sides of
# the 16 ... 512 column lengths, every mix of periodic axes
BLOCKS = [((20, 12, nz), (False,) * 3) for nz in (2, 3, 4, 5, 6, 7, 8, 9)] + \
    [((100, 60, 20), (False,) * 3), ((33, 17, 24), (False,) * 3), ((6, 5, 25), (False,) * 3), ((9, 33, 48), (False,) * 3),
     ((8, 6, 97), (False,) * 3), ((6, 97, 5), (False,) * 3), ((7, 193, 3), (False,) * 3), ((6, 300, 2), (False,) * 3),
     ((4, 400, 3), (False,) * 3), ((70, 6, 17), (False,) * 3), ((24, 10, 3), (True, False, False)),
     ((64, 10, 3), (True, False, False)), ((30, 24, 5), (False, True, False)), ((30, 96, 4), (False, True, False)),
     ((40, 48, 9), (True, True, False)), ((14, 192, 2), (False, True, False)), ((20, 9, 6), (False, False, True)),
     ((20, 18, 4), (True, True, True)), ((10, 9, 10), (True, True, True)), ((6, 100, 3), (False, True, True)),
     ((6, 10, 40), (False, False, True)), ((12, 7, 8), (True, True, True))]


def maxrel(a, b):
    a = np.asarray(a, dtype=np.float64).reshape(3, -1)
    b = np.asarray(b, dtype=np.float64).reshape(3, -1)
    return float(np.max(np.linalg.norm(a - b, axis=0)) / np.max(np.linalg.norm(b, axis=0)))


def results(lib, prob, m0):
    s = lib.Solver(0)
    s.set_problem(prob)
    s.set_m(m0)
    h = s.eval_heff()
    s.step("rk4", 5e-14, 3)
    m = s.get_m()
    s.set_m(m0)
    s.run(5e-13, 1e-5, 1e-14)
    out = h, m, s.get_m(), s.attempts()
    s.close()
    return out


def check(lib, monkeypatch, n, pbc):
    prob, m0 = workloads.small_problem(n, pbc=pbc, seed=n[0] + 3 * n[1] + 7 * n[2], **ALL)
    monkeypatch.delenv("LLG_FORCE_GENERIC", raising=False)
    h, m, ma, att = results(lib, prob, m0)
    eh = maxrel(h, fields.heff(m0.astype(np.float64), prob))
    o = ollg.Solver(prob, m0)
    o.step("rk4", 5e-14, 3)
    em = maxrel(m, o.m)
    o = ollg.Solver(prob, m0)
    o.replay([(dt, ok) for dt, _, ok in att])
    ea = maxrel(ma, o.m)
    monkeypatch.setenv("LLG_FORCE_GENERIC", "1")
    hg, mg, mag, _ = results(lib, prob, m0)
    print(n, pbc, "H_eff", eh, "rk4", em, "dp45", ea, "against runtime-length kernels", maxrel(h, hg), maxrel(m, mg),
          flush=True)
    assert max(eh, em, ea) <= 1e-5
    assert max(maxrel(h, hg), maxrel(m, mg)) <= 1e-5


@pytest.mark.parametrize("n,pbc", FILMS)
def test_films(lib, monkeypatch, n, pbc):
    check(lib, monkeypatch, (n[0], n[1], 1), (pbc[0], pbc[1], False))


@pytest.mark.parametrize("n,pbc", BLOCKS)
def test_blocks(lib, monkeypatch, n, pbc):
    check(lib, monkeypatch, n, pbc)


def test_tuning_calls_as_before(lib):
    """The tuning calls serve the geometries whose shortest lengths are
    compiled, and refuse the others, which run on longer ones."""
    s = lib.Solver(0)
    for n, ok in (((250, 64, 1), False), ((256, 63, 1), False), ((256, 64, 1), True), ((768, 768, 1), True)):
        prob, m0 = workloads.small_problem(n)
        s.set_problem(prob)
        if ok:
            assert s.get_variants() == (0, 0)
            continue
        s.set_m(m0)
        for call in (lambda: s.get_variants(), lambda: s.set_variants(0, 0), lambda: s.autotune(1)):
            with pytest.raises(lib.LLGError) as e:
                call()
            assert e.value.code == lib.LLG_E_UNSUPPORTED
    with pytest.raises(lib.LLGError) as e:       # x padded beyond 2048 and no compiled 4096
        s.set_geometry((1100, 8, 1))
    assert e.value.code == lib.LLG_E_UNSUPPORTED
    s.close()


def test_noalloc_beyond_the_static_array(lib):
    """A geometry whose spectra fit the static array at the shortest lengths
    (27.6 MB) but not at the compiled ones (71 MB): accepted, the same bits as
    the ordinary evaluation."""
    import torch

    prob, m0 = workloads.small_problem((140, 100, 40), pbc=(False, True, False), seed=5)
    s = lib.Solver(0)
    s.set_problem(prob)
    s.set_m(m0)
    h = s.eval_heff()
    m_dev = torch.from_numpy(s.get_m()).to("cuda:0")
    h_dev = torch.empty_like(m_dev)
    torch.cuda.synchronize()
    for _ in range(2):
        s.eval_heff_noalloc(m_dev, h_dev)
        assert np.array_equal(h_dev.cpu().numpy().reshape(-1), np.asarray(h).reshape(-1))
    s.close()
