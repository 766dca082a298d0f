"""The no-allocation evaluation of a field that starts on any float of the
caller's memory (a slice of a larger tensor), on geometries whose rows are read
16 bytes at a time: the same bits as from aligned memory."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,pbc", [((100, 36, 1), (False,) * 3), ((256, 64, 1), (False,) * 3), ((48, 36, 1), (True, True, False)),
                                   ((40, 20, 5), (False,) * 3), ((64, 32, 16), (True, False, False))])
def test_field_on_any_float(lib, n, pbc):
    import torch

    prob, m0 = workloads.small_problem(n, pbc=pbc, seed=n[0])
    s = lib.Solver(0)
    s.set_problem(prob)
    s.set_m(m0)
    ref = np.asarray(s.eval_heff()).reshape(-1)
    m = torch.from_numpy(s.get_m()).reshape(-1).to("cuda:0")
    for off in (0, 1, 2, 3):
        src = torch.zeros(m.numel() + 8, device="cuda:0")
        dst = torch.zeros(m.numel() + 8, device="cuda:0")
        src[off:off + m.numel()] = m
        torch.cuda.synchronize()
        shape = (3, n[2], n[1], n[0])
        s.eval_heff_noalloc(src[off:off + m.numel()].view(shape), dst[off:off + m.numel()].view(shape))
        out = dst.cpu().numpy()
        assert np.array_equal(out[off:off + m.numel()], ref), off
        assert not out[:off].any() and not out[off + m.numel():].any()
    s.close()
