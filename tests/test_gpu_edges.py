"""Edges of the launch rules: fixed steps replayed in chunks against single
steps, the state record of the no-allocation evaluation, and the surrogate's
convolution kernels at sides around their tiles."""
import numpy as np
import pytest

import workloads
from oracle import surrogate as osg
from test_gpu_surrogate import LAYERS, bf16, rel_max, rounded_params

pytestmark = pytest.mark.gpu


# 15: single steps; 16: two chunks of eight; 17, 31: chunks and singles
@pytest.mark.parametrize("nsteps", [15, 16, 17, 31])
@pytest.mark.parametrize("method,n", [("euler", (33, 20, 1)), ("heun", (33, 20, 1)), ("rk3", (33, 20, 1)),
                                      ("rk4", (33, 20, 1)), ("heun", (12, 10, 4)), ("rk4", (40, 50, 20))])
def test_step_chunks_equal_single_steps(lib, method, n, nsteps):
    """One call of many steps and as many calls of one step: the same bits
    (thermal field on: every step draws by its own counter)."""
    out = []
    for split in (False, True):
        prob, m0 = workloads.small_problem(n, seed=4, alpha=0.2, T=300.0)
        s = lib.Solver(0)
        s.set_problem(prob)
        s.set_m(m0)
        if split:
            for _ in range(nsteps):
                s.step(method, 5e-14, 1)
        else:
            s.step(method, 5e-14, nsteps)
        out.append((s.get_m(), s.stats()))
        s.close()
    assert np.array_equal(out[0][0], out[1][0])
    assert out[0][1] == out[1][1]


@pytest.mark.parametrize("T", [0.0, 300.0])
def test_noalloc_follows_the_step_counter(lib, T):
    """The draw of the no-allocation evaluation moves with the solver's steps."""
    import torch

    prob, m0 = workloads.small_problem((30, 20, 1), seed=6, alpha=0.2, T=T)
    s = lib.Solver(0)
    s.set_problem(prob)
    s.set_m(m0)
    for _ in range(3):
        s.step("heun", 5e-14, 2)
        h = s.eval_heff()
        m_dev = torch.from_numpy(s.get_m()).to("cuda:0")
        h_dev = torch.empty_like(m_dev)
        torch.cuda.synchronize()
        s.eval_heff_noalloc(m_dev, h_dev)
        assert np.array_equal(h_dev.cpu().numpy().reshape(-1), np.asarray(h).reshape(-1))
    s.close()


@pytest.mark.parametrize("layer", [0, 2, 5])
@pytest.mark.parametrize("H,W", [(1, 1), (1, 16), (3, 15), (2, 17), (5, 63), (4, 64), (3, 65), (17, 130)])
def test_conv_sides(lib, layer, H, W):
    """Forward, weight, bias and input gradients of one layer against the FP64
    oracle on the same BF16 operands (FP32 sums of at most 288 products or
    H W N pixels: 1e-5 of the largest value)."""
    N = 2
    ci, co = LAYERS[layer]
    params = rounded_params(3)
    sur = lib.Surrogate(H, W, max_batch=N)
    sur.set_params(params)
    rng = np.random.default_rng(100 * H + W + layer)
    x = bf16(rng.standard_normal((N, H, W, 32)))
    gy = bf16(rng.standard_normal((N, H, W, 32)))
    y, gx, gw, gb = sur.conv_check(layer, x, gy)
    w, b = params[layer]
    gw_ref = np.zeros_like(w)
    gb_ref = np.zeros_like(b)
    for n in range(N):
        xo = x[n, :, :, :ci].transpose(2, 0, 1).astype(np.float64)
        go = gy[n, :, :, :co].transpose(2, 0, 1).astype(np.float64)
        y_ref = osg.conv3x3(xo, w, b)
        gx_ref, gwn, gbn = osg.conv3x3_backward(xo, w, go)
        gw_ref += gwn
        gb_ref += gbn
        assert rel_max(y[n, :, :, :co].transpose(2, 0, 1), y_ref) <= 1e-5
        assert rel_max(gx[n, :, :, :ci].transpose(2, 0, 1), gx_ref) <= 1e-5
    assert rel_max(gw, gw_ref) <= 1e-5
    assert rel_max(gb, gb_ref) <= 1e-5
