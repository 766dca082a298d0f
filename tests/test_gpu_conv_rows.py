"""The surrogate's convolutions where a block works through many rows: the
six-step rotation of the row fragments and its wrap, the two-rows-ahead reads,
ragged last blocks, and launches of more than one round of blocks."""
import numpy as np
import pytest

from oracle import surrogate as osg
from test_gpu_surrogate import LAYERS, bf16, rel_max, rounded_params

pytestmark = pytest.mark.gpu

ROUND = 5 * 256      # forward blocks the card holds at a time


def block_rows(N, H, W):
    """Rows of a forward block (at most 24, whole rounds of blocks, an image's
    rows dealt evenly over its blocks)."""
    rb = (W + 63) // 64 * H * N
    rounds = -(-rb // (ROUND * 24))
    most = -(-rb // (ROUND * rounds))
    parts = -(-H // most)
    return -(-H // parts), rounds


# (layer, N, H, W): rows per forward block, the last block's, rounds
@pytest.mark.parametrize("layer,N,H,W,rows,last,rounds", [
    (2, 128, 62, 5, 7, 6, 1),        # one row past the rotation
    (2, 128, 31, 66, 7, 3, 1),       # two column tiles
    (0, 160, 77, 5, 10, 7, 1),
    (5, 160, 77, 5, 10, 7, 1),
    (1, 64, 256, 3, 13, 9, 1),       # as 16 states of 256 x 256
    (2, 320, 95, 2, 24, 23, 1),      # the longest block
    (2, 160, 211, 3, 14, 1, 2),      # two rounds, a last block of one row
    (0, 1111, 12, 12, 6, 6, 1),      # 11 rows fit, dealt evenly
])
def test_conv_many_rows(lib, layer, N, H, W, rows, last, rounds):
    """Forward, weight, bias and input gradients of one layer against the FP64
    oracle on the same BF16 operands (FP32 sums of at most 288 products or H W N
    pixels: 1e-5 of the largest value)."""
    assert block_rows(N, H, W) == (rows, rounds) and (H % rows or rows) == last
    ci, co = LAYERS[layer]
    params = rounded_params(3)
    sur = lib.Surrogate(H, W, max_batch=N)
    sur.set_params(params)
    rng = np.random.default_rng(N + H)
    x = bf16(rng.standard_normal((N, H, W, 32)))
    gy = bf16(rng.standard_normal((N, H, W, 32)))
    y, gx, gw, gb = sur.conv_check(layer, x, gy)
    w, b = params[layer]
    gw_ref = np.zeros_like(w)
    gb_ref = np.zeros_like(b)
    for n in range(N):
        xo = x[n, :, :, :ci].transpose(2, 0, 1).astype(np.float64)
        go = gy[n, :, :, :co].transpose(2, 0, 1).astype(np.float64)
        gx_ref, gwn, gbn = osg.conv3x3_backward(xo, w, go)
        gw_ref += gwn
        gb_ref += gbn
        assert rel_max(y[n, :, :, :co].transpose(2, 0, 1), osg.conv3x3(xo, w, b)) <= 1e-5
        assert rel_max(gx[n, :, :, :ci].transpose(2, 0, 1), gx_ref) <= 1e-5
    assert rel_max(gw, gw_ref) <= 1e-5
    assert rel_max(gb, gb_ref) <= 1e-5
