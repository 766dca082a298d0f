"""The memory a surrogate holds for the weight gradients, and that the gradients
do not depend on it."""
import numpy as np
import pytest

from oracle import surrogate as osg

pytestmark = pytest.mark.gpu


def test_partials_are_bounded_and_the_gradients_the_same(lib):
    """8 x 8 films: a batch of up to 8192 holds at least one weight-gradient
    block (36 KiB a layer) per film, 302 MB for one layer and 1.8 GB for all.
    A step on three films gives the same bits whether the partial sums of all
    layers are held or of one."""
    import torch

    H = W = 8
    N = 8192
    rng = np.random.default_rng(1)
    m = rng.standard_normal((2, 3, 3, H, W)).astype(np.float32)
    m /= np.linalg.norm(m, axis=2, keepdims=True)
    B = rng.uniform(-0.03, 0.03, (3, 3))
    flat = lib.Surrogate.pack(osg.init_params(2))
    torch.cuda.synchronize()
    out = []
    for cap in (3, N):
        before = torch.cuda.mem_get_info(0)[0]
        sur = lib.Surrogate(H, W, max_batch=cap)
        used = before - torch.cuda.mem_get_info(0)[0]
        if cap == N:
            cells, layer = N * H * W, N * 9 * 32 * 32 * 4
            print("held", used / 1e6, "MB", flush=True)
            assert used <= 1444 * cells + 1.1 * layer + (64 << 20)
        sur.set_params(flat)
        loss = [sur.train_step(m[0], m[1], B, lr=1e-3) for _ in range(2)]
        out.append((loss, sur.get_grads(), sur.get_params()))
        sur.close()
    assert out[0][0] == out[1][0]
    assert np.array_equal(out[0][1], out[1][1]) and np.any(out[0][1])
    assert np.array_equal(out[0][2], out[1][2])
