"""Shapes on both sides of the padding rule, and films periodic in y with fewer
rows than a block holds: as in test_gpu_padding.py, against the oracle and the
runtime-length kernels."""
import pytest

from test_gpu_padding import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,pbc", [
    ((64, 5, 1), (True, True, False)), ((192, 3, 1), (True, True, False)), ((128, 4, 1), (False, True, False)),
    # more than 256 planes, more than 512 cells along y: runtime-length passes
    # beside padded and unpadded axes
    ((5, 3, 258), (False,) * 3), ((63, 4, 260), (False,) * 3), ((6, 31, 257), (False,) * 3),
    ((4, 6, 270), (False, False, True)), ((5, 520, 3), (False,) * 3), ((63, 513, 2), (False,) * 3),
    ((40, 515, 3), (False,) * 3), ((4, 525, 10), (False, True, False))])
def test_shapes(lib, monkeypatch, n, pbc):
    check(lib, monkeypatch, n, pbc)
