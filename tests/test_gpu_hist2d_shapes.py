"""2D histograms at the edges of the counting kernel's layout, against the
oracle, bit for bit: widths around the lanes' 8 columns, the row groups of 16,
32 and 64 lanes and the chunks of wide rows; more images than workgroups
(whole images stored, the rest split); image starts at odd addresses; cells
past 16 bits (one gray level, two levels, clamp corners)."""
import numpy as np
import pytest

import oracle
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2012_10684_amd import api  # noqa: E402


def _check(imgs, lo, hi, L, dv=None):
    n, H, W = imgs.shape
    dv = to_dev(imgs) if dv is None else dv
    h = api.histogram2d(api.Batch([d.reshape(-1) for d in dv]), H, W, api.binning(lo, hi, L)).cpu().numpy()
    for i in range(n):
        want = oracle.histogram2d(imgs[i], lo, hi, L)
        assert np.array_equal(h[i].view(np.uint32), want), i


@pytest.mark.parametrize("W", [1, 2, 7, 8, 9, 120, 127, 128, 129, 136, 255, 256, 257, 415, 511, 512, 513, 520, 1023,
                               1025, 2056, 4095, 4096])
def test_widths(W):
    rng = np.random.default_rng(W)
    for H in (1, 2, 35):
        _check(rng.normal(-600, 400, (2, H, W)).clip(-32768, 32767).astype(np.int16), -1024, -200, 256)


@pytest.mark.parametrize("n,H,W,L", [(300, 20, 24, 16), (520, 33, 40, 15), (257, 17, 130, 31), (5, 700, 64, 255)])
def test_many_images(n, H, W, L):
    rng = np.random.default_rng(n)
    _check(rng.integers(-40, 300, (n, H, W)).astype(np.int16), 0, 255, L)


def test_odd_starts():
    rng = np.random.default_rng(8)
    H, W = 37, 61
    flat = rng.integers(0, 256, 3 * H * W + 1).astype(np.int16)
    imgs = flat[1:].reshape(3, H, W)
    _check(imgs, 0, 255, 100, dv=to_dev(flat)[1:].reshape(3, H, W))


@pytest.mark.parametrize("n", [1, 256])
def test_cells_past_16_bits(n):
    H, W = (900, 512) if n == 1 else (300, 260)  # one workgroup counts 78000 pixels of an image with n = 256
    base = np.zeros((4, H, W), np.int16)
    base[0] = 77                 # one inner cell
    base[1, :, ::2] = 40         # two levels in turn: few cells
    base[2] = 255                # the upper corner
    base[3, : H // 2] = 9        # half a level, half the lower corner
    imgs = base[:n] if n < 4 else np.concatenate([base, np.full((n - 4, H, W), 13, np.int16)])
    _check(imgs, 0, 255, 256)
