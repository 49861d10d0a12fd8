"""Gray-level maps whose 24-bit product reaches 2^31 (windows of some thousand
values that the levels do not divide evenly): every kernel that maps voxels,
against the oracle.  The product taken as a signed number gave bins below 0."""
import numpy as np
import pytest

import oracle
from gpu_util import to_dev, u32

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2012_10684_amd import api  # noqa: E402

# (levels, values of the window): shifts 26 down to 20 of the product
WINDOWS = [(64, 7995), (100, 6693), (200, 7189), (250, 4097), (250, 3867), (256, 8564)]
MORE = [(1024, 2239), (2048, 7727), (4095, 1964), (4096, 3208)]


def _volume(W, n, size, seed):
    v = np.random.default_rng(seed).integers(-1024, -1024 + W, (n, size)).astype(np.int16)
    v[0, :2] = -1024 + W - 1, -1024 + W - 2
    return v


@pytest.mark.parametrize("L,W", WINDOWS + MORE)
def test_histograms(L, W):
    v, lo, hi = _volume(W, 3, 70001, L), -1024, -1024 + W - 1
    batch, binn = api.Batch([x for x in to_dev(v)]), api.binning(lo, hi, L)
    want = np.stack([oracle.histogram(x, lo, hi, L) for x in v])
    assert np.array_equal(u32(api.histogram(batch, binn)), want)
    if L < 2048:  # one workgroup, and several, per problem
        for parts in (1, 4):
            h, (thr, obj, st), _ = api.segment(batch, binn, 1, 0.8, tune={"segment_parts": parts})
            assert np.array_equal(u32(h), want)
            P, Q = api.prefix(h, 0.8)
            assert torch.equal(thr, api.threshold_search(P, Q, 1, 0.8)[0])
    h, _, _ = api.segment(api.Batch([to_dev(v[0])]), binn, 1, 0.8)  # one small problem
    assert np.array_equal(u32(h)[0], want[0])


@pytest.mark.parametrize("L,W", WINDOWS)
@pytest.mark.parametrize("width", [1, 64, 61])
def test_images(L, W, width):
    H = 7 if width == 1 else 45  # 7 pixels: the kernel of tiny images
    v, lo, hi = _volume(W, 2, H * width, L).reshape(2, H, width), -1024, -1024 + W - 1
    b, binn = api.Batch.slices(to_dev(v)), api.binning(lo, hi, L)
    h = u32(api.histogram2d(b, H, width, binn))
    o, r, r16 = (x.cpu().numpy() for x in api.open2d(b, H, width, binn, 2, want=("opened", "residue", "residue16")))
    for i in range(2):
        assert np.array_equal(h[i], oracle.histogram2d(v[i], lo, hi, L))
        wo, wr = oracle.opening(oracle.gray(v[i], lo, hi, L), 2)
        assert np.array_equal(o[i], wo) and np.array_equal(r[i], wr) and np.array_equal(r16[i], wr)
