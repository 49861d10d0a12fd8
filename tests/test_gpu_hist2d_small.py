"""2D histograms of narrow, flat and small images and of few levels, against the
oracle: row groups of one lane upwards, several workgroups per CU, a second
round of whole images, copies of the plane with counts past 16 bits; and their
time against images that fill the lanes."""
import numpy as np
import pytest

import oracle
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2012_10684_amd import api  # noqa: E402


def _check(imgs, lo, hi, L, every=1):
    n, H, W = imgs.shape
    h = api.histogram2d(api.Batch.slices(to_dev(imgs)), H, W, api.binning(lo, hi, L)).cpu().numpy()
    assert (h.view(np.uint32).reshape(n, -1).sum(1) == H * W).all()
    for i in range(0, n, every):
        assert np.array_equal(h[i].view(np.uint32), oracle.histogram2d(imgs[i], lo, hi, L)), i


@pytest.mark.parametrize("W", [1, 3, 8, 9, 16, 17, 31, 32, 33, 64, 65, 127])
@pytest.mark.parametrize("n,H,L", [(1, 9, 256), (1, 3000, 64), (5, 700, 30), (2, 1030, 256)])
def test_narrow(n, H, W, L):
    rng = np.random.default_rng(W + H)
    _check(rng.normal(-600, 400, (n, H, W)).clip(-32768, 32767).astype(np.int16), -1024, -200, L)


# images per CU: up to one, up to two, more; planes per CU: one, four, eight
@pytest.mark.parametrize("n", [4, 256, 257, 512, 513, 2100])
@pytest.mark.parametrize("H,W,L", [(1, 40, 256), (8, 8, 64), (33, 21, 64), (1, 2049, 16), (64, 64, 128), (65, 66, 130)])
def test_many_small(n, H, W, L):
    rng = np.random.default_rng(n + W)
    _check(rng.integers(-40, L + 20, (n, H, W)).astype(np.int16), 0, L - 1, L, every=max(1, n // 40))


@pytest.mark.parametrize("L", [2, 15, 32, 33])
@pytest.mark.parametrize("n,H,W", [(3, 2600, 2600), (300, 250, 225)])
def test_few_levels(n, H, W, L):
    rng = np.random.default_rng(L)
    v = rng.integers(0, L, (n, H, W)).astype(np.int16)
    v[0] = L // 2                 # one cell with every pixel
    v[1, :, ::2] = L - 1          # two levels in turn
    v[n - 1, : H // 2] = 0        # the lower corner and the rest
    _check(v, 0, L - 1, L, every=max(1, n // 12))
    _check(np.concatenate([v[:2], v[-1:]]), 0, L - 1, L)


def _us(f, reps=9, calls=20):
    f()
    t = []
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(calls):
            f()
        b.record()
        b.synchronize()
        t.append(a.elapsed_time(b) * 1e3 / calls)
    return sorted(t)[reps // 2]


def _hist(n, H, W, L):
    v = torch.randint(0, L, (n, H, W), device="cuda").to(torch.int16)
    b, out = api.Batch.slices(v), torch.empty((n, L, L), dtype=torch.int32, device="cuda")
    return lambda: api.histogram2d(b, H, W, api.binning(0, L - 1, L), out=out)


# as many pixels in images that fill the lanes; twice their time at most
@pytest.mark.parametrize("narrow,wide", [((300, 4096, 8), (300, 128, 256)), ((20, 65536, 1), (20, 256, 256)),
                                         ((300, 1, 4096), (300, 64, 64))])
def test_time_of_narrow_and_flat(narrow, wide):
    assert _us(_hist(*narrow, 64)) <= 2 * _us(_hist(*wide, 64))


def test_time_of_many_small():
    # each of the 5000 histograms has to be written: three times as long at most
    out = torch.empty((5000, 64, 64), dtype=torch.int32, device="cuda")
    assert _us(_hist(5000, 8, 8, 64)) <= 3 * _us(lambda: out.zero_())
