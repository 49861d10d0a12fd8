"""Labels of 9 to 16 thresholds in up to four sets: whole tiles, pieces and
problems labelled voxel by voxel, aligned and not, against the oracle's rule;
and three sets take no longer than three passes over one."""
import numpy as np
import pytest

import oracle
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2012_10684_amd import api  # noqa: E402

L = 200


def _thresholds(rng, n, k):
    t = np.sort(np.stack([rng.permutation(L - 1)[:k] for _ in range(n)]), 1).astype(np.int32)
    t[n // 2] = -1  # a problem without thresholds
    return t


@pytest.mark.parametrize("k", [9, 12, 16])
@pytest.mark.parametrize("nsets", [1, 2, 3, 4])
def test_labels(k, nsets):
    rng = np.random.default_rng(16 * k + nsets)
    sizes = [20000, 8, 4097, 1, 0, 4096, 333, 12288, 7] + [5] * 900 + [1500, 1501, 2]
    flat = rng.integers(-1100, 300, sum(sizes) + 1).astype(np.int16)
    d = to_dev(flat)
    for shift in (0, 1):
        at = np.concatenate([[0], np.cumsum(sizes)]) + shift
        batch = api.Batch([d[a:b] for a, b in zip(at, at[1:])])
        thr = [_thresholds(rng, len(sizes), k) for _ in range(nsets)]
        out = api.label_sets(batch, api.binning(-1024, -200, L), [to_dev(t) for t in thr], k)
        for u in range(nsets):
            got = torch.cat(out[u]).cpu().numpy()
            for i in [0, 1, 2, 3, 5, 6, 7, 8, 9, len(sizes) // 2, len(sizes) - 3, len(sizes) - 2, len(sizes) - 1]:
                a, b = at[i] - shift, at[i + 1] - shift
                want = oracle.label(flat[at[i]:at[i + 1]], -1024, -200, L, thr[u][i])
                assert np.array_equal(got[a:b], want), (u, i, shift)


def _us(f, reps=7, calls=5):
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


def test_time_of_three_sets():
    n, size, k = 20000, 1000, 16
    v = torch.randint(-1100, 300, (n * size,), device="cuda").to(torch.int16)
    at = torch.arange(n, device="cuda") * size
    batch = api.Batch(list(v.split(size)))
    thr = torch.arange(10, 10 + 10 * k, 10, dtype=torch.int32, device="cuda").repeat(n, 1)
    out = torch.empty((3, n * size), dtype=torch.uint8, device="cuda")
    ptrs = [o.data_ptr() + at for o in out]
    binn = api.binning(-1024, -200, L)
    t1, t3 = (_us(lambda: api.label_sets(batch, binn, [thr] * m, k, outs=[], out_ptrs=ptrs[:m])) for m in (1, 3))
    assert t3 <= 3 * t1, (t1, t3)
