"""ts_segment's prefix sums inside the search's launches, and the re-check split
over workgroups: bit for bit what the prefix pass and the search give as
separate calls on both search paths, over numbers of levels at the edges of
the scan's and the tiles' layout, for few and many problems, on histograms
with one, several and very many tuples near the best."""
import numpy as np
import pytest

from gpu_util import to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2012_10684_amd import api  # noqa: E402


def _voxels(rng, L):
    """Voxel lists whose levels under the identity binning have chosen counts."""
    flat = np.full(L, 6)                                  # near-ties everywhere
    rand = rng.integers(0, 40, L)
    rand[rng.random(L) < 0.4] = 0
    rand[[0, L // 2, L - 1]] = 9
    few = np.zeros(L, int)
    few[rng.permutation(L)[:3]] = 50                      # fewer classes than k = 3 needs
    sym = np.minimum(np.arange(L), np.arange(L)[::-1]) + 1  # mirror tuples tie
    return [rng.permutation(np.repeat(np.arange(L), c)).astype(np.int16) for c in (flat, rand, few, sym)]


@pytest.mark.parametrize("k,L", [(1, 2), (1, 3), (1, 255), (1, 1025), (1, 4096), (2, 3), (2, 4), (2, 65), (2, 256),
                                 (2, 257), (2, 384), (2, 385), (2, 1000), (2, 1024), (2, 1100), (3, 4), (3, 5), (3, 9),
                                 (3, 40), (3, 256), (3, 300), (3, 1030)])
def test_segment_equals_separate_calls(k, L):
    rng = np.random.default_rng(7 * L + k)
    vox = [to_dev(v) for v in _voxels(rng, L)]
    qs = (0.8, 1.0, 2.0)
    for copies in ((1,) if L > 300 else (1, 9)):  # few problems, and enough for the other path
        batch = api.Batch(vox * copies)
        binn = api.binning(0, L - 1, L)
        h, (thr, obj, st), labels = api.segment(batch, binn, k, qs)
        assert torch.equal(h, api.histogram(batch, binn))
        P, Q = api.prefix(h, qs)
        for path in (0, 2) if k == 3 else (0, 1, 2):
            if path == 1 and k == 2 and L > 1024:
                continue
            t2, o2, s2 = api.threshold_search(P, Q, k, qs, tune={"search_path": path} if path else None)
            assert torch.equal(st, s2), path
            assert torch.equal(thr, t2), path
            assert torch.equal(obj.view(torch.int64), o2.view(torch.int64)), path
        for j in range(len(qs)):
            want = torch.cat(api.label(batch, binn, thr[j], k))
            assert torch.equal(torch.cat(labels[j]), want), j


@pytest.mark.parametrize("k,L", [(2, 600), (3, 60)])
def test_every_tuple_rechecked(k, L):
    """An index so large that class sums leave the FP32 range: the error bound
    is infinite and every tuple is evaluated in FP64."""
    rng = np.random.default_rng(L)
    batch = api.Batch([to_dev(v) for v in _voxels(rng, L)[:2]])
    binn = api.binning(0, L - 1, L)
    h, (thr, obj, st), _ = api.segment(batch, binn, k, (12.0,))
    P, Q = api.prefix(h, (12.0,))
    t2, o2, s2 = api.threshold_search(P, Q, k, (12.0,), mode=api.SEARCH_FP64)
    assert torch.equal(st, s2)
    assert torch.allclose(obj, o2, rtol=1e-12, atol=0.0)


@pytest.mark.parametrize("L", [4, 5, 33, 257, 700])
def test_k3_on_few_occupied_bins(L):
    """k = 3 walks only the bins that can be thresholds: the same thresholds
    as the FP64 search over all bins, from no occupied bin at the ends to one
    bin in twenty."""
    rng = np.random.default_rng(L)
    rows = []
    for keep in (1.0, 0.5, 0.05):
        c = rng.integers(1, 1000, L)
        c[rng.random(L) >= keep] = 0
        rows.append(c)
    rows.append(np.where(np.arange(L) < L // 2, 0, rows[0]))
    rows.append(np.where(np.arange(L) < (L + 1) // 2, rows[0], 0))
    h = to_dev(np.array(rows).astype(np.int32))
    P, Q = api.prefix(h, (0.8, 1.0, 2.0))
    thr, obj, st = api.threshold_search(P, Q, 3, (0.8, 1.0, 2.0))
    t2, o2, s2 = api.threshold_search(P, Q, 3, (0.8, 1.0, 2.0), mode=api.SEARCH_FP64)
    assert torch.equal(st, s2)
    ok = st == 0
    assert torch.equal(thr[ok], t2[ok])
    assert torch.allclose(obj[ok], o2[ok], rtol=1e-12, atol=0.0)
