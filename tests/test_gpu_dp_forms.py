"""The forms of the dynamic-programming search agree bit for bit at the edges of
their ranges (one workgroup per problem with eight and with four wavefronts, a
launch per level with one and with four rows per workgroup), agree with the
exhaustive FP64 search for up to three thresholds, and the form chosen by the
sizes is not much slower than the others where they differ most: histograms
with counts in every bin, few thresholds."""
import numpy as np
import pytest

from gpu_util import to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2012_10684_amd import api  # noqa: E402


def _hists(rng, L, n):
    H = rng.integers(1, 4000, (n, L))
    for i in range(n):  # from every bin down to none
        H[i, rng.permutation(L)[:L * (i % 8) // 7]] = 0
    H[::9, 1::3] = 7  # equal counts: exact ties
    return H.astype(np.uint32)


def _padded(X, n, width):
    """The first n rows with bins without counts appended: no class sum changes."""
    return torch.cat([X[:n], X[:n, -1:].expand(n, width - X.shape[1])], 1).contiguous()


# 257 levels and more: a launch per level, one row per workgroup below 7168 / (L - 1) problems
@pytest.mark.parametrize("L", [2, 8, 9, 63, 65, 66, 100, 200, 255, 256])
@pytest.mark.parametrize("k", [1, 2, 3, 5, 9])
def test_forms_agree(L, k):
    if L <= k:
        pytest.skip("no tuple")
    n = 300  # more than one problem per CU: four wavefronts, below it eight
    P, Q = api.prefix(to_dev(_hists(np.random.default_rng(L * k), L, n).view(np.int32)), 0.7)
    want = [x.cpu().numpy() for x in api.threshold_search_dp(_padded(P, 20, 270), _padded(Q, 20, 270), k, 0.7)]
    for m, width in ((n, L), (200, L), (9, L), (n, 270)):
        p, q = (_padded(X, m, width) if width > L else X[:m].contiguous() for X in (P, Q))
        got = [x.cpu().numpy() for x in api.threshold_search_dp(p, q, k, 0.7)]
        c = min(m, 20)
        for a, b in zip(got, want):
            assert a[:c].tobytes() == b[:c].tobytes(), (m, width)


@pytest.mark.parametrize("L,n", [(40, 1), (66, 5), (100, 300), (300, 2), (300, 40)])
@pytest.mark.parametrize("k", [1, 2, 3])
def test_against_the_exhaustive_search(L, n, k):
    rng = np.random.default_rng(L + k)
    h = rng.integers(1, 4000, (n, L))
    h[:, rng.permutation(L)[:L // 4]] = 0
    P, Q = api.prefix(to_dev(h.astype(np.uint32).view(np.int32)), 0.7)
    thr, obj, st = api.threshold_search_dp(P, Q, k, 0.7)
    t2, o2, s2 = api.threshold_search(P, Q, k, 0.7, api.SEARCH_FP64)
    assert torch.equal(thr, t2) and torch.equal(st, s2)
    # the class terms are added in another order: k + 1 roundings of terms up to |1-q| ln L
    assert (obj - o2).abs().max().item() <= 8 * (k + 1) * 2.0**-53 * obj.abs().max().item()


# eight wavefronts up to two problems per CU from 128 levels (k <= 4) or 192 (k <= 8)
@pytest.mark.parametrize("L,k", [(127, 2), (128, 2), (128, 5), (191, 8), (192, 8), (256, 4)])
def test_two_problems_per_cu(L, k):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    P, Q = api.prefix(to_dev(_hists(np.random.default_rng(L * k), L, 2 * cus + 1).view(np.int32)), 0.7)
    want = api.threshold_search_dp(P, Q, k, 0.7)
    for n in (cus, cus + 1, 2 * cus):
        for a, b in zip(api.threshold_search_dp(P[:n].contiguous(), Q[:n].contiguous(), k, 0.7), want):
            rows = b.view(2 * cus + 1, -1)[:n]  # as bytes: the objective of an empty problem is NaN
            assert a.cpu().numpy().tobytes() == rows.cpu().numpy().tobytes(), n


def _us(P, Q, k, reps=9, calls=50):
    n, L = P.shape
    ws = torch.empty(api.workspace_dp_bytes(n, L, k), dtype=torch.uint8, device="cuda")
    out = api.threshold_search_dp(P, Q, k, 0.7, ws=ws)
    t = []
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(calls):
            api.threshold_search_dp(P, Q, k, 0.7, ws=ws, out=out)
        b.record()
        b.synchronize()
        t.append(a.elapsed_time(b) * 1e3 / calls)
    return sorted(t)[reps // 2]


def _dense(L, n):
    h = np.random.default_rng(L + n).integers(1000, 9000, (n, L))
    return api.prefix(to_dev(h.astype(np.uint32).view(np.int32)), 0.7)


@pytest.mark.parametrize("L,n,k", [(64, 100, 1), (64, 1, 2), (100, 24, 2), (256, 12, 8), (256, 257, 2)])
def test_choice(L, n, k):
    P, Q = _dense(L, n)
    # the same problems where only the level form runs, which must form the same terms
    assert _us(P, Q, k) <= 1.15 * _us(_padded(P, n, 257), _padded(Q, n, 257), k)


def test_first_level_of_many_problems():
    # V_0 comes with the first level: at most half a level more
    P, Q = _dense(1024, 30)
    t1, t2, t3 = (_us(P, Q, k) for k in (1, 2, 3))
    assert t2 - t1 <= 1.5 * (t3 - t2), (t1, t2, t3)
