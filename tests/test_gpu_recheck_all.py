"""The search where no FP32 error bound is finite (a bin of a few voxels
among 5e8, q = 2), so that every tuple is re-checked in FP64: the same thresholds,
objectives (bit for bit) and statuses as the plain form, which evaluates every
tuple the same way one thread at a time, and in no more time than it."""
import numpy as np
import pytest

from gpu_util import to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2012_10684_amd import api  # noqa: E402

Q = 2.0


def _hists(L, n, sparse, seed):
    """n histograms of about 5e8 voxels with a bin of 20; sparse: gaps
    of bins without counts, the first and the last among them in some."""
    rng = np.random.default_rng(seed)
    h = rng.integers(10**8 // L, 10**9 // L, (n, L))
    if sparse:
        h[rng.random((n, L)) < 0.4] = 0
    if L > 8:
        h[0, :2] = h[-1, -1] = 5000
    h[np.arange(n), rng.integers(0, L, n)] = 20
    return h.astype(np.uint32)


def _prefix(h):
    P, Qs = api.prefix(to_dev(h.view(np.int32)), Q)
    # the relative error of a class sum's difference of split prefixes, whose
    # bound must be below 1e-3 for a finite bound of the keys
    step = np.abs(np.diff(Qs.cpu().numpy(), axis=1, prepend=0.0))
    step[step == 0] = np.inf
    assert (4 * 2.0**-48 * Qs.cpu().numpy()[:, -1] / step.min(1) > 1e-3).all()
    return P, Qs


@pytest.mark.parametrize("sparse", [False, True])
@pytest.mark.parametrize("k,L", [(2, 3), (2, 66), (2, 130), (2, 257), (2, 700), (3, 4), (3, 5), (3, 66), (3, 130), (3, 300)])
def test_every_tuple(k, L, sparse):
    P, Qs = _prefix(_hists(L, 3, sparse and L > 8, L))
    want = api.threshold_search(P, Qs, k, Q, api.SEARCH_PLAIN)
    got = api.threshold_search(P, Qs, k, Q, tune={"search_path": 2})
    for a, b in zip(got, want):
        assert torch.equal(a, b)


def test_rows_over_one_chunk():  # k = 3 beyond 1024 columns: two chunks per row
    h = _hists(1100, 1, True, 5)
    h[0, 1028:1090] = 3000000
    P, Qs = _prefix(h)
    want = api.threshold_search(P, Qs, 3, Q, api.SEARCH_PLAIN)
    for a, b in zip(api.threshold_search(P, Qs, 3, Q), want):
        assert torch.equal(a, b)


def _us(f, reps=5):
    f()
    t = []
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        b.synchronize()
        t.append(a.elapsed_time(b) * 1e3)
    return sorted(t)[reps // 2]


def test_no_slower_than_the_plain_form():
    P, Qs = _prefix(_hists(512, 1, False, 9))
    full = _us(lambda: api.threshold_search(P, Qs, 3, Q))
    plain = _us(lambda: api.threshold_search(P, Qs, 3, Q, api.SEARCH_PLAIN))
    assert full <= plain, (full, plain)


@pytest.mark.parametrize("block", [256, 512, 1024])
@pytest.mark.parametrize("L", [3, 5, 66, 130, 257, 400, 1000])
def test_every_tuple_in_one_workgroup(L, block):
    P, Qs = _prefix(_hists(L, 3, L > 8, L + block))
    want = api.threshold_search(P, Qs, 2, Q, api.SEARCH_PLAIN)
    got = api.threshold_search(P, Qs, 2, Q, tune={"search_path": 1, "search_block": block})
    for a, b in zip(got, want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("tune", [{"segment_parts": 1}, {"search_path": 1}, {"search_path": 2}])
def test_every_tuple_in_segment(tune):
    v = torch.randint(0, 200, (1, 8, 512, 512), device="cuda").to(torch.int16)
    v[0, 0, 0, :3] = 230  # three voxels among two million: no finite bound at q = 3
    batch, binn = api.Batch.whole(v), api.binning(0, 255, 256)
    hist, got, _ = api.segment(batch, binn, 2, 3.0, tune=tune)
    P, Qs = api.prefix(hist, 3.0)
    want = api.threshold_search(P, Qs, 2, 3.0, api.SEARCH_PLAIN)
    for a, b in zip(got, want):
        assert torch.equal(a, b)


def test_one_workgroup_time():
    # 32640 tuples in one workgroup: the finite call takes about a tenth of the
    # logarithms; six times its time is twice what the FP64 issue rate asks for
    P, Qs = _prefix(_hists(256, 1, False, 3))
    P1, Q1 = api.prefix(to_dev(_hists(256, 1, False, 3).view(np.int32)), 0.8)
    full = _us(lambda: api.threshold_search(P, Qs, 2, Q, tune={"search_path": 1}), 15)
    finite = _us(lambda: api.threshold_search(P1, Q1, 2, 0.8, tune={"search_path": 1}), 15)
    assert full <= 6 * finite, (full, finite)
