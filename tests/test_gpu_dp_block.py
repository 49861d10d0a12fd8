"""The dynamic-programming search's two forms agree bit for bit: problems of
up to 256 levels (a workgroup each when there are enough of them) against the
same prefix sums with repeating bins appended past 256 levels (one launch per
level), over candidate counts around the 64-candidate wavefronts and every
number of thresholds' kernel instance."""
import numpy as np
import pytest

from gpu_util import to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2012_10684_amd import api  # noqa: E402


def _hists(rng, L):
    H = []
    for occ in (0, 1, 2, 5, 63, 64, 65, 66, 127, 129, 193, L - 1, L):
        h = np.zeros(L, np.uint32)
        occ = min(occ, L)
        h[np.sort(rng.permutation(L)[:occ])] = rng.integers(1, 4000, occ)
        H.append(h)
    h = np.zeros(L, np.uint32)
    h[1::3] = 7  # equal counts: exact ties
    H.append(h)
    return np.stack(H)


@pytest.mark.parametrize("L", [17, 64, 66, 100, 256])
@pytest.mark.parametrize("k", [1, 4, 5, 8, 9, 16])
def test_block_form_equals_level_form(L, k):
    H = _hists(np.random.default_rng(31 * L + k), L)
    n = len(H)
    rep = -(-256 // n)  # enough problems for a workgroup each, at every k
    for q in (0.5, 1.0, 1.7):
        P, Q = api.prefix(to_dev(np.tile(H, (rep, 1)).view(np.int32)), q)
        thr, obj, st = (x.cpu().numpy() for x in api.threshold_search_dp(P, Q, k, q))
        # bins without counts after the last: no tuple and no class sum changes
        P2, Q2 = (torch.cat([x[:n], x[:n, -1:].expand(n, 300 - L)], 1).contiguous() for x in (P, Q))
        t2, o2, s2 = (x.cpu().numpy() for x in api.threshold_search_dp(P2, Q2, k, q))
        assert st[:n].tolist() == s2.tolist(), q
        assert thr[:n].tolist() == t2.tolist(), q
        assert np.array_equal(obj[:n].view(np.int64), o2.view(np.int64)), q
        for r in range(1, rep):  # every copy of a problem agrees
            assert np.array_equal(thr[r * n:(r + 1) * n], thr[:n]) and np.array_equal(st[r * n:(r + 1) * n], st[:n])
