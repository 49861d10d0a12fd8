"""The 2D search where its block layout can go wrong, against the oracle:
fewer rows with counts than wavefronts, levels that are no multiple of the
lane's columns, counts past the table of terms (with candidates in neighbouring
rows), and problems enough for the smaller workgroups."""
import numpy as np
import pytest

import oracle
from gpu_util import to_dev
from test_gpu_2d import check_pair

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2012_10684_amd import api  # noqa: E402


def _hists(rng, L):
    out = []
    for rows in (1, 2, 3, min(9, L), min(17, L), L):
        h = np.zeros((L, L), np.uint32)
        r = np.sort(rng.permutation(L)[:rows])
        h[r] = rng.integers(0, 40, (len(r), L))
        h[:, rng.random(L) < 0.3] = 0  # whole empty columns
        out.append(h)
    h = rng.integers(0, 6, (L, L)).astype(np.uint32)
    h[rng.random((L, L)) < 0.02] = 1 << 13  # past the table, in many rows
    out.append(h)
    out.append(np.full((L, L), 5000, np.uint32))  # every pair near the best: many candidate rows
    return np.stack(out)


@pytest.mark.parametrize("L", [2, 3, 15, 30, 61, 64])
@pytest.mark.parametrize("q", [0.8, 1.0, 2.5])
def test_layout_edges(L, q):
    H = _hists(np.random.default_rng(L), L)
    n = len(H)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    few = [x.cpu().numpy() for x in api.threshold_search2d(to_dev(H.view(np.int32)), q)]
    for i in range(n):
        check_pair(H[i], q, few[0][:, i], few[1][i], few[2][i])
    rep = cus // n + 1
    many = [x.cpu().numpy() for x in api.threshold_search2d(to_dev(np.tile(H, (rep, 1, 1)).view(np.int32)), q)]
    for r in range(rep):
        s = slice(r * n, (r + 1) * n)
        assert np.array_equal(many[2][s], few[2])
        ok = few[2] == 0
        # the blocks differ, so the sums' order does: the pair by its objective
        assert np.allclose(many[1][s][ok], few[1][ok], rtol=1e-12, atol=1e-12)
        if r == 0:
            for i in range(n):
                check_pair(H[i], q, many[0][:, i], many[1][i], many[2][i])
