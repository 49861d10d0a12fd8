"""Labels of problems at any alignment: tiles over one, a few and many
problems, every cut-count instance, outputs packed back to back between guard
bytes.  Labels are whole numbers: equal to the oracle's, nothing else written."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, to_dev
from paper_2012_10684_amd import api

pytestmark = pytest.mark.gpu

WIN = (-1024, -200, 100)
# problem sizes around the default tile of 4096 voxels: a tile in one problem, over two to five problems (empty ones
# among them), and over many
SIZES = {
    "one": [4096, 1, 4095, 8193],
    "few": [4097, 1365, 0, 1366, 1364, 3, 4090, 1023, 1025, 0, 0, 2047],
    "many": [700] * 3 + [5, 0, 17, 1, 1, 2, 3] * 40 + [9000],
}


def _packed(sizes, seed, shift):
    rng = np.random.default_rng(seed)
    host = rng.integers(-1100, -100, sum(sizes) + shift).astype(np.int16)
    d = to_dev(host)
    at = np.concatenate([[0], np.cumsum(sizes)]) + shift
    return host, [d[at[i]:at[i + 1]] for i in range(len(sizes))], at


def _outs(sizes, nsets, shift):
    """One buffer per set with the problems' labels back to back from byte
    `shift`, filled with 0xEE."""
    bufs = [torch.full((sum(sizes) + shift + 16,), 0xEE, dtype=torch.uint8, device=dev()) for _ in range(nsets)]
    at = np.concatenate([[0], np.cumsum(sizes)]) + shift
    return bufs, [[b[at[i]:at[i + 1]] for i in range(len(sizes))] for b in bufs]


def _check(buf, host, sizes, at, shift, thr):
    want = np.full(buf.numel(), 0xEE, np.uint8)
    o = shift
    for i, n in enumerate(sizes):
        if n:
            want[o:o + n] = oracle.label(host[at[i]:at[i + 1]], *WIN, thr[i])
        o += n
    assert np.array_equal(buf.cpu().numpy(), want)


@pytest.mark.parametrize("k", [1, 2, 4, 5, 8, 9])
@pytest.mark.parametrize("sizes", SIZES, ids=str)
def test_label_pieces(sizes, k):
    sizes = SIZES[sizes]
    for shift, oshift, nsets in ((0, 0, 1), (1, 0, 2), (3, 5, 3)):
        host, segs, at = _packed(sizes, 7 * k + shift, shift)
        bufs, outs = _outs(sizes, nsets, oshift)
        rng = np.random.default_rng(k)
        thrs = [np.stack([np.sort(rng.choice(99, k, replace=False)) for _ in sizes]).astype(np.int32) for _ in range(nsets)]
        api.label_sets(api.Batch(segs), api.binning(*WIN), [to_dev(t) for t in thrs], k, outs=outs)
        torch.cuda.synchronize()
        for u in range(nsets):
            _check(bufs[u], host, sizes, at, oshift, thrs[u])


@pytest.mark.parametrize("sizes,k", [([7001], 1), ([7001, 0, 5, 4999, 8192], 1), ([7001, 0, 5, 4999, 8192], 2)])
@pytest.mark.parametrize("shift", [0, 1, 3])
def test_segment_labels_any_alignment(sizes, k, shift):
    """The one-problem launch and the one-workgroup-per-problem launch."""
    host, segs, at = _packed(sizes, 11 + shift, shift)
    nq = 1 if len(sizes) == 1 else 2
    bufs, outs = _outs(sizes, nq, shift)
    tune = None if len(sizes) == 1 else {"segment_parts": 1}
    ptrs = [api.device_table([o.data_ptr() for o in oj], dev()) for oj in outs]
    _, (thr, _, _), _ = api.segment(api.Batch(segs), api.binning(*WIN), k, [0.8, 1.5][:nq], out_ptrs=ptrs, tune=tune)
    torch.cuda.synchronize()
    t = thr.cpu().numpy()
    for u in range(nq):
        _check(bufs[u], host, sizes, at, shift, t[u])
