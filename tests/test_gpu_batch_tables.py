"""batch_segment's problem tables: volumes without slices between others,
non-contiguous volumes and no volumes at all give what one Batch per problem
list gives, per slice and per volume, with and without the opening."""
import numpy as np
import pytest

from gpu_util import to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2012_10684_amd import api  # noqa: E402


@pytest.mark.parametrize("radius", [None, 3])
@pytest.mark.parametrize("per", ["slice", "volume"])
def test_tables(per, radius):
    if per == "volume" and radius is not None:
        pytest.skip("the opening works per slice")
    rng = np.random.default_rng(4)
    shapes = [(3, 21, 17), (0, 21, 17), (2, 30, 8), (1, 5, 5)]
    vols = [to_dev(rng.integers(-1100, 300, s).astype(np.int16)) for s in shapes]
    vols[2] = to_dev(rng.integers(-1100, 300, (2, 8, 30)).astype(np.int16)).transpose(1, 2)
    binn = api.binning(-1024, -200, 64)
    r = api.batch_segment(vols, binn, 2, (0.8, 1.5), per=per, open_radius=radius)
    src = [v.contiguous() for v in vols]
    if radius is not None:
        src = [api.open2d(api.Batch.slices(v), v.shape[1], v.shape[2], binn, radius, want=("residue16",))[2] for v in src]
        assert all(torch.equal(a, b) for a, b in zip(r.residues, src))
        binn = api.binning(0, 63, 64)
    segs = [x.reshape(-1) for v in src for x in (v if per == "slice" else [v])]
    batch = api.Batch(segs)
    h = api.histogram(batch, binn)
    P, Q = api.prefix(h, (0.8, 1.5))
    thr, obj, st = api.threshold_search(P, Q, 2, (0.8, 1.5))
    assert torch.equal(r.hist, h) and torch.equal(r.thr, thr) and torch.equal(r.status, st)
    for j in range(2):
        want = torch.cat(api.label(batch, binn, thr[j], 2))
        assert [tuple(x.shape) for x in r.labels[j]] == [tuple(v.shape) for v in vols]
        assert torch.equal(torch.cat([x.reshape(-1) for x in r.labels[j]]), want)


def test_no_volumes():
    r = api.batch_segment([], api.binning(0, 63, 64), 2, 0.8)
    assert r.hist.shape == (0, 64) and r.thr.shape == (1, 0, 2) and r.labels == [[]]
