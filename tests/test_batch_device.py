"""batch_segment works on the device of its first problem: a volume without
slices holds none, and its device decides nothing, wherever it stands."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2012_10684_amd import api  # noqa: E402


class _OnGpu:
    """A (2, 4, 4) volume that says it is a contiguous CUDA tensor; its device
    is one that torch can make tensors on without a GPU."""

    shape, dtype, is_cuda, device = torch.Size((2, 4, 4)), torch.int16, True, torch.device("meta")

    def contiguous(self):
        return self

    def numel(self):
        return 32

    def element_size(self):
        return 2

    def data_ptr(self):
        return 4096


class _Chosen(Exception):
    pass


@pytest.mark.parametrize("order", ["first", "between", "last"])
def test_device_of_the_first_problem(order, monkeypatch):
    empty, vol = torch.empty((0, 4, 4), dtype=torch.int16), _OnGpu()
    vols = {"first": [empty, vol], "between": [vol, empty, vol], "last": [vol, empty]}[order]

    def tables(_tables, device):
        raise _Chosen(device)

    monkeypatch.setattr(api, "_device_tables", tables)
    with pytest.raises(_Chosen) as e:
        api.batch_segment(vols, api.binning(0, 63, 64), 2, 0.8)
    assert e.value.args[0] == vol.device


def test_no_problem_is_the_gpu(monkeypatch):
    def tables(_tables, device):
        raise _Chosen(device)

    monkeypatch.setattr(api, "_device_tables", tables)
    with pytest.raises(_Chosen) as e:
        api.batch_segment([torch.empty((0, 4, 4), dtype=torch.int16)], api.binning(0, 63, 64), 2, 0.8)
    assert e.value.args[0] == torch.device("cuda")


@pytest.mark.gpu
def test_empty_host_volume_first():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    v = torch.from_numpy(np.random.default_rng(2).integers(-1100, 300, (3, 9, 14)).astype(np.int16)).cuda()
    binn = api.binning(-1024, -200, 32)
    want = api.batch_segment([v], binn, 2, 0.8)
    r = api.batch_segment([torch.empty((0, 5, 5), dtype=torch.int16), v], binn, 2, 0.8)
    assert r.hist.is_cuda and torch.equal(r.hist, want.hist) and torch.equal(r.thr, want.thr)
    assert [tuple(x.shape) for x in r.labels[0]] == [(0, 5, 5), (3, 9, 14)]
    assert torch.equal(r.labels[0][1], want.labels[0][0])
