"""batch_segment's problem tables against one slice view after the other, and
their time for many small volumes, which a call needs about four times."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2012_10684_amd import api  # noqa: E402

SHAPES = {
    "one": [(3, 5, 7)],
    "none": [],
    "empty": [(0, 4, 4)],
    "three": [(2, 5, 7), (0, 5, 7), (4, 2, 3)],
    "mixed": [(2, 5, 7), (0, 5, 7), (1, 1, 1), (4, 2, 0), (3,), (2, 3, 4, 5)],
    "many": [(1 + i % 3, 4, 4 + i % 5) for i in range(50)],
}


@pytest.mark.parametrize("shapes", SHAPES, ids=str)
@pytest.mark.parametrize("dtype", [torch.int16, torch.uint8])
@pytest.mark.parametrize("per", ["slice", "volume"])
def test_tables(shapes, dtype, per):
    vols = [torch.zeros(s, dtype=dtype) for s in SHAPES[shapes]]
    ptrs, sizes = api._problems(vols, per)
    segs = [v[z].reshape(-1) for v in vols for z in range(v.shape[0])] if per == "slice" else [v.reshape(-1) for v in vols]
    assert ptrs.dtype == sizes.dtype == np.int64
    assert sizes.tolist() == [s.numel() for s in segs]
    assert [p for p, n in zip(ptrs.tolist(), sizes.tolist()) if n] == [s.data_ptr() for s in segs if s.numel()]


def test_time_of_many_volumes():
    vols = [torch.zeros((1, 4, 4), dtype=torch.int16) for _ in range(500)]

    def best(f):
        t = []
        for _ in range(9):
            t0 = time.perf_counter()
            f()
            t.append(time.perf_counter() - t0)
        return min(t)

    views = best(lambda: [v[z].reshape(-1).data_ptr() for v in vols for z in range(v.shape[0])])
    assert best(lambda: api._problems(vols, "slice")) <= views  # the views they replace
