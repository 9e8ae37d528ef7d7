"""COO -> CRS where one row holds more entries than a bucket may: every way of
seeing that before and after the passes (too many entries for all buckets, one
pass, counted buckets, after the passes), entries shuffled, by columns and by
rows, and just as many entries as still fit.  Bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import to_dev, to_np

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_0910_4836_amd")


@pytest.mark.parametrize("order", ["shuffled", "columns", "rows"])
@pytest.mark.parametrize("n_rows,per_row,extra", [
    (1, 0, 8192), (1, 0, 8193), (3, 0, 30_000),                     # one bucket, and more than all hold
    (2000, 15, 8300), (2000, 15, 7000), (20_000, 15, 60_000),       # one pass
    (40_000, 15, 9000), (40_000, 15, 7000), (300, 2500, 0), (300, 2500, 9000),      # counted
    (140_000, 15, 9000)])                                           # two passes, not counted
def test_row_of_many_entries(n_rows, per_row, extra, order):
    rng = np.random.default_rng(n_rows + extra)
    n_cols = 70_000
    r = np.concatenate([np.repeat(np.arange(n_rows), per_row), np.full(extra, n_rows // 3)]).astype(np.int32)
    c = rng.integers(0, n_cols, r.size).astype(np.int32)
    at = {"shuffled": rng.permutation(r.size), "columns": np.argsort(c, kind="stable"), "rows": np.arange(r.size)}[order]
    r, c = r[at], c[at]
    for dtype in (np.float64, np.float32):
        v = rng.standard_normal(r.size).astype(dtype)
        A = sp.csr_from_coo(n_rows, n_cols, to_dev(r), to_dev(c), to_dev(v))
        # duplicates summed in input order, in the values' type
        key = np.argsort(r.astype(np.int64) * n_cols + c, kind="stable")
        rs, cs, vs = r[key], c[key], v[key]
        head = np.concatenate([[True], (np.diff(rs) != 0) | (np.diff(cs) != 0)])
        first = np.flatnonzero(head)
        want = vs[first].copy()
        length = np.diff(np.concatenate([first, [r.size]]))
        for d in range(1, length.max()):
            more = length > d
            want[more] += vs[first[more] + d]
        assert np.array_equal(to_np(A.row_ptr), np.searchsorted(rs[first], np.arange(n_rows + 1)))
        assert np.array_equal(to_np(A.col_idx), cs[first]) and np.array_equal(to_np(A.val), want)
    R = oracle.csr_from_coo(n_rows, n_cols, r, c, v.astype(np.float64))
    assert np.array_equal(R.row_ptr, to_np(A.row_ptr)) and np.array_equal(R.col, to_np(A.col_idx))
