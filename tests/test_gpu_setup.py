"""Matrix construction at the sizes where its kernels can go wrong: tile edges
of the radix passes, row and column counts that change the number of passes.
Integer and index work, and values that are only moved: bit-exact."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import gpu_csr, to_np

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_0910_4836_amd")


def coo(seed, n_rows, n_cols, count):
    """`count` unordered triplets, some positions given more than once."""
    rng = np.random.default_rng(seed)
    row = rng.integers(0, n_rows, count).astype(np.int32)
    col = rng.integers(0, n_cols, count).astype(np.int32)
    dup = rng.integers(0, count, count // 8)
    row[:dup.size], col[:dup.size] = row[dup], col[dup]
    return row, col, rng.standard_normal(count)


def check_csr(A, R):
    assert np.array_equal(to_np(A.row_ptr), R.row_ptr)
    assert np.array_equal(to_np(A.col_idx), R.col)
    assert np.array_equal(to_np(A.val), R.val)


@pytest.mark.parametrize("count", [1, 2, 8191, 8192, 8193, 17 * 8192 + 5])
@pytest.mark.parametrize("n_rows,n_cols", [(3, 200), (300, 70_000), (70_000, 300)])
def test_csr_from_coo_and_transpose_at_tile_edges(count, n_rows, n_cols):
    row, col, val = coo(count, n_rows, n_cols, count)
    A = gpu_csr(sp, row, col, val, n_rows, n_cols)
    R = oracle.csr_from_coo(n_rows, n_cols, row, col, val)
    check_csr(A, R)
    rowT, colT, tmap = sp.spmv_transpose_csr(A)
    order = np.argsort(R.col, kind="stable")
    assert np.array_equal(to_np(tmap), order)
    assert np.array_equal(to_np(colT), np.repeat(np.arange(n_rows), np.diff(R.row_ptr))[order])
    assert np.array_equal(to_np(rowT), np.searchsorted(R.col[order], np.arange(n_cols + 1)))
