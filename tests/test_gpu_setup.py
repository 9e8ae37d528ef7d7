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


@pytest.mark.parametrize("n_rows,n_cols,count", [
    (1, 1, 5000),                         # one key, summed in input order
    (1, 9000, 2048), (1, 9000, 2049),     # small and large sort of one bucket
    (1, 90_000, 8192), (1, 90_000, 8193), # the largest bucket, and one too many
    (5000, 5000, 1024), (5000, 5000, 1025),
    (70_000, 1000, 262_144), (70_000, 1000, 262_145),       # one radix pass, two
    (400, 1 << 30, 30_000),               # 64-bit keys
    (3_000_000, 40, 3000),                # mostly empty rows
    (1_200_000, 3, 600_000)])
@pytest.mark.parametrize("order", ["shuffled", "rows"])
def test_csr_from_coo_buckets(n_rows, n_cols, count, order):
    row, col, val = coo(count + n_rows, n_rows, n_cols, count)
    if order == "rows":
        by = np.argsort(row, kind="stable")
        row, col, val = row[by], col[by], val[by]
    check_csr(gpu_csr(sp, row, col, val, n_rows, n_cols), oracle.csr_from_coo(n_rows, n_cols, row, col, val))


@pytest.mark.parametrize("heavy", [3000, 8192, 20_000])
def test_csr_from_coo_one_heavy_row(heavy):
    row, col, val = coo(heavy, 40_000, 50_000, 300_000)
    row[::300_000 // heavy][:heavy] = 777
    A = gpu_csr(sp, row, col, val, 40_000, 50_000)
    check_csr(A, oracle.csr_from_coo(40_000, 50_000, row, col, val))
    # values in 32 bits: no two of one position, so that nothing is summed
    once = np.unique(row.astype(np.int64) * 50_000 + col, return_index=True)[1]
    row, col, val = row[once], col[once], val[once]
    by = np.random.default_rng(1).permutation(row.size)
    F = gpu_csr(sp, row[by], col[by], val[by], 40_000, 50_000, torch.float32)
    R = oracle.csr_from_coo(40_000, 50_000, row, col, val.astype(np.float32).astype(np.float64))
    check_csr(F, R)


@pytest.mark.parametrize("at", [0, 4999, 299_999])
@pytest.mark.parametrize("bad", [(-1, 0), (40_000, 0), (0, -5), (0, 50_000)])
def test_csr_from_coo_refuses_an_index_out_of_range(at, bad):
    row, col, val = coo(2, 40_000, 50_000, 300_000)
    row[at], col[at] = bad
    with pytest.raises(sp.SpmvError, match="out of range"):
        gpu_csr(sp, row, col, val, 40_000, 50_000)


def host_plan(A, block_nnz):
    """The plan of the host planner (spmv_crs_plan)."""
    import ctypes as C
    from paper_0910_4836_amd import _lib
    nb = C.c_int32(0)
    plan = torch.empty(2 * A.n_rows + 2, dtype=torch.int32, device="cuda")
    _lib.call("spmv_crs_plan", A.n_rows, C.c_void_p(A.row_ptr.data_ptr()), block_nnz, C.c_void_p(plan.data_ptr()),
              plan.numel(), C.byref(nb), None)
    return to_np(plan)[:nb.value + 1]


def csr_of_lengths(lengths):
    rp = torch.from_numpy(np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)).cuda()
    nnz = int(rp[-1])
    return sp.CSR(len(lengths), 8, rp, torch.zeros(nnz, dtype=torch.int32, device="cuda"),
                  torch.zeros(nnz, dtype=torch.float64, device="cuda"))


@pytest.mark.parametrize("n", [1, 255, 257, 2047, 2049, 4095, 4096, 4097, 6144, 8193, 4096 * 33 + 17])
@pytest.mark.parametrize("kind", ["empty", "short", "edge", "long", "mixed", "sparse"])
def test_plan_on_the_gpu_is_the_host_plan(n, kind):
    rng = np.random.default_rng(n)
    lengths = {"empty": lambda: np.zeros(n, int), "short": lambda: rng.integers(0, 2, n),
               "edge": lambda: rng.integers(14, 19, n), "long": lambda: rng.integers(200, 1200, n),
               "mixed": lambda: np.where(rng.random(n) < 0.002, 5000, rng.integers(0, 40, n)),
               "sparse": lambda: np.where(rng.random(n) < 0.0007, 17, 0)}[kind]()
    A = csr_of_lengths(lengths)
    for block_nnz in (0, 256, 1000, 4096):
        sp.spmv_crs_plan(A, block_nnz)
        assert np.array_equal(to_np(A.plan), host_plan(A, block_nnz)), block_nnz


def test_plan_refuses_a_decreasing_row_ptr():
    A = csr_of_lengths(np.full(9000, 3))
    A.row_ptr[8000] += 4
    with pytest.raises(sp.SpmvError, match="decreases"):
        sp.spmv_crs_plan(A)
    with pytest.raises(sp.SpmvError, match="block_nnz"):
        sp.spmv_crs_plan(csr_of_lengths(np.full(10, 3)), 100)


def csr_of_rows(lengths, n_cols, seed):
    """CRS whose row i has lengths[i] entries in distinct ascending columns (an arithmetic run of them)."""
    rng = np.random.default_rng(seed)
    rp = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    at = np.arange(rp[-1]) - np.repeat(rp[:-1], lengths)
    step = np.repeat(np.maximum(n_cols // np.maximum(lengths, 1), 1), lengths)
    col = (at * step + np.repeat(rng.integers(0, 2, len(lengths)), lengths) * (step > 1)).astype(np.int32)
    return rp, col, rng.standard_normal(rp[-1])


SHAPES = {
    "one row": lambda rng: np.array([7]),
    "short": lambda rng: rng.integers(0, 9, 3000),
    "edge of short": lambda rng: rng.integers(7, 11, 1000),
    "tile edges": lambda rng: np.repeat([31, 32, 33, 63, 64, 65], [65, 64, 63, 1, 2, 129]),
    "long": lambda rng: np.concatenate([[5000, 4097, 300], rng.integers(0, 50, 700)]),
    "empty rows": lambda rng: np.where(rng.random(2000) < 0.7, 0, rng.integers(0, 20, 2000)),
    "more than 65504 diagonals": lambda rng: np.concatenate([[70_000], rng.integers(0, 12, 300)]),
}


@pytest.mark.parametrize("shape", list(SHAPES))
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32, torch.bfloat16, torch.int32])
def test_jds_and_blocked_at_tile_edges(shape, dtype):
    lengths = SHAPES[shape](np.random.default_rng(11))
    n_cols = max(int(lengths.max()), len(lengths))
    rp, col, val = csr_of_rows(lengths, n_cols, 3)
    val = torch.from_numpy(val * 100).to(dtype)
    R = oracle.CSR(len(lengths), n_cols, rp, col, val.double().numpy())
    A = sp.CSR(len(lengths), n_cols, torch.from_numpy(rp).cuda(), torch.from_numpy(col).cuda(), val.cuda())
    J, RJ = sp.jds_from_csr(A), oracle.jds_from_csr(R)
    for got, want in ((J.perm, RJ.perm), (J.iperm, RJ.iperm), (J.jd_ptr, RJ.jd_ptr), (J.jd_col, RJ.jd_col),
                      (J.jd_val.double(), RJ.jd_val)):
        assert np.array_equal(to_np(got), want)
    assert np.array_equal(J.h_jd_ptr, RJ.jd_ptr)
    B = sp.jds_to_csr(J)
    for got, want in ((B.row_ptr, rp), (B.col_idx, col), (B.val.double(), R.val)):
        assert np.array_equal(to_np(got), want)
    for C_ in (64, 192):
        K, RK = sp.jds_blocked_from_jds(J, C_), oracle.blocked_from_jds(RJ, C_)
        assert np.array_equal(to_np(K.slice_ptr), RK.slice_ptr)
        assert np.array_equal(to_np(K.bl_col), RK.bl_col)
        assert np.array_equal(to_np(K.bl_val.double()), RK.bl_val)


@pytest.mark.parametrize("n", [1, 4096, 4097, 20_000])
def test_plan_reports_the_longest_row(n):
    lengths = np.random.default_rng(n).integers(0, 30, n)
    lengths[n // 2] = 77
    assert sp.spmv_crs_plan(csr_of_lengths(lengths)).longest == 77
