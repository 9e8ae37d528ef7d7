"""Multi-vector products at ragged vector counts: row widths that are padded
and not padded in the staged copy of X, column groups that the last lanes do
not fill, and the row counts at which the JDS launch changes."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import FP64_TOL, gpu_csr, rand_coo, to_np

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_0910_4836_amd")

def block(rng, n, k, dtype):
    return torch.from_numpy(np.ascontiguousarray(rng.uniform(-1, 1, (n, k)).T)).to(dtype).to("cuda").t()


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("k", [1, 2, 3, 5, 7, 9, 13, 16, 17, 24, 25, 31, 33, 41, 49, 63, 64])
def test_ragged_vector_counts(k, dtype):
    r, c, v, nr, nc, rng = rand_coo(500 + k, 2500, 2500, 0.003, empty_rows=0.1, long_rows=5, long_len=1600)
    v = v.astype(np.float32).astype(np.float64)
    R = oracle.csr_from_coo(nr, nc, r, c, v)
    A = gpu_csr(sp, r, c, v, nr, nc, dtype)
    Xd = block(rng, nc, k, dtype)
    X = to_np(Xd).astype(np.float64)
    J = sp.jds_from_csr(A)
    B = sp.jds_blocked_windowed_from_csr(A, 64, 256)
    want = oracle.spmm_crs(R, X)
    D = np.stack([oracle.row_absdot(R, X[:, j]) for j in range(k)], axis=1)
    # FP32: a sum of m products in any order is off by at most m roundings of
    # 2^-24 on the absolute sum, and the result by one more for alpha and beta
    tol = FP64_TOL if dtype == torch.float64 else (np.diff(R.row_ptr)[:, None] + 2) * 2.0 ** -24
    esize = torch.empty(0, dtype=dtype).element_size()
    tight = (nc * k * esize + 255) // 256 * 256 + 256       # rows of k elements, not padded
    for size in (None, tight):
        ws = None if size is None else torch.empty(size, dtype=torch.uint8, device="cuda")
        for name, f, M in (("crs", sp.spmm_crs, A), ("jds", sp.spmm_jds, J), ("windowed", sp.spmm_jds_blocked, B)):
            got = to_np(f(M, Xd, ws=ws)).astype(np.float64)
            assert (oracle.rel_err(got, want, D) <= tol).all(), (name, size)


@pytest.mark.parametrize("k", [3, 13])
@pytest.mark.parametrize("n", [149_999, 150_000, 299_999, 300_000])
def test_jds_launch_changes_with_the_row_count(n, k):
    rng = np.random.default_rng(n + k)
    r = np.concatenate([np.arange(n), np.full(1100, 7), np.full(270, n - 1)]).astype(np.int32)
    c = rng.integers(0, n, r.size).astype(np.int32)
    v = rng.standard_normal(r.size)
    R = oracle.csr_from_coo(n, n, r, c, v)
    J = sp.jds_from_csr(gpu_csr(sp, r, c, v, n, n))
    Xd = block(rng, n, k, torch.float64)
    X = to_np(Xd)
    got, want = to_np(sp.spmm_jds(J, Xd)), oracle.spmm_crs(R, X)
    for j in range(k):
        assert oracle.rel_err(got[:, j], want[:, j], oracle.row_absdot(R, X[:, j])).max() <= FP64_TOL


@pytest.mark.parametrize("k", [4, 5])
@pytest.mark.parametrize("n,longest", [(59_999, 20), (60_000, 20), (60_000, 64), (60_000, 65), (149_999, 20),
                                       (150_000, 20)])
def test_jds_launch_changes_with_the_longest_row_and_vector_count(n, longest, k):
    rng = np.random.default_rng(n + k)
    r = np.concatenate([np.arange(n), np.full(longest - 1, 7)]).astype(np.int32)
    c = rng.integers(0, n, r.size).astype(np.int32)
    c[n:], c[7] = np.arange(1, longest), 0                   # row 7: `longest` distinct columns
    v = rng.standard_normal(r.size)
    R = oracle.csr_from_coo(n, n, r, c, v)
    J = sp.jds_from_csr(gpu_csr(sp, r, c, v, n, n))
    Xd = block(rng, n, k, torch.float64)
    X = to_np(Xd)
    got, want = to_np(sp.spmm_jds(J, Xd)), oracle.spmm_crs(R, X)
    for j in range(k):
        assert oracle.rel_err(got[:, j], want[:, j], oracle.row_absdot(R, X[:, j])).max() <= FP64_TOL


@pytest.mark.parametrize("n", [149_999, 150_000])
def test_windowed_launch_changes_with_the_row_count(n):
    rng = np.random.default_rng(n)
    r = np.concatenate([np.arange(n), np.full(300, 11), np.full(70, n - 2)]).astype(np.int32)
    c = rng.integers(0, n, r.size).astype(np.int32)
    v = rng.standard_normal(r.size)
    R = oracle.csr_from_coo(n, n, r, c, v)
    B = sp.jds_blocked_windowed_from_csr(gpu_csr(sp, r, c, v, n, n), 64, 4096)
    Xd = block(rng, n, 13, torch.float64)
    X = to_np(Xd)
    got, want = to_np(sp.spmm_jds_blocked(B, Xd)), oracle.spmm_crs(R, X)
    for j in range(13):
        assert oracle.rel_err(got[:, j], want[:, j], oracle.row_absdot(R, X[:, j])).max() <= FP64_TOL
