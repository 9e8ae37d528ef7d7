"""Staged CRS products at the row lengths where the trips over a lane's share
of a row change (5, 8 and 10 entries per lane), alone and beside other rows,
for blocks of up to 1,024 entries and larger ones."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import FP64_TOL, gpu_csr, max_err, to_dev

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_0910_4836_amd")


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("block_nnz", [256, 1024, 2048])
@pytest.mark.parametrize("length", [1, 4, 5, 6, 8, 9, 10, 11, 16, 17, 18, 19, 20, 21, 33, 36, 40, 41, 80, 81, 170])
def test_row_lengths(length, block_nnz, mixed):
    rng = np.random.default_rng(length + block_nnz)
    n, n_cols = 307, 900
    lengths = np.full(n, length)
    if mixed:
        lengths[rng.integers(0, n, 40)] = rng.integers(0, length + 1, 40)
    r = np.repeat(np.arange(n), lengths).astype(np.int32)
    c = np.concatenate([rng.choice(n_cols, k, replace=False) for k in lengths]).astype(np.int32)
    v, x = rng.standard_normal(r.size), rng.uniform(-1, 1, n_cols)
    A = sp.spmv_crs_plan(gpu_csr(sp, r, c, v, n, n_cols), block_nnz)
    A.staged = True
    R = oracle.csr_from_coo(n, n_cols, r, c, v)
    assert max_err(sp.spmv_crs(A, to_dev(x)), oracle.spmv_crs(R, x), oracle.row_absdot(R, x)) <= FP64_TOL
    # FP32: a sum of m products in any order is off by at most m roundings
    vf, xf = v.astype(np.float32), x.astype(np.float32)
    R = oracle.csr_from_coo(n, n_cols, r, c, vf.astype(np.float64))
    Af = A.with_values(sp.spmv_convert_values(A.val, torch.float32))
    Af.staged = True
    err = oracle.rel_err(sp.spmv_crs(Af, to_dev(xf)).cpu().numpy(), oracle.spmv_crs(R, xf.astype(np.float64)),
                         oracle.row_absdot(R, xf.astype(np.float64)))
    assert np.all(err <= (R.row_lengths() + 1) * 2.0 ** -24 * 1.001)


@pytest.mark.parametrize("length,longest,block_nnz,staged", [
    (16, 16, 0, True), (15, 64, 0, False), (17, 64, 0, True), (17, 65, 0, False), (20, 20, 1024, True),
    (20, 20, 512, False), (20, 20, 2048, False)])
def test_kernel_follows_from_the_rows(monkeypatch, length, longest, block_nnz, staged):
    from paper_0910_4836_amd import spmv as module
    rng = np.random.default_rng(length + longest)
    n = 2000
    lengths = np.full(n, length)
    lengths[5] = longest
    r = np.repeat(np.arange(n), lengths).astype(np.int32)
    c = np.concatenate([rng.choice(n, k, replace=False) for k in lengths]).astype(np.int32)
    v, x = rng.standard_normal(r.size), rng.uniform(-1, 1, n)
    A = sp.spmv_crs_plan(gpu_csr(sp, r, c, v, n, n), block_nnz)
    names, call = [], module.call
    monkeypatch.setattr(module, "call", lambda name, *args: (names.append(name), call(name, *args))[1])
    y = sp.spmv_crs(A, to_dev(x))
    assert names == ["spmv_crs_staged" if staged else "spmv_crs"]
    R = oracle.csr_from_coo(n, n, r, c, v)
    assert max_err(y, oracle.spmv_crs(R, x), oracle.row_absdot(R, x)) <= FP64_TOL
