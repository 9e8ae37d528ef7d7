"""The entry-order CRS kernel on rows for which a product without a choice
takes the staged one."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import FP64_TOL, gpu_csr, max_err, to_dev

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_0910_4836_amd")


@pytest.mark.parametrize("n", [1, 51, 52, 257, 200_000])
def test_entry_order_kernel(n):
    rng = np.random.default_rng(n)
    r = np.repeat(np.arange(n), 20).astype(np.int32)
    c = np.concatenate([np.sort(rng.choice(2000, 20, replace=False)) for _ in range(min(n, 257))]).astype(np.int32)
    c = np.resize(c, r.size)
    v, x = rng.standard_normal(r.size), rng.uniform(-1, 1, 2000)
    A = gpu_csr(sp, r, c, v, n, 2000)
    A.staged = False
    R = oracle.csr_from_coo(n, 2000, r, c, v)
    assert max_err(sp.spmv_crs(A, to_dev(x)), oracle.spmv_crs(R, x), oracle.row_absdot(R, x)) <= FP64_TOL
    # FP32: a sum of m products in any order is off by at most m roundings
    vf, xf = v.astype(np.float32), x.astype(np.float32)
    R = oracle.csr_from_coo(n, 2000, r, c, vf.astype(np.float64))
    y = sp.spmv_crs(A.with_values(sp.spmv_convert_values(A.val, torch.float32)), to_dev(xf)).cpu().numpy()
    err = oracle.rel_err(y, oracle.spmv_crs(R, xf.astype(np.float64)), oracle.row_absdot(R, xf.astype(np.float64)))
    assert np.all(err <= 21 * 2.0 ** -24 * 1.001)
