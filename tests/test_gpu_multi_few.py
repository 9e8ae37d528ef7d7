"""JDS products of one to four vectors and one more, on both sides of the row
count where a row's diagonals are split further.  Small whole numbers: every
sum is exact in FP32, so the results are compared for equality."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import gpu_csr, to_dev, to_np

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_0910_4836_amd")


@pytest.mark.parametrize("n,longest", [(1, 3), (700, 40), (299_999, 70), (300_001, 70), (300_001, 9)])
def test_few_vectors(n, longest):
    rng = np.random.default_rng(n + longest)
    lengths = rng.integers(0, 6, n)
    lengths[rng.integers(0, n, 1 + n // 1000)] = longest
    r = np.repeat(np.arange(n), lengths).astype(np.int32)
    start = rng.integers(0, 5000 - longest, n)
    c = (np.repeat(start - np.cumsum(lengths) + lengths, lengths) + np.arange(r.size)).astype(np.int32)
    v = rng.integers(-3, 4, r.size).astype(np.float64)
    A = oracle.csr_from_coo(n, 5000, r, c, v)
    X = rng.integers(-3, 4, (5000, 5)).astype(np.float64)
    want = oracle.spmm_crs(A, X)
    J = sp.jds_from_csr(gpu_csr(sp, r, c, v, n, 5000))
    for val, vec in ((torch.float64, torch.float64), (torch.float32, torch.float32), (torch.bfloat16, torch.float32)):
        Jq = J.with_values(J.jd_val if val == torch.float64 else sp.spmv_convert_values(J.jd_val, val))
        for k in (1, 2, 3, 4, 5):
            Xd = to_dev(X[:, :k].T.copy()).to(vec).t()
            assert np.array_equal(to_np(sp.spmm_jds(Jq, Xd)).astype(np.float64), want[:, :k]), (val, k)
