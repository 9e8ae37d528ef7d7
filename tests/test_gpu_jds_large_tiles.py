"""JDS tile plans on both sides of the row counts and longest rows where the
launch and the runs of records change.  Small whole numbers: every sum is exact
in FP32, so the results are compared for equality."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import gpu_csr, to_dev, to_np

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_0910_4836_amd")


@pytest.mark.parametrize("n,longest", [(1_749_999, 70), (1_750_000, 70), (1_999_999, 40), (2_000_000, 40),
                                       (2_000_000, 33), (2_000_000, 32), (2_000_000, 65)])
def test_tiles(n, longest):
    rng = np.random.default_rng(n + longest)
    lengths = rng.integers(0, 5, n)
    lengths[rng.integers(0, n, 20_000)] = rng.integers(5, longest + 1, 20_000)
    lengths[n // 2] = longest
    r = np.repeat(np.arange(n), lengths).astype(np.int32)
    m = 50_000
    start = rng.integers(0, m - longest, n)
    c = (np.repeat(start - np.cumsum(lengths) + lengths, lengths) + np.arange(r.size)).astype(np.int32)
    v, x = rng.integers(-3, 4, r.size).astype(np.float64), rng.integers(-3, 4, m).astype(np.float64)
    want = oracle.spmv_crs(oracle.csr_from_coo(n, m, r, c, v), x)
    J = sp.jds_from_csr(gpu_csr(sp, r, c, v, n, m))
    assert np.array_equal(to_np(sp.spmv_jds_tiled(J, to_dev(x))), want)
    Jf = J.with_values(sp.spmv_convert_values(J.jd_val, torch.float32))
    y = sp.spmv_jds_tiled(Jf, to_dev(x).float())
    assert np.array_equal(to_np(y).astype(np.float64), want)
    # the summed value gradient walks the same plan
    g = to_dev(rng.integers(-3, 4, n).astype(np.float64))
    pairs = [(1.0, g, to_dev(x)), (2.0, g * 2, to_dev(x) + 1)]
    total = sp.spmv_grad_vals_jds(J, pairs[0][1], pairs[0][2])
    sp.spmv_grad_vals_jds(J, pairs[1][1], pairs[1][2], total, 2.0, 1.0)
    assert torch.equal(sp.spmv_grad_vals_jds_sum(J, pairs), total)
