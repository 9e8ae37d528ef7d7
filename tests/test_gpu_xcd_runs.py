"""Workgroups and tile records dealt to the XCDs in runs: sizes whose last
runs are not whole, and both sides of the sizes at which runs begin."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import FP64_TOL, gpu_csr, max_err, to_dev, to_np

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_0910_4836_amd")


def matrix(n, lengths, seed):
    rng = np.random.default_rng(seed)
    r = np.repeat(np.arange(n, dtype=np.int32), lengths)
    # distinct columns of a row: one in each of its equal strata
    pos = np.arange(r.size) - np.repeat(np.cumsum(lengths) - lengths, lengths)
    per = n // np.repeat(lengths, lengths)
    c = (pos * per + (rng.random(r.size) * per).astype(np.int64)).astype(np.int32)
    v = rng.standard_normal(r.size)
    x = rng.uniform(-1, 1, n)
    R = oracle.csr_from_coo(n, n, r, c, v)
    return gpu_csr(sp, r, c, v, n, n), x, oracle.spmv_crs(R, x), oracle.row_absdot(R, x), R, rng


def check_forms(A, x, want, D):
    J = sp.jds_from_csr(A)
    B = sp.jds_blocked_from_jds(J, 64)
    xd = to_dev(x)
    for f, M in ((sp.spmv_jds, J), (sp.spmv_jds_tiled, J), (sp.spmv_jds_blocked, B), (sp.spmv_jds_blocked_tiled, B)):
        assert max_err(f(M, xd), want, D) <= FP64_TOL, f.__name__
    return J


@pytest.mark.parametrize("longest", [32, 33, 200])
@pytest.mark.parametrize("n", [300, 1000, 4100, 8192, 8193, 33_000])
def test_partial_runs(n, longest):
    lengths = np.random.default_rng(n).integers(1, longest + 1, n)
    lengths[0] = longest
    A, x, want, D, R, rng = matrix(n, lengths, n + longest)
    J = check_forms(A, x, want, D)
    X = rng.uniform(-1, 1, (n, 3))
    Y, W = to_np(sp.spmm_jds(J, torch.from_numpy(np.ascontiguousarray(X.T)).to("cuda").t())), oracle.spmm_crs(R, X)
    for j in range(3):
        assert oracle.rel_err(Y[:, j], W[:, j], oracle.row_absdot(R, X[:, j])).max() <= FP64_TOL


@pytest.mark.parametrize("n,usual,longest", [(999_999, 1, 20), (1_000_001, 1, 20), (1_500_001, 2, 60), (99_999, 5, 60),
                                             (100_001, 5, 60)])
def test_sizes_at_which_runs_begin(n, usual, longest):
    lengths = np.full(n, usual)
    lengths[np.random.default_rng(n).integers(0, n, 3001)] = longest
    check_forms(*matrix(n, lengths, n)[:4])
