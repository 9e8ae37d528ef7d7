"""Batched products whose x is staged in LDS: the depths at which the pass over
a row's entries changes, the widths at which x takes one, two and more pieces
or is gathered directly, every alignment of x, groups of several matrices,
rows that accumulate in FP64 and values that are not finite."""
import numpy as np
import pytest
import torch

import oracle
from gpu_common import gpu_csr, to_dev, to_np

pytestmark = pytest.mark.gpu
sp = pytest.importorskip("paper_0910_4836_amd")

PIECE, WHOLE = 9980, 19964              # columns of one of two pieces, of a single one


def matrix(rng, n, n_cols, depth):
    """Rows of 1 to `depth` entries, some empty; columns 0 and n_cols - 1 used."""
    lengths = rng.integers(1, depth + 1, n)
    lengths[rng.integers(0, n, n // 10)] = 0
    lengths[0] = depth
    r = np.repeat(np.arange(n), lengths).astype(np.int32)
    c = np.concatenate([np.sort(rng.choice(n_cols, k, replace=False)) for k in lengths]).astype(np.int32)
    c[0], c[depth - 1] = 0, n_cols - 1
    return r, c, rng.standard_normal(r.size).astype(np.float32).astype(np.float64), n, n_cols


def check(mats, rng, skew=0, heights=(64,), **kw):
    B = sp.Batched([sp.jds_blocked_from_jds(sp.jds_from_csr(gpu_csr(sp, r, c, v, n, m, torch.float32)),
                                            heights[i % len(heights)]) for i, (r, c, v, n, m) in enumerate(mats)], **kw)
    x = rng.uniform(-1, 1, B.total_cols).astype(np.float32)
    xd = torch.empty(x.size + 4, device="cuda")[skew:skew + x.size]
    xd.copy_(to_dev(x))
    y = to_np(B(xd)).astype(np.float64)
    row = col = 0
    for r, c, v, n, m in mats:
        R, xm = oracle.csr_from_coo(n, m, r, c, v), x[col:col + m].astype(np.float64)
        # a sum of k FP32 products in any order is off by at most k roundings,
        # and one more where an FP64 sum is rounded to the result
        bound = (R.row_lengths() + 1) * 2.0 ** -24 * 1.001 * oracle.row_absdot(R, xm)
        assert np.all(np.abs(y[row:row + n] - oracle.spmv_crs(R, xm)) <= bound), (n, m)
        row, col = row + n, col + m


@pytest.mark.parametrize("depth", [1, 2, 7, 8, 9, 16, 17, 24, 25, 32, 33, 40, 41, 80, 81, 130])
def test_depths(depth):
    rng = np.random.default_rng(depth)
    check([matrix(rng, n, 900, depth) for n in (512, 1, 1100, 63)], rng)


@pytest.mark.parametrize("skew", [0, 1, 2, 3])
@pytest.mark.parametrize("n_cols", [45, WHOLE, WHOLE + 1, 2 * PIECE, 2 * PIECE + 1, 3 * PIECE, 3 * PIECE + 1, 39_999,
                                    200_000])
def test_widths_and_alignment(n_cols, skew):
    rng = np.random.default_rng(n_cols + skew)
    # 512 rows are one group: as many columns per slot as four allow, and more
    check([matrix(rng, 512, n_cols, 40), matrix(rng, 700, n_cols, 30)], rng, skew)


def test_groups_of_several_matrices_and_slice_heights():
    rng = np.random.default_rng(7)
    check([matrix(rng, int(n), int(n) + 50, 12) for n in rng.integers(1, 400, 60)], rng, heights=(64, 128, 256))


def test_rows_beyond_the_wide_length_and_other_forms():
    rng = np.random.default_rng(8)
    mats = [matrix(rng, 800, 6000, 20), matrix(rng, 70, 6000, 4200)]
    check(mats, rng)
    check(mats, rng, rows_per_wave=16)
    check(mats, rng, n_workgroups=64)


def test_values_that_are_not_finite_stay_in_their_rows():
    rng = np.random.default_rng(9)
    r, c, v, n, m = matrix(rng, 512, 30_000, 20)
    bad = np.unique(rng.integers(0, r.size, 6))
    v[bad] = np.array([np.inf, -np.inf, np.nan] * 2)[:bad.size]
    B = sp.Batched([sp.jds_blocked_from_jds(sp.jds_from_csr(gpu_csr(sp, r, c, v, n, m, torch.float32)), 64)])
    y = to_np(B(torch.ones(m, device="cuda")))
    want = np.zeros(n)
    np.add.at(want, r, v)
    assert np.array_equal(np.isnan(y), np.isnan(want)) and np.array_equal(np.isposinf(y), np.isposinf(want))
    assert np.array_equal(np.isneginf(y), np.isneginf(want))
    fin = np.isfinite(want)
    assert np.all(np.abs(y[fin] - want[fin]) <= 21 * 2.0 ** -24 * np.bincount(r, np.abs(v), n)[fin])
