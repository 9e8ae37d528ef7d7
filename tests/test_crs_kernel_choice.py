"""Which CRS kernel a product launches: the one A.staged asks for, or, where it
asks for none, the one the rows favour; the autotuner times what it says and
leaves its choice in A.staged.  On the CPU, with the library calls recorded in
place of made."""
import pytest
import torch

from paper_0910_4836_amd import autotune, spmv as S


@pytest.fixture
def launched(monkeypatch):
    names = []
    monkeypatch.setattr(S, "call", lambda name, *args: names.append(name))
    monkeypatch.setattr(S, "_check_dev", lambda *ts: None)
    monkeypatch.setattr(S, "_stream", lambda: 0)

    def plan(A, block_nnz=0):
        A.plan, A.n_blocks, A.block_nnz, A.longest = torch.zeros(2, dtype=torch.int32), 1, block_nnz, 20
        return A
    monkeypatch.setattr(S, "spmv_crs_plan", plan)
    return names


def rows_of(length, staged=None):
    """64 rows of `length` entries with the plan that spmv_crs_plan would leave (longest row 20)."""
    n = 64
    A = S.CSR(n, n, torch.zeros(n + 1, dtype=torch.int32), torch.zeros(n * length, dtype=torch.int32),
              torch.zeros(n * length, dtype=torch.float64))
    if staged is not None:
        A.staged = staged
    return A


@pytest.mark.parametrize("length,staged,kernel", [
    (20, None, "spmv_crs_staged"), (20, False, "spmv_crs"), (20, True, "spmv_crs_staged"),
    (7, None, "spmv_crs"), (7, False, "spmv_crs"), (7, True, "spmv_crs_staged")])
def test_what_is_asked_for_is_launched(launched, length, staged, kernel):
    A = rows_of(length, staged)
    x = torch.zeros(64, dtype=torch.float64)
    S.spmv_crs(A, x)
    S.spmv_crs(A.with_values(A.val.float()), x)
    assert launched == [kernel] * 2
    S.spmv_crs(A, x, use_plan=False)
    assert launched[2] == "spmv_crs"


def test_tuner_times_what_it_stores(launched, monkeypatch, tmp_path):
    timed = []

    def time(fn, **kw):
        fn()
        timed.append(launched[-1])
        return 1.0 if len(timed) == 2 else 2.0           # the second candidate wins
    monkeypatch.setattr(autotune, "_time", time)
    monkeypatch.setattr(autotune, "_device_key", lambda: "cpu")
    tuner = autotune.Autotuner(str(tmp_path / "tune.json"))
    A = rows_of(20)
    bn = autotune.tune_crs(tuner, A, torch.zeros(64, dtype=torch.float64), 20)
    plain, staged = len(autotune.BLOCK_NNZ_CANDIDATES), len(autotune.STAGED_BLOCK_NNZ_CANDIDATES)
    assert timed == ["spmv_crs"] * plain + ["spmv_crs_staged"] * staged
    assert bn == autotune.BLOCK_NNZ_CANDIDATES[1] == 1024 and A.staged is False
    S.spmv_crs(A, torch.zeros(64, dtype=torch.float64))
    assert launched[-1] == "spmv_crs"
