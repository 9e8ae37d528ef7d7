"""Which form a batched product runs: staged in LDS where nothing else is asked
for at 64 rows per wavefront, the plain form with the diagonals per trip that
were given otherwise; the autotuner times each form once."""
import numpy as np
import pytest
import torch

from paper_0910_4836_amd import autotune, spmv as S


BATCHED = S.Batched


def batched(rows_per_wave, unroll, n_workgroups):
    B = object.__new__(BATCHED)
    B.rows_per_wave, B.unroll, B.n_workgroups = rows_per_wave, unroll, n_workgroups
    B.n_tiles, B.total_rows = 1, 4
    B.plan = B.perm = B.bl_col = torch.zeros(4, dtype=torch.int32)
    B.bl_val = torch.zeros(4)
    return B


@pytest.mark.parametrize("rows_per_wave,unroll,n_workgroups,passed", [
    (64, 0, 0, (0, 0)), (0, 0, 0, (0, 0)),                                      # staged
    (64, 2, 0, (2, 0)), (64, 4, 0, (4, 0)), (64, 8, 0, (8, 0)), (64, 3, 0, (3, 0)),
    (64, 0, 96, (0, 96)), (64, 8, 96, (8, 96)), (16, 0, 0, (4, 0)), (16, 2, 0, (2, 0))])
def test_the_library_gets_what_was_asked_for(monkeypatch, rows_per_wave, unroll, n_workgroups, passed):
    calls = []
    monkeypatch.setattr(S, "call", lambda name, *args: calls.append(args))
    monkeypatch.setattr(S, "_stream", lambda: 0)
    batched(rows_per_wave, unroll, n_workgroups)(torch.zeros(4), torch.zeros(4))
    assert calls[0][7:9] == passed


@pytest.mark.parametrize("n_workgroups", [0, 96])
def test_tuner_times_every_form_once(monkeypatch, tmp_path, n_workgroups):
    timed = []

    monkeypatch.setattr(S, "Batched", lambda mats, rows_per_wave=64, unroll=0, n_workgroups=0:
                        batched(rows_per_wave, unroll, n_workgroups))
    monkeypatch.setattr(S, "jds_blocked_from_jds", lambda J, C: None)
    monkeypatch.setattr(autotune, "_device_key", lambda: "cpu")
    launches = []
    monkeypatch.setattr(S, "call", lambda name, *args: launches.append(args[7:9]))
    monkeypatch.setattr(S, "_stream", lambda: 0)

    def time(fn, **kw):
        fn()
        timed.append(launches[-1])
        return 1.0 if launches[-1] == (0, 0) else 2.0
    monkeypatch.setattr(autotune, "_time", time)
    J = S.JDS(4, 4, None, None, None, np.array([0, 4], np.int32), None, torch.zeros(4))
    tuner = autotune.Autotuner(str(tmp_path / "tune.json"), cs=(64,))
    got = tuner.tune_batched([J], n_workgroups=n_workgroups)
    plain = [(u, n_workgroups) for u in (2, 4, 8)]
    if n_workgroups:
        assert timed == plain * 3 and got == (64, 64, 2)
    else:
        assert timed == plain + [(0, 0)] + plain * 2 and got == (64, 64, 0)
    # the choice comes back from the cache, for the number of workgroups it was made for
    again = autotune.Autotuner(str(tmp_path / "tune.json"), cs=(64,))
    assert again.tune_batched([J], n_workgroups=n_workgroups) == got and not again.log
    assert again.lookup("batched:" + again._batch_signature([J]), ("C", "R", "U")) is None


@pytest.mark.gpu
@pytest.mark.parametrize("unroll", [2, 4, 8])
def test_plain_form_at_64_rows(unroll):
    import oracle
    from gpu_common import gpu_csr, to_dev, to_np
    rng = np.random.default_rng(unroll)
    mats, blocked = [], []
    for n, m, per_row in ((1, 60, 3), (700, 2500, 41), (64, 9000, 7)):
        r = np.repeat(np.arange(n), per_row).astype(np.int32)
        c = np.concatenate([np.sort(rng.choice(m, per_row, replace=False)) for _ in range(n)]).astype(np.int32)
        v = rng.integers(-3, 4, r.size).astype(np.float64)
        mats.append((oracle.csr_from_coo(n, m, r, c, v), m))
        blocked.append(S.jds_blocked_from_jds(S.jds_from_csr(gpu_csr(S, r, c, v, n, m, torch.float32))))
    x = rng.integers(-3, 4, sum(m for _, m in mats)).astype(np.float32)          # whole numbers: exact in FP32
    y = to_np(S.Batched(blocked, unroll=unroll)(to_dev(x)))
    at = np.cumsum([0] + [m for _, m in mats])
    want = np.concatenate([oracle.spmv_crs(R, x[a:b].astype(np.float64)) for (R, _), a, b in zip(mats, at, at[1:])])
    assert np.array_equal(y.astype(np.float64), want)
    with pytest.raises(S.SpmvError, match="unroll must be"):
        S.Batched(blocked, unroll=3)(to_dev(x))
