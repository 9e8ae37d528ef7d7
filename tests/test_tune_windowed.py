"""The windowed autotuner times the library's own launch among its candidates:
rows split where the library splits them, every number of wavefronts it uses."""
import torch

from paper_0910_4836_amd import autotune, spmv as S


def test_the_default_launch_is_a_candidate(monkeypatch, tmp_path):
    launches = []
    monkeypatch.setattr(S, "jds_blocked_windowed_from_csr", lambda A, C, sigma: (C, sigma))
    monkeypatch.setattr(S, "spmv_jds_blocked_tiled", lambda B, x, y, **kw: launches.append((B, kw)))
    monkeypatch.setattr(autotune, "_device_key", lambda: "cpu")
    monkeypatch.setattr(autotune, "_time", lambda fn, **kw: (fn(), float(len(launches)))[1])
    A = S.CSR(4, 4, torch.zeros(5, dtype=torch.int32), torch.zeros(8, dtype=torch.int32), torch.zeros(8))
    tuner = autotune.Autotuner(str(tmp_path / "tune.json"))
    got = tuner.tune_windowed(A, torch.zeros(4), 2)
    assert all(kw.get("max_iters", 0) == 0 for _, kw in launches)
    for B in {B for B, _ in launches}:
        assert {(kw["unroll"], kw["wg_waves"]) for b, kw in launches if b == B} == {(u, w) for u in (4, 8) for w in (4, 8, 16)}
    again = autotune.Autotuner(str(tmp_path / "tune.json"))
    assert again.tune_windowed(A, torch.zeros(4), 2) == got and not again.log
