"""Autotuner for the SpMV launch parameters: the CRS plan's entries per
block, and for the JDS and blocked-JDS products the slice height C, rows per
wavefront R, diagonals per trip U, diagonals per wavefront before a row is
split (max_iters) and wavefronts per workgroup W, chosen per row-length
signature and cached.

The signature of a matrix is (log2 of its row count, its longest row, its
mean row length rounded to a power of two); matrices that share it share the
best layout.  Tuning times candidate layouts with HIP events (the library's
own kernels, nothing else) on a sample of the matrices of one signature and
keeps the fastest.  The cache is a JSON file keyed by device name and
signature, so a later run with the same kind of matrices skips the search.

Tuning is a host-side choice of launch parameters; every candidate computes
the same y up to summation order.
"""
from __future__ import annotations

import json
import math
import os
from typing import Dict, Iterable, List, Sequence, Tuple

import numpy as np
import torch

from . import spmv as S

DEFAULT_CACHE = os.path.join(os.path.expanduser("~"), ".cache", "spmv_autotune.json")
C_CANDIDATES = (64, 128, 256)
R_CANDIDATES = (0, 64, 32, 16)      # 0: the library's choice per length class
U_CANDIDATES = (2, 4, 8)
MAX_ITERS_CANDIDATES = (0, 64, 128)  # 0: the library default
W_CANDIDATES = (16, 8, 4)            # wavefronts per workgroup
BLOCK_NNZ_CANDIDATES = (512, 1024, 2048)
STAGED_BLOCK_NNZ_CANDIDATES = (512, 1024, 2048, 4096)
SIGMA_CANDIDATES = (16384, 65536, 262144)   # windowed order: rows per window


def signature(n_rows: int, longest: int, nnz: int) -> str:
    """(log2 of the row count, the longest row, the mean row length rounded
    to a power of two)."""
    if n_rows == 0 or nnz == 0:
        return "empty"
    mean = nnz / n_rows
    return f"n2^{int(math.log2(max(n_rows, 1)))}/max{longest}/mean2^{int(round(math.log2(max(mean, 1.0))))}"


def _device_key() -> str:
    """The GPU architecture and compute-unit count (the marketing name can be
    empty, e.g. under a profiler)."""
    p = torch.cuda.get_device_properties(torch.cuda.current_device())
    return f"{getattr(p, 'gcnArchName', '') or p.name}/{p.multi_processor_count}CU"


def _load(path):
    try:
        with open(path) as f:
            return json.load(f)
    except (OSError, ValueError):
        return {}


def _store(path, data):
    os.makedirs(os.path.dirname(path) or ".", exist_ok=True)
    tmp = path + ".tmp"
    with open(tmp, "w") as f:
        json.dump(data, f, indent=1, sort_keys=True)
    os.replace(tmp, path)


def _time(fn, reps=10, warm=2) -> float:
    for _ in range(warm):
        fn()
    a = torch.cuda.Event(enable_timing=True)
    b = torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    a.record()
    for _ in range(reps):
        fn()
    b.record()
    torch.cuda.synchronize()
    return a.elapsed_time(b) / reps


class Autotuner:
    """Chooses (C, R, U) for blocked-JDS matrices; results cached per signature."""

    def __init__(self, cache_path: str = DEFAULT_CACHE, cs=C_CANDIDATES, rs=R_CANDIDATES, us=U_CANDIDATES,
                 ws=W_CANDIDATES):
        self.cache_path = cache_path
        self.cs, self.rs, self.us, self.ws = tuple(cs), tuple(rs), tuple(us), tuple(ws)
        self.cache = _load(cache_path)
        self.log: List[dict] = []

    def lookup(self, sig: str, keys: Sequence[str]):
        ent = self.cache.get(_device_key(), {}).get(sig)
        if ent is None or any(k not in ent for k in keys):
            return None
        return tuple(ent[k] for k in keys)

    def _record(self, sig, keys, best, timings):
        ent = dict(zip(keys, best))
        ent["ms"] = round(timings[best], 5)
        self.cache.setdefault(_device_key(), {})[sig] = ent
        _store(self.cache_path, self.cache)

    def tune_batched(self, jds_list: Sequence[S.JDS], sample: int = 16,
                     n_workgroups: int = 0) -> Tuple[int, int, int]:
        """Best (C, R, U) for a batch of matrices sharing one signature: builds
        the blocked layout of up to `sample` of them for each C and times the
        launch of n_workgroups for each (R, U) of the plain form and, where no
        number of workgroups is given, the staged form (U = 0) at 64 rows per
        wavefront."""
        sig = f"batched2:{f'wg{n_workgroups}:' if n_workgroups else ''}" + self._batch_signature(jds_list)
        hit = self.lookup(sig, ("C", "R", "U"))
        if hit is not None:
            return hit
        pick = list(jds_list[:: max(1, len(jds_list) // sample)])[:sample]
        timings: Dict[Tuple[int, int, int], float] = {}
        staged: Dict[Tuple[int, int, int], float] = {}
        # 0 rows per wavefront are 64 here
        rs = [R for R in self.rs if R or 64 not in self.rs]
        xs = [torch.rand(J.n_cols, dtype=torch.float32, device=J.jd_val.device) for J in pick]
        x = torch.cat(xs)
        for C in self.cs:
            mats = [S.jds_blocked_from_jds(J, C) for J in pick]
            for R in rs:
                Bt = S.Batched(mats, rows_per_wave=R, n_workgroups=n_workgroups)
                y = torch.empty(Bt.total_rows, dtype=torch.float32, device=x.device)
                for U in self.us:
                    Bt.unroll = U
                    timings[(C, R, U)] = _time(lambda: Bt(x, y))
                if R in (0, 64) and n_workgroups == 0:
                    Bt.unroll = 0
                    staged[(C, R, 0)] = _time(lambda: Bt(x, y))
            del mats
        self.log.append({"signature": sig, "timings_ms": {f"C{c}_R{r}_U{u}": round(t, 5)
                                                          for (c, r, u), t in timings.items()},
                         "staged_ms": {f"C{c}": round(t, 5) for (c, _, _), t in staged.items()}})
        timings.update(staged)
        best = min(timings, key=timings.get)
        self._record(sig, ("C", "R", "U"), best, timings)
        return best

    @staticmethod
    def _batch_signature(jds_list: Iterable[S.JDS]) -> str:
        mx, tot, rows, nmat = 0, 0, 0, 0
        for J in jds_list:
            mx = max(mx, J.ndiag)
            tot += J.nnz
            rows += J.n
            nmat += 1
        mean = tot / max(rows, 1)
        return f"mats{nmat}/max{mx}/mean2^{int(round(math.log2(max(mean, 1.0))))}"

    def tune_blocked(self, J: S.JDS, x: torch.Tensor) -> Tuple[int, int, int, int]:
        """Best (C, R, U, W) for one large matrix in blocked-JDS storage."""
        sig = "single:" + signature(J.n, J.ndiag, int(J.h_jd_ptr[J.ndiag]))
        keys = ("C", "R", "U", "W")
        hit = self.lookup(sig, keys)
        if hit is not None:
            return hit
        timings = {}
        y = torch.empty(J.n, dtype=x.dtype, device=x.device)
        for C in self.cs:
            B = S.jds_blocked_from_jds(J, C)
            for R in self.rs:
                for U in self.us:
                    for W in self.ws:
                        timings[(C, R, U, W)] = _time(lambda: S.spmv_jds_blocked(B, x, y, rows_per_wave=R, unroll=U,
                                                                                 wg_waves=W))
            del B
        best = min(timings, key=timings.get)
        self.log.append({"signature": sig, "timings_ms": {f"C{c}_R{r}_U{u}_W{w}": round(t, 5)
                                                          for (c, r, u, w), t in timings.items()}})
        self._record(sig, keys, best, timings)
        return best


    def tune_windowed(self, A: S.CSR, x: torch.Tensor, longest: int, sigmas=SIGMA_CANDIDATES,
                      Cs=(64, 128), Us=(4, 8), Ws=(4, 8, 16)) -> Tuple[int, int, int, int]:
        """Best (sigma, C, U, W) for one large matrix in windowed blocked-JDS
        storage launched from its tile plan, with rows split where the library
        splits them (max_iters 0: with 32 the power-law rows of 2 M take 312 us
        at best, of 60 k 38, with the library's choice 291 and 20)."""
        sig = "windowed2:" + signature(A.n_rows, longest, A.nnz)
        keys = ("sigma", "C", "U", "W")
        hit = self.lookup(sig, keys)
        if hit is not None:
            return hit
        timings = {}
        y = torch.empty(A.n_rows, dtype=x.dtype, device=x.device)
        for sg in sigmas:
            for C in Cs:
                B = S.jds_blocked_windowed_from_csr(A, C, sg)
                for U in Us:
                    for W in Ws:
                        timings[(sg, C, U, W)] = _time(lambda: S.spmv_jds_blocked_tiled(B, x, y, unroll=U,
                                                                                        wg_waves=W))
                del B
        best = min(timings, key=timings.get)
        self.log.append({"signature": sig, "timings_ms": {f"s{a}_C{c}_U{u}_W{w}": round(t, 5)
                                                          for (a, c, u, w), t in timings.items()}})
        self._record(sig, keys, best, timings)
        return best

    def tune_jds(self, J: S.JDS, x: torch.Tensor, mis=MAX_ITERS_CANDIDATES) -> Tuple[int, int, int]:
        """Best (U, max_iters, W) for one large matrix in JDS storage."""
        sig = "jds:" + signature(J.n, J.ndiag, int(J.h_jd_ptr[J.ndiag]))
        keys = ("U", "max_iters", "W")
        hit = self.lookup(sig, keys)
        if hit is not None:
            return hit
        timings = {}
        y = torch.empty(J.n, dtype=x.dtype, device=x.device)
        for U in self.us:
            for mi in mis:
                for W in self.ws:
                    timings[(U, mi, W)] = _time(lambda: S.spmv_jds(J, x, y, unroll=U, max_iters=mi, wg_waves=W))
        best = min(timings, key=timings.get)
        self.log.append({"signature": sig, "timings_ms": {f"U{u}_mi{m}_W{w}": round(t, 5)
                                                          for (u, m, w), t in timings.items()}})
        self._record(sig, keys, best, timings)
        return best

    def _tune_launch(self, sig: str, plain, tiled, reps: int = 20) -> bool:
        hit = self.lookup(sig, ("tiled",))
        if hit is not None:
            return bool(hit[0])
        # alternate the two launches so that clock and cache drift hit both alike
        t = {False: 0.0, True: 0.0}
        for _ in range(3):
            t[False] += _time(plain, reps=reps)
            t[True] += _time(tiled, reps=reps)
        timings = {(False,): t[False] / 3, (True,): t[True] / 3}
        best = min(timings, key=timings.get)
        self.log.append({"signature": sig, "timings_ms": {"plain": round(timings[(False,)], 5),
                                                          "tiled": round(timings[(True,)], 5)}})
        self._record(sig, ("tiled",), best, timings)
        return bool(best[0])

    def tune_jds_launch(self, J: S.JDS, x: torch.Tensor, U: int, mi: int, W: int) -> bool:
        """Whether the XCD-local tile plan (spmv_jds_tiled) beats the class
        plan (spmv_jds) for J at this launch shape."""
        sig = f"jds_launch:U{U}_mi{mi}_W{W}:" + signature(J.n, J.ndiag, int(J.h_jd_ptr[J.ndiag]))
        y = torch.empty(J.n, dtype=x.dtype, device=x.device)
        return self._tune_launch(sig, lambda: S.spmv_jds(J, x, y, unroll=U, max_iters=mi, wg_waves=W),
                                 lambda: S.spmv_jds_tiled(J, x, y, unroll=U, max_iters=mi, wg_waves=W))

    def tune_blocked_launch(self, B: S.Blocked, x: torch.Tensor, R: int, U: int, W: int) -> bool:
        """Whether the tile plan (spmv_jds_blocked_tiled; XCD-local on the
        globally sorted order) beats the class plan (spmv_jds_blocked) for B
        at this launch shape."""
        sig = f"blocked_launch:C{B.C}_R{R}_U{U}_W{W}:" + signature(B.n, int(B.h_slice_nd[0]) if len(B.h_slice_nd)
                                                                    else 0, B.padded)
        y = torch.empty(B.n, dtype=x.dtype, device=x.device)
        return self._tune_launch(sig, lambda: S.spmv_jds_blocked(B, x, y, rows_per_wave=R, unroll=U, wg_waves=W),
                                 lambda: S.spmv_jds_blocked_tiled(B, x, y, unroll=U, rows_per_wave=R, wg_waves=W))


def tune_crs(tuner: "Autotuner", A: S.CSR, x: torch.Tensor, longest: int,
             candidates=BLOCK_NNZ_CANDIDATES, staged_candidates=STAGED_BLOCK_NNZ_CANDIDATES) -> int:
    """Best CRS plan for one large matrix (its longest row passed by the
    caller): entries per block, and whether the gathers go in entry order
    (spmv_crs) or row order (spmv_crs_staged).  A's plan is rebuilt with the
    choice and A.staged set; the block size is returned."""
    sig = "crs3:" + signature(A.n_rows, longest, A.nnz)
    ent = tuner.cache.get(_device_key(), {}).get(sig)
    if ent is None:
        timings = {}
        y = torch.empty(A.n_rows, dtype=x.dtype, device=x.device)
        for staged, cands in ((False, candidates), (True, staged_candidates)):
            for bn in cands:
                Ab = S.spmv_crs_plan(S.CSR(A.n_rows, A.n_cols, A.row_ptr, A.col_idx, A.val), bn)
                Ab.staged = staged
                timings[(staged, bn)] = _time(lambda: S.spmv_crs(Ab, x, y))
                del Ab
        best = min(timings, key=timings.get)
        tuner.log.append({"signature": sig, "timings_ms": {("staged" if st else "block") + str(b): round(t, 5)
                                                            for (st, b), t in timings.items()}})
        ent = {"block_nnz": best[1], "staged": best[0], "ms": round(timings[best], 5)}
        tuner.cache.setdefault(_device_key(), {})[sig] = ent
        _store(tuner.cache_path, tuner.cache)
    S.spmv_crs_plan(A, ent["block_nnz"])
    A.staged = bool(ent["staged"])
    return ent["block_nnz"]


def tune_crs_sym(tuner: "Autotuner", M: S.SymCSR, x: torch.Tensor, longest: int,
                 candidates=BLOCK_NNZ_CANDIDATES, staged_candidates=STAGED_BLOCK_NNZ_CANDIDATES) -> int:
    """Best plan of a one-triangle matrix (longest row of its upper triangle
    passed by the caller): entries per block, and whether the kernel walks
    the entries in entry order (spmv_crs_sym) or row order
    (spmv_crs_sym_staged).  M's plan is rebuilt with the choice and
    M.upper.staged set; the block size is returned."""
    U = M.upper
    sig = "crs_sym2:" + signature(U.n_rows, longest, U.nnz)
    ent = tuner.cache.get(_device_key(), {}).get(sig)
    if ent is None:
        timings = {}
        y = torch.empty(U.n_rows, dtype=x.dtype, device=x.device)
        for staged, cands in ((False, candidates), (True, staged_candidates)):
            for bn in cands:
                Mb = S.SymCSR(S.spmv_crs_plan(S.CSR(U.n_rows, U.n_cols, U.row_ptr, U.col_idx, U.val), bn))
                Mb.upper.staged = staged
                timings[(staged, bn)] = _time(lambda: S.spmv_crs_sym(Mb, x, y))
                del Mb
        best = min(timings, key=timings.get)
        tuner.log.append({"signature": sig, "timings_ms": {("staged" if st else "block") + str(b): round(t, 5)
                                                            for (st, b), t in timings.items()}})
        ent = {"block_nnz": best[1], "staged": best[0], "ms": round(timings[best], 5)}
        tuner.cache.setdefault(_device_key(), {})[sig] = ent
        _store(tuner.cache_path, tuner.cache)
    S.spmv_crs_plan(U, ent["block_nnz"])
    U.staged = bool(ent["staged"])
    return ent["block_nnz"]


def tune_spmm_crs(tuner: "Autotuner", A: S.CSR, k: int, dtype: torch.dtype, longest: int,
                  candidates=(256, 512, 1024)) -> S.CSR:
    """The CRS plan (entries per block) for k-vector products with A: returns a
    copy of A's structure carrying the best plan for spmm_crs (A's own plan,
    used by the single-vector product, is left alone)."""
    sig = f"spmm_crs:k{k}:{str(dtype).replace('torch.', '')}:" + signature(A.n_rows, longest, A.nnz)
    ent = tuner.cache.get(_device_key(), {}).get(sig)
    plans = {}
    if ent is None:
        X = S.colmajor(A.n_cols, k, dtype, A.device)
        X.copy_(torch.rand(A.n_cols, k, dtype=dtype, device=A.device))
        Y = S.colmajor(A.n_rows, k, dtype, A.device)
        ws = S.spmm_workspace(A.n_cols, k, dtype, A.device)
        timings = {}
        for bn in candidates:
            Ab = S.spmv_crs_plan(S.CSR(A.n_rows, A.n_cols, A.row_ptr, A.col_idx, A.val), bn)
            plans[bn] = Ab
            timings[bn] = _time(lambda: S.spmm_crs(Ab, X, Y, ws=ws), reps=5, warm=1)
        best = min(timings, key=timings.get)
        tuner.log.append({"signature": sig, "timings_ms": {f"block{b}": round(t, 5) for b, t in timings.items()}})
        ent = {"block_nnz": best, "ms": round(timings[best], 5)}
        tuner.cache.setdefault(_device_key(), {})[sig] = ent
        _store(tuner.cache_path, tuner.cache)
        del X, Y, ws
    bn = ent["block_nnz"]
    return plans.get(bn) or S.spmv_crs_plan(S.CSR(A.n_rows, A.n_cols, A.row_ptr, A.col_idx, A.val), bn)


def build_batched(jds_list: Sequence[S.JDS], tuner: Autotuner = None, n_workgroups: int = 0) -> S.Batched:
    """Blocked layouts and the persistent plan for many matrices, with the
    slice height / rows per wavefront / unroll the autotuner picks."""
    tuner = tuner or Autotuner()
    C, R, U = tuner.tune_batched(jds_list, n_workgroups=n_workgroups)
    mats = [S.jds_blocked_from_jds(J, C) for J in jds_list]
    return S.Batched(mats, rows_per_wave=R, unroll=U, n_workgroups=n_workgroups)
