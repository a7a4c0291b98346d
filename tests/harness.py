"""Shared helpers of the GPU parity tests: run the oracle on host copies of the
inputs and compare, element by element, with what the HIP library produced.

Tolerances (fp32 results; ``eps32 = 1e-5`` is the stated relative tolerance):
  pooled output   |gpu - ref| <= eps32 * max(|ref|, absum)      absum = sum |terms|
  updated row     |gpu - ref| <= eps32 * max(|ref|, |W_old| + lr)
  accumulator     |gpu - ref| <= eps32 * S_ref + 2 * eps32 * mean_d(Gabs_d^2)
(the last from d(G^2) = 2 |G| dG with dG <= eps32 * Gabs).  Where a bf16 value
is written the same forms are used with 1e-2.
"""
from __future__ import annotations

from typing import Dict, List, Optional, Sequence

import numpy as np
import torch

from oracle import emb_oracle as oracle
from paper_2508_05700_amd import binding as emb
from paper_2508_05700_amd import workloads as wl

EPS32 = 1e-5
EPS_BF16 = 1e-2
DEV = "cuda:0"


def dev(a: np.ndarray) -> torch.Tensor:
    if a.dtype == np.uint64:
        a = a.view(np.int64)
    if a.dtype == np.uint16:      # bf16 bit patterns
        return torch.from_numpy(a.view(np.int16)).to(DEV).view(torch.bfloat16)
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def host_table(t: torch.Tensor) -> np.ndarray:
    """Device table -> numpy in the oracle's storage format."""
    if t.dtype == torch.bfloat16:
        return t.view(torch.int16).cpu().numpy().view(np.uint16)
    return t.cpu().numpy()


def assert_pooled_close(gpu: np.ndarray, ref: np.ndarray, absum: np.ndarray, eps: float = EPS32, what: str = ""):
    gpu = gpu.reshape(ref.shape).astype(np.float64)
    err = np.abs(gpu - ref.astype(np.float64))
    bound = eps * np.maximum(np.abs(ref.astype(np.float64)), absum)
    bad = err > bound
    assert not bad.any(), "%s: %d of %d pooled values off; worst err/bound %.3g" % (
        what, int(bad.sum()), bad.size, float((err / np.maximum(bound, 1e-300)).max()))
    assert np.isfinite(gpu).all()


def assert_rows_close(gpu: np.ndarray, ref: np.ndarray, old: np.ndarray, lr: float, eps: float = EPS32,
                      what: str = ""):
    gpu, ref, old = (x.astype(np.float64) for x in (gpu, ref, old))
    err = np.abs(gpu - ref)
    bound = eps * np.maximum(np.abs(ref), np.abs(old) + lr)
    bad = err > bound
    assert not bad.any(), "%s: %d of %d row elements off; worst err/bound %.3g" % (
        what, int(bad.sum()), bad.size, float((err / bound).max()))


def assert_accum_close(gpu: np.ndarray, ref: np.ndarray, gabs: np.ndarray, eps: float = EPS32, what: str = ""):
    gpu, ref = gpu.astype(np.float64), ref.astype(np.float64)
    err = np.abs(gpu - ref)
    bound = eps * ref + 2 * eps * (gabs ** 2).mean(axis=1) + 1e-38
    bad = err > bound
    assert not bad.any(), "%s: %d of %d accumulators off; worst err/bound %.3g" % (
        what, int(bad.sum()), bad.size, float((err / bound).max()))


def as_f32(table_np: np.ndarray) -> np.ndarray:
    return wl.bf16_bits_to_f32(table_np) if table_np.dtype == np.uint16 else table_np


def random_case(rng, T: int, B: int, D: int, Rs: Sequence[int], max_len: int, dtype: str = "f32",
                empty_frac: float = 0.15, scale: float = 1.0, hot_row_frac: float = 0.0):
    """Random tables, lengths, rows; optionally a fraction of lookups hit row 0."""
    tables = []
    for R in Rs:
        v = (rng.standard_normal((R, D)) * scale).astype(np.float32)
        tables.append(wl.f32_to_bf16_bits(v).reshape(R, D) if dtype == "bf16" else v)
    lengths = rng.integers(0, max_len + 1, size=T * B).astype(np.int32)
    lengths[rng.random(T * B) < empty_frac] = 0
    off = np.concatenate([[0], np.cumsum(lengths.astype(np.int64))]).astype(np.int64)
    parts = []
    for t in range(T):
        n = int(lengths[t * B:(t + 1) * B].sum())
        r = rng.integers(0, Rs[t], size=n)
        if hot_row_frac > 0:
            r[rng.random(n) < hot_row_frac] = 0
        parts.append(r)
    rows = np.concatenate(parts).astype(np.int64) if parts else np.zeros(0, np.int64)
    return tables, lengths, off, rows


def make_tableset(tables_np: List[np.ndarray], dtype: str, with_accum: bool = False, salts=None,
                  accum_np: Optional[List[np.ndarray]] = None):
    w = [dev(t) for t in tables_np]
    if accum_np is not None:
        acc = [dev(a) for a in accum_np]
    else:
        acc = [torch.zeros(t.shape[0], dtype=torch.float32, device=DEV) for t in tables_np] if with_accum else None
    return emb.TableSet(w, tables_np[0].shape[1], dtype, accum=acc, salts=salts, device=torch.device(DEV)), w, acc


MANY_TABLES = 512   # added to a batch's tables: more than the routes for few lookups take, so it goes the general way


def add_empty_tables(extra: int, tables: List[np.ndarray], off: np.ndarray, dout: np.ndarray):
    """(tables, offsets, gradient) with `extra` tables of one row behind the others, without lookups."""
    if not extra:
        return tables, off, dout
    B, D = dout.shape[1:]
    return (tables + [np.zeros((1, D), dtype=tables[0].dtype)] * extra,
            np.concatenate([off, np.full(extra * B, off[-1], dtype=np.int64)]),
            np.concatenate([dout, np.zeros((extra, B, D), dtype=np.float32)]))


def gpu_forward(ts, rows_np, off_np, B, mode):
    out = torch.full((ts.T, B, ts.D), float("nan"), dtype=torch.float32, device=DEV)
    status = torch.zeros(1, dtype=torch.int32, device=DEV)
    emb.emb_bag_forward(ts, dev(rows_np), dev(off_np), B, mode, out, status)
    torch.cuda.synchronize()
    return out.cpu().numpy(), int(status.item())


_side = None


def side_stream():
    """One emb_side_stream for the whole test session."""
    global _side
    if _side is None:
        _side = emb.SideStream(torch.device(DEV))
    return _side


def gpu_backward(ts, rows_np, off_np, B, mode, dout_np, lr, eps, want_unique=True, side=True):
    """side=True: the long-run path runs on a second stream beside the short-run update."""
    nnz = rows_np.size
    ws = torch.empty(emb.emb_bag_backward_workspace_bytes(ts.T, B, nnz, ts.total_rows, ts.D, ts.dtype), dtype=torch.uint8, device=DEV)
    uk = torch.full((max(nnz, 1),), -7, dtype=torch.int64, device=DEV)
    uc = torch.full((max(nnz, 1),), -7, dtype=torch.int32, device=DEV)
    nu = torch.full((1,), -7, dtype=torch.int64, device=DEV)
    status = torch.zeros(1, dtype=torch.int32, device=DEV)
    emb.emb_bag_backward_rowwise_adagrad(ts, dev(rows_np), dev(off_np), B, mode, dev(dout_np), lr, eps, ws,
                                         uk if want_unique else None, uc if want_unique else None, nu, status,
                                         None, side_stream() if side else None)
    torch.cuda.synchronize()
    U = int(nu.item())
    return {"unique_keys": uk[:U].cpu().numpy(), "unique_counts": uc[:U].cpu().numpy(), "U": U,
            "status": int(status.item())}


def cache_select_large(freq: np.ndarray, num_hot: int, decay_shift: int = 0) -> np.ndarray:
    """The rule of ``cache_select`` evaluated with numpy's selection instead of a full sort, for tables of
    hundreds of millions of rows where the sorting definition takes minutes: the num_hot-th largest counter is
    the threshold; every row above it is kept, and of the rows equal to it the smallest row numbers, as many
    as still fit.  freq is aged in place.  Test-side arithmetic, not part of the oracle: the CPU tests pin it to ``oracle.cache_select`` (the sorting
    definition) on inputs with many ties and at the extremes of num_hot."""
    assert freq.dtype == np.uint32 and freq.flags["C_CONTIGUOUS"]
    R = freq.size
    assert 0 <= num_hot <= R and 0 <= decay_shift <= 31
    if num_hot == 0:
        hot = np.zeros(0, dtype=np.int64)
    else:
        thr = np.partition(freq, R - num_hot)[R - num_hot]           # the num_hot-th largest value
        above = np.flatnonzero(freq > thr)
        tied = np.flatnonzero(freq == thr)[:num_hot - above.size]      # flatnonzero is ascending
        hot = np.sort(np.concatenate([above, tied])).astype(np.int64)
    freq >>= np.uint32(decay_shift)
    return hot
