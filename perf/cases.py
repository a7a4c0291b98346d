"""The calls that a user of this package makes, with the sizes they are made at.

A case names one pass through the public entry points: a pooled lookup over row numbers, a serving lookup from raw
IDs and bag lengths, a training step (lookup, sparse backward, row-wise Adagrad), a lookup over hosted tables with an
HBM cache, a lookup over tables of different width, or one round of the cache policy.  Sizes are those of the
package's own workloads (``workloads.WORKLOADS``) or of its tests, and ``draw`` spreads over the same ranges.
"""
import functools
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2508_05700_amd import binding as emb
from paper_2508_05700_amd import pipeline
from paper_2508_05700_amd import workloads as wl

MIX = "16:f32:2000000*6,32:bf16:5000000*6,64:f32:10000000*8,128:f32:2000000*4"


def _case(**kw):
    c = dict(kind="serve", T=16, R=10_000_000, D=64, dtype="f32", B=8192, length="poisson", mean_len=20, max_len=100,
             ids="zipf", alpha=1.05, n_keys=10 ** 9, pool="mean")
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one table, IDs that are row numbers already, 512 bags of 8 (latency and launches)
        _case(name="rows_small", T=1, R=100_000, D=32, B=512, length="fixed", mean_len=8, max_len=0, ids="rows",
              alpha=0.0, n_keys=0, pool="sum"),
        # one ranking request: sixteen ID features, a handful of candidates
        _case(name="serve_request", R=1_000_000, B=16, n_keys=10 ** 8),
        # a serving batch over sixteen large tables, IDs with popular heads
        _case(name="serve_zipf"),
        # the same with IDs that hardly repeat: every row comes from HBM; the caller gives the streaming hint
        _case(name="serve_uniform", ids="uniform", alpha=0.0, n_keys=0, streaming=True),
        # the same batch over tables stored as INT4 rows
        _case(name="serve_int4", dtype="int4"),
        # one very large bf16 table, long bags, strong skew
        _case(name="serve_bf16", T=1, R=1_000_000_000, D=32, dtype="bf16", B=65536, mean_len=50, max_len=0, alpha=1.2,
              n_keys=10 ** 12, pool="sum"),
        # a training step of a small model, or of one small micro-batch
        _case(name="train_small", kind="train", T=3, R=200_000, B=512, n_keys=10 ** 7),
        # a training step of odd sizes over bf16 rows whose width is no power of two, distinct rows listed
        _case(name="train_ragged", kind="train", T=7, R=1_000_003, D=48, dtype="bf16", B=1931, mean_len=11, n_keys=10 ** 8,
              pool="sum", unique=True),
        # the training step at full size: fine-tuning sixteen large tables
        _case(name="train_zipf", kind="train"),
        # a table in pinned host memory behind an HBM cache of its 5 % hottest rows: misses cross the link
        _case(name="hosted", kind="hosted", T=1, R=4_000_000, B=16384, mean_len=30, max_len=0, alpha=1.1,
              n_keys=16_000_000, pool="sum", hot=0.05),
        # 24 tables of four widths and two storage types, one concatenated vector per sample
        _case(name="mix", kind="mix", T=24, R=0, D=0, dtype="", tables=MIX),
        # one round of the cache policy of a hosted INT4 table: watch a million lookups, choose the rows, refill
        _case(name="refresh", kind="refresh", T=1, R=20_000_000, dtype="int4", B=0, mean_len=0, max_len=0, alpha=1.1,
              n_keys=80_000_000, pool="", hot=0.05, watched=1_000_000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _row_bytes(D, dtype):
    return {"f32": 4 * D, "bf16": 2 * D, "int8": (8 + D + 15) // 16 * 16, "int4": (8 + D // 2 + 15) // 16 * 16}[dtype]


def _dim(rng, dtype):
    # common widths, and in one case of three any width the storage type allows
    if rng.random() < 0.67:
        return rng.choice([16, 32, 64, 128])
    step = {"f32": 4, "bf16": 8}.get(dtype, 16)
    return step * rng.randint(max(1, 16 // step), 192 // step)


def draw(rng):
    kind = rng.choice(["serve", "serve", "serve", "train", "train", "train", "hosted", "mix", "refresh"])
    alpha = round(rng.uniform(1.02, 1.25), 3)
    mean_len = _log(rng, 1, 60)
    pool = rng.choice(["sum", "mean"])
    if kind == "refresh":
        dtype = rng.choice(["f32", "int4"])
        D = rng.choice([16, 32, 64, 128])
        R = _log(rng, 100_000, min(20_000_000, 960_000_000 // _row_bytes(D, dtype)))
        return _case(kind=kind, T=1, R=R, D=D, dtype=dtype, B=0, mean_len=0, max_len=0, alpha=alpha, n_keys=4 * R, pool="",
                     hot=round(rng.uniform(0.01, 0.08), 3), watched=_log(rng, 10_000, 1_000_000))
    if kind == "hosted":
        dtype = rng.choice(["f32", "int4"])
        D = rng.choice([16, 32, 64, 128])
        T = rng.randint(1, 4)
        R = _log(rng, 50_000, 960_000_000 // _row_bytes(D, dtype) // T)
        lookups = 490_000 * 256 // max(_row_bytes(D, dtype), 256)
        B = _log(rng, 16, min(16384, lookups // mean_len) // T)
        return _case(kind=kind, T=T, R=R, D=D, dtype=dtype, B=B, mean_len=mean_len, max_len=0, alpha=alpha, n_keys=4 * R,
                     pool=pool, hot=round(rng.uniform(0.02, 0.1), 3))
    if kind == "mix":
        groups = []
        T, lookups = 0, 0
        for D in rng.sample([16, 32, 64, 128], rng.randint(2, 4)):
            n = rng.randint(1, 6)
            groups.append("%d:%s:%d*%d" % (D, rng.choice(["f32", "bf16"]), _log(rng, 10_000, 10_000_000 * 64 // max(D, 64)), n))
            T += n
            lookups += n * max(D, 64)
        B = _log(rng, 8, min(8192, 20 * 8192 * 1600 // lookups // mean_len))
        return _case(kind=kind, T=T, R=0, D=0, dtype="", B=B, mean_len=mean_len, alpha=alpha, pool=pool, tables=",".join(groups))
    train = kind == "train"
    dtype = rng.choice(["f32", "f32", "bf16"] if train else ["f32", "f32", "bf16", "int8", "int4"])
    D = _dim(rng, dtype)
    T = _log(rng, 1, 24)
    R = _log(rng, 10_000, min(10_000_000, 10_240_000_000 // (T * max(D, 64))))
    ids = rng.choice(["zipf", "zipf", "zipf", "uniform", "rows"])
    most = 2_600_000 * 64 // max(D, 64) // T // mean_len     # bags per table at the cost of the largest listed case
    B = _log(rng, 4, min(65536, most))
    c = _case(kind=kind, T=T, R=R, D=D, dtype=dtype, B=B, length=rng.choice(["poisson", "poisson", "poisson", "fixed"]),
              mean_len=mean_len, ids=ids, alpha=alpha if ids == "zipf" else 0.0, n_keys=100 * R if ids == "zipf" else 0, pool=pool)
    if train:
        c["unique"] = rng.random() < 0.3
    else:
        c["streaming"] = ids == "uniform" and rng.random() < 0.5
    return c


# ---------------------------------------------------------------------------
# inputs, made on the GPU
# ---------------------------------------------------------------------------
def _signed(v):
    v %= 1 << 64
    return v - (1 << 64) if v >= 1 << 63 else v


def _fmix64(z):
    """workloads.fmix64 on int64 tensors (logical shifts, wrapping products)."""
    for mul in (int(wl._FMIX_C1), int(wl._FMIX_C2)):
        z = (z ^ ((z >> 33) & 0x7FFFFFFF)) * _signed(mul)
    return z ^ ((z >> 33) & 0x7FFFFFFF)


@functools.lru_cache(maxsize=4)
def _zipf(n_keys, alpha):
    z = wl.BoundedZipf(n_keys, alpha)
    return z, torch.from_numpy(z.cum).cuda()


def _zipf_raw(n_keys, alpha, n, gen, key):
    """n raw 64-bit IDs whose popularity ranks follow the bounded Zipf law (workloads.BoundedZipf)."""
    z, cum = _zipf(n_keys, alpha)
    u = torch.rand(n, generator=gen, device="cuda", dtype=torch.float64) * z.H
    ranks = torch.searchsorted(cum, u, right=True) + 1
    if z.tail_mass > 0.0:
        a1 = z.a - 1.0
        x = (z.lo_pow - a1 * (u - z.head_mass)).clamp_(min=1e-300) ** (-1.0 / a1)
        ranks = torch.where(u < z.head_mass, ranks, x.round().clamp_(z.M + 1, z.N).to(torch.int64))
    return _fmix64(ranks.clamp_(1, z.N) + _signed(key))


def _lengths(c, gen):
    n = c["T"] * c["B"]
    if c["length"] == "fixed":
        return torch.full((n,), c["mean_len"], dtype=torch.int32, device="cuda")
    L = torch.poisson(torch.full((n,), float(c["mean_len"]), device="cuda"), generator=gen)
    if c["max_len"]:
        L.clamp_(max=c["max_len"])
    return L.to(torch.int32)


def _raw_ids(c, per_table, gen, seed):
    """Raw IDs, table after table; every ID feature has its own popular IDs."""
    parts = []
    for t, n in enumerate(per_table):
        if c["ids"] == "zipf":
            parts.append(_zipf_raw(c["n_keys"], c["alpha"], n, gen, wl._stream_key(seed, t)))
        else:
            parts.append(torch.randint(-1 << 63, (1 << 63) - 1, (n,), generator=gen, device="cuda"))
    return torch.cat(parts)


def _batch(c, gen, seed):
    lengths = _lengths(c, gen)
    per_table = lengths.view(c["T"], c["B"]).sum(1).tolist()
    b = SimpleNamespace(lengths=lengths, nnz=sum(per_table), raw=None, rows_given=None, dout=None)
    if c["ids"] == "rows":
        b.rows_given = torch.randint(0, c["R"], (b.nnz,), generator=gen, device="cuda")
    else:
        b.raw = _raw_ids(c, per_table, gen, seed)
    return b


def _capacity(c):
    """Lookups that a batch's buffers are made for: no batch of these lengths exceeds it in practice."""
    n = c["T"] * c["B"] * c["mean_len"]
    return int(n + 10 * math.sqrt(n)) + 64


def _workload(c):
    quant = c["dtype"] if c["dtype"] in emb.QUANT_DTYPES else None
    return wl.Workload(c.get("name", "case"), T=c["T"], R=c["R"], D=c["D"], dtype="f32" if quant else c["dtype"], B=c["B"],
                       length=c["length"], mean_len=c["mean_len"], max_len=c["max_len"] or None, ids=c["ids"],
                       pool=c["pool"], backward=c["kind"] == "train", quant=quant, streaming=c.get("streaming", False))


def _host_table(R, D, dtype, seed):
    """A table in pinned host memory, filled from the device; (tensor, device pointer)."""
    width = emb.emb_row_bytes(D, dtype)
    host = torch.empty((R, width), dtype=torch.uint8, pin_memory=True)
    ptr = emb.emb_host_device_pointer(int(host.data_ptr()))
    if dtype == "f32":
        emb.emb_table_fill(ptr, R, D, dtype, seed)
    else:
        full = torch.empty((R, D), dtype=torch.float32, device="cuda")
        emb.emb_table_fill(full, R, D, "f32", seed)
        emb.emb_quantize_rows(full, dtype, ptr)
    return host, ptr


def _hosted_cache(c, t, seed):
    host, ptr = _host_table(c["R"], c["D"], c["dtype"], 1000 * seed + t)
    cache = pipeline.HotRowCache(ptr, c["R"], c["D"], c["dtype"], max(1, int(c["hot"] * c["R"])), t, torch.device("cuda"))
    return host, cache


def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dev = torch.device("cuda")
    s = SimpleNamespace(case=c)
    if c["kind"] in ("serve", "train"):
        w = s.w = _workload(c)
        s.tables = pipeline.DeviceTables(w, seed, "cuda")
        s.batch = _batch(c, gen, seed)
        s.buf = pipeline.StepBuffers(w, _capacity(c), s.tables.set.total_rows, dev, want_unique=c.get("unique", False))
        if w.backward:
            s.batch.dout = torch.randn((w.T, w.B, w.D), generator=gen, device="cuda")
            if c.get("unique"):
                s.buf.unique_keys.zero_()
                s.buf.unique_counts.zero_()
    elif c["kind"] == "mix":
        shapes = []
        for part in c["tables"].split(","):
            D, dtype, rest = part.split(":")
            R, n = rest.split("*")
            shapes += [(int(D), dtype, int(R))] * int(n)
        weights = []
        for t, (D, dtype, R) in enumerate(shapes):
            weights.append(torch.empty((R, D), dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device="cuda"))
            emb.emb_table_fill(weights[t], R, D, dtype, 1000 * seed + t)
        s.tables = emb.MixedTables(weights, c["B"], "concat", device=dev)
        s.batch = _batch(c, gen, seed)
        s.offsets = torch.empty(c["T"] * c["B"] + 1, dtype=torch.int64, device="cuda")
        s.rows = torch.zeros(_capacity(c), dtype=torch.int64, device="cuda")
        s.out = torch.empty((c["B"], sum(s.tables.Ds)), dtype=torch.float32, device="cuda")
        s.status = torch.zeros(1, dtype=torch.int32, device="cuda")
    elif c["kind"] == "hosted":
        made = [_hosted_cache(c, t, seed) for t in range(c["T"])]
        s.hosts = [h for h, _ in made]
        for t, (_, cache) in enumerate(made):      # the rows of the most popular IDs
            ranks = torch.arange(1, cache.capacity + 1, device="cuda")
            rows = torch.empty_like(ranks)
            emb.emb_hash_ids(_fmix64(ranks + _signed(wl._stream_key(seed, t))), t, c["R"], rows)
            cache.set_static(torch.unique(rows))
        s.set = pipeline.HostedTableSet([cache for _, cache in made], dev)
        s.batch = _batch(c, gen, seed)
        n = c["T"] * c["B"]
        s.offsets = torch.empty(n + 1, dtype=torch.int64, device="cuda")
        s.scratch = torch.empty(emb.emb_offsets_scratch_bytes(n), dtype=torch.uint8, device="cuda")
        s.out = torch.empty((c["T"], c["B"], c["D"]), dtype=torch.float32, device="cuda")
    else:
        # a policy that has been running: the cache holds what earlier traffic chose
        s.host, s.cache = _hosted_cache(c, 0, seed)
        key = wl._stream_key(seed, 0)
        s.traffic = [_zipf_raw(c["n_keys"], c["alpha"], c["watched"], gen, key) for _ in range(4)]
        s.at = 0
        for raw in s.traffic[1:]:
            s.cache.observe(raw)
        s.cache.refresh()
    return s


def run(state):
    s, c = state, state.case
    if c["kind"] in ("serve", "train"):
        pipeline.run_step(s.w, s.tables.set, s.batch, s.buf)
        out = [s.buf.out, s.buf.offsets]
        if c["kind"] == "train":
            out += [s.tables.weights, s.tables.accum, s.buf.num_unique, s.buf.unique_keys, s.buf.unique_counts]
        return out
    if c["kind"] == "mix":
        rows = s.rows[:s.batch.nnz]
        emb.emb_lengths_to_offsets(s.batch.lengths, s.offsets, s.status)
        emb.emb_hash_ids_tables(s.tables.tables, s.batch.raw, s.offsets, c["B"], rows, s.status)
        emb.emb_bag_forward_mixed(s.tables, rows, s.offsets, c["pool"], s.out, s.status)
        return [s.out, s.offsets, s.rows]
    if c["kind"] == "hosted":
        h = s.set
        if c["T"] == 1:
            k = h.caches[0]
            emb.emb_bag_forward_cached_hashed_lengths(k.table_ptr, k.R, k.D, k.dtype, k.rows[k.active], k.index[k.active],
                                                      k.num_hot, k.salt, s.batch.raw, s.batch.lengths, c["B"], c["pool"],
                                                      s.out, s.offsets, s.scratch, h.hit_miss, h.status)
        else:
            emb.emb_bag_forward_cached_tables_hashed_lengths(h.tables, s.batch.raw, s.batch.lengths, c["B"], c["pool"],
                                                             s.out, s.offsets, s.scratch, h.hit_miss, h.status)
        return [s.out, s.offsets, h.hit_miss]
    k = s.cache
    k.observe(s.traffic[s.at])
    s.at = (s.at + 1) % len(s.traffic)
    k.refresh()
    return [k.hot, k.rows[k.active], k.index[k.active], k.freq, k.info, k.moved]


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _distinct(c, n, R):
    """Expected number of distinct rows among n lookups of a table of R rows."""
    keys = float(n)
    if c["ids"] == "zipf":
        a = c["alpha"]
        edges = np.unique(np.concatenate([np.arange(1.0, 2049.0), np.geomspace(2048.0, c["n_keys"] + 1.0, 4096)]))
        width = np.diff(edges)
        mass = (edges[:-1] ** (1 - a) - edges[1:] ** (1 - a)) / (a - 1)   # integral of k**-a over the bin
        mass[edges[:-1] < 2048] = edges[:-1][edges[:-1] < 2048] ** -a     # single ranks
        mass /= mass.sum()
        keys = float((width * -np.expm1(-n * mass / width)).sum())
    return -R * math.expm1(-keys / R)


def work(case):
    c = case
    if c["kind"] == "refresh":
        hot = c["hot"] * c["R"]
        fresh = min(_distinct(c, c["watched"], c["R"]), hot)
        # IDs, the counters read and aged, the chosen rows written, the cache and its index written, its rows read
        return {"bytes": 8.0 * c["watched"] + 8.0 * c["R"] + 8.0 * hot + hot * _row_bytes(c["D"], c["dtype"]) + c["R"] / 4.0
                + fresh * _row_bytes(c["D"], c["dtype"]), "flops": 0.0}
    if c["kind"] == "mix":
        shapes = []
        for part in c["tables"].split(","):
            D, dtype, rest = part.split(":")
            R, n = rest.split("*")
            shapes += [(int(D), dtype, int(R))] * int(n)
    else:
        shapes = [(c["D"], c["dtype"], c["R"])] * c["T"]
    n = c["B"] * c["mean_len"]
    total = 4.0 * c["T"] * c["B"] + 8.0 * (c["T"] * c["B"] + 1)       # lengths in, offsets out
    flops = 0.0
    for D, dtype, R in shapes:
        d, rb = _distinct(c, n, R), _row_bytes(D, dtype)
        total += 8.0 * n + d * rb + 4.0 * D * c["B"]                  # IDs, rows, pooled output
        flops += n * D
        if c["kind"] == "train":
            total += 4.0 * D * c["B"] + d * (rb + 8.0)                # gradient, rows written, accumulators
            flops += 2.0 * n * D + 6.0 * d * D
        if c["kind"] == "mix":
            total += 8.0 * n                                          # row numbers, an output of this route
    return {"bytes": total, "flops": flops}


def tolerance(case):
    if case["kind"] == "refresh":
        return "exact"
    if case["kind"] == "train" and case["dtype"] == "bf16":
        return {"rel": 1e-3, "max": 2e-2}      # a stored row may round to the neighbouring bf16 value
    return {"rel": 1e-5}
