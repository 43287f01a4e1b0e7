"""The attention calls that a serving engine built on this library makes, as
cases that can be prepared, run, priced and checked one by one.

A case is a dict of plain values:

  kind       "step"     one decode step of a ``PagedBatch``: decode (+ reduce)
             "append"   the serving loop's iteration: the new token's K/V rows
                        appended and the step decoded in one launch (+ reduce)
             "noalloc"  ``paged_attn_decode_noalloc``
             "extend"   ``paged_attn_extend``: chunked prefill
  hq, hkv, d geometry
  batch      sequences, or ``requests`` of 1..5 sequences each (the retries of
             one request, consecutive in the batch)
  prefix     tokens that all sequences share as the same blocks
  mid        tokens that the retries of one request share after the prefix
  lo, hi     each sequence's own tokens after what it shares: spread evenly
             over [lo, hi], or lognormal (mean 1500, sigma 0.8) clipped to it
  chunk_lo, chunk_hi  extend: new tokens per sequence; they come after its own
             ``lo .. hi`` resident ones
  partition  split-KV partition size (0: one pass)
  prefix_partition  cascade: prefix partition size (0: no cascade, the shared
             blocks are read through every table)
  schedule   whether the per-sequence partitions come from a host work list

The lengths of a case are fixed; a seed draws their order, the placement of
the blocks in the pool and the values (N(0, 1) in bf16).
"""
import math
from statistics import NormalDist
from types import SimpleNamespace

import numpy as np
import torch

from paper_2510_14126_amd import binding
from paper_2510_14126_amd.device import PagedBatch

BLOCK = 16
DEVICE = "cuda:0"


def _case(name, kind, hq, hkv, d, **kw):
    c = dict(name=name, kind=kind, hq=hq, hkv=hkv, d=d, batch=0, requests=0, prefix=0, mid=0, lo=1, hi=1,
             lengths="even", chunk_lo=0, chunk_hi=0, partition=512, prefix_partition=0, schedule=False)
    c.update(kw)
    return c


def listed():
    return [
        # A small model's engine with a few calls in flight: launch-bound.
        _case("tiny_step", "step", 8, 2, 64, batch=4, lo=100, hi=300),
        # One call alone over a long context, in a loop that may not allocate.
        _case("single_long_noalloc", "noalloc", 64, 8, 128, batch=1, lo=30011, hi=30011),
        # SQL-generator stage: every call starts from one 2048-token schema
        # prompt; the cascade computes it once for the batch.
        _case("generator_step", "step", 32, 8, 128, batch=64, prefix=2048, lo=64, hi=512,
              prefix_partition=512, schedule=True),
        # The same batch in an engine that shares the prompt's blocks but does
        # not use the cascade, with the defaults of PagedBatch.
        _case("generator_no_cascade", "step", 32, 8, 128, batch=64, prefix=2048, lo=64, hi=512),
        # SQL-error-fixer stage: 32 requests of 1..5 retries that share the
        # schema and the failed first attempt; a decode iteration of the loop.
        _case("fixer_iteration", "append", 32, 8, 128, requests=32, prefix=2048, mid=256, lo=128, hi=1024,
              partition=1024, prefix_partition=1024, schedule=True),
        # One engine pool without stage isolation: mixed lengths, nothing shared.
        _case("shared_pool_step", "step", 32, 8, 128, batch=256, lo=64, hi=8192, lengths="lognormal",
              partition=8192, schedule=True),
        # Long-context stage, grouped-query 8, 512-token partitions.
        _case("long_context_step", "step", 64, 8, 128, batch=128, prefix=4096, lo=4096, hi=28672,
              prefix_partition=512, schedule=True),
        # One GPU's share of the long-context model under tensor parallelism
        # over its KV heads.
        _case("one_head_shard_step", "step", 8, 1, 128, batch=32, prefix=4096, lo=4096, hi=28672,
              prefix_partition=512, schedule=True),
        # head_dim 64 with eight query heads per KV head, ragged lengths, the
        # plain split-KV grid.
        _case("head64_step", "step", 32, 4, 64, batch=48, lo=61, hi=4093, partition=1024),
        # Prefill of one fixer request's retries as it arrives.
        _case("retry_prefill", "extend", 32, 8, 128, batch=3, prefix=2304, lo=0, hi=0, chunk_lo=128, chunk_hi=1024),
        # Prefill of the fixer stage's whole batch.
        _case("fixer_prefill", "extend", 32, 8, 128, requests=32, prefix=2048, mid=256, lo=0, hi=0,
              chunk_lo=128, chunk_hi=1024),
        # A long-context stage's first prompts, nothing resident yet.
        _case("prompt_prefill", "extend", 64, 8, 128, batch=2, lo=0, hi=0, chunk_lo=4001, chunk_hi=8191),
    ]


HEADS_128 = [(32, 8), (64, 8), (8, 1), (4, 1), (8, 2), (16, 2), (12, 3), (40, 5), (28, 7)]
HEADS_64 = [(8, 2), (32, 8), (32, 4), (64, 8), (24, 3), (4, 1)]


def _logint(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5)))))))


def draw(rng):
    while True:
        c = _draw_one(rng)
        w = work(c)
        if w["bytes"] <= 3e9 and w["flops"] <= (1.2e12 if c["kind"] == "extend" else 1e15):
            return c


def _draw_one(rng):
    what = rng.choice(["step", "step", "append", "noalloc", "cascade", "cascade", "groups", "extend", "extend"])
    d = 64 if what in ("step", "append", "noalloc") and rng.random() < 0.35 else 128
    hq, hkv = rng.choice(HEADS_64 if d == 64 else HEADS_128)
    hi = _logint(rng, 16, 32768)
    c = _case("", what, hq, hkv, d, batch=_logint(rng, 1, 256), hi=hi, lo=_logint(rng, 1, hi),
              partition=rng.choice([256, 512, 1024, 2048]), schedule=rng.random() < 0.5)
    del c["name"]
    if what in ("step", "append"):
        if c["hi"] <= 8192 and rng.random() < 0.3:
            c["partition"] = 0
        if rng.random() < 0.25:
            c["prefix"] = BLOCK * _logint(rng, 1, 256)
    elif what == "noalloc":
        c.update(batch=_logint(rng, 1, 16), schedule=False)
    elif what in ("cascade", "groups"):
        c.update(kind=rng.choice(["step", "append"]), prefix=BLOCK * _logint(rng, 4, 256),
                 prefix_partition=rng.choice([256, 512, 1024]))
        if what == "groups":
            c.update(batch=0, requests=_logint(rng, 1, 64), mid=BLOCK * _logint(rng, 1, 64))
    else:
        c["prefix"] = BLOCK * rng.randint(0, 256)
        own = 8192 - c["prefix"]
        c["chunk_hi"] = _logint(rng, 1, own)
        c["chunk_lo"] = _logint(rng, 1, c["chunk_hi"])
        c["hi"] = rng.choice([0, _logint(rng, 1, max(1, own - c["chunk_hi"]))]) if own > c["chunk_hi"] else 0
        c.update(lo=min(c["hi"], rng.choice([0, c["hi"]])), batch=_logint(rng, 1, 128), schedule=False)
    return c


# --------------------------------------------------------------------------
# lengths and work
# --------------------------------------------------------------------------

def _spread(n, lo, hi, how):
    u = [(i + 0.5) / n for i in range(n)]
    if how == "lognormal":
        mu = math.log(1500.0) - 0.8 * 0.8 / 2
        x = [math.exp(mu + 0.8 * NormalDist().inv_cdf(v)) for v in u]
    else:
        x = [lo + v * (hi - lo) for v in u]
    return np.array([min(hi, max(lo, round(v))) for v in x], dtype=np.int64)


def _sizes(c):
    """Sequences of each request (requests), or one request per sequence."""
    return [1 + i % 5 for i in range(c["requests"])] if c["requests"] else [1] * c["batch"]


def _lengths(c):
    """(own resident tokens, new tokens of the chunk) per sequence, sorted."""
    n = sum(_sizes(c))
    own = _spread(n, c["lo"], c["hi"], c["lengths"])
    chunk = _spread(n, c["chunk_lo"], c["chunk_hi"], "even") if c["kind"] == "extend" else np.zeros(n, np.int64)
    return own, chunk


def work(c):
    own, chunk = _lengths(c)
    n = len(own)
    shared = c["prefix"] + c["mid"]
    tokens = c["prefix"] + c["mid"] * len(_sizes(c)) + int(own.sum() + chunk.sum())
    rows = int(chunk.sum()) if c["kind"] == "extend" else n
    nbytes = tokens * 2 * c["hkv"] * c["d"] * 2 + 2 * rows * c["hq"] * c["d"] * 2
    ctx = shared + own + chunk
    nbytes += int(((ctx + BLOCK - 1) // BLOCK).sum()) * 4 + 4 * n
    if c["kind"] == "append":
        nbytes += 2 * 2 * n * c["hkv"] * c["d"] * 2
    if c["kind"] == "extend":
        visible = float((chunk * (shared + own.mean())).sum() + (chunk * (chunk + 1) / 2).sum())
    else:
        visible = float(ctx.sum())
    return {"bytes": int(nbytes), "flops": int(4 * c["hq"] * c["d"] * visible)}


def tolerance(c):
    # bf16 outputs: rounding alone is 1.7e-3 of the result (2-norm) and half a
    # unit in the last place, 2^-8 of a value, at most; four times that.
    return {"rel": 7e-3, "max": 1.6e-2}


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

def _structure(c, seed):
    """Lengths in the seed's order, and the block tables over a shuffled pool
    1.2 times as large as needed."""
    rng = np.random.default_rng(seed)
    own, chunk = _lengths(c)
    own, chunk = rng.permutation(own), rng.permutation(chunk)
    sizes = rng.permutation(np.array(_sizes(c)))
    ctx = c["prefix"] + c["mid"] + own + chunk
    n_pre, n_mid = c["prefix"] // BLOCK, c["mid"] // BLOCK
    tail = (own + chunk + BLOCK - 1) // BLOCK
    needed = n_pre + n_mid * len(sizes) + int(tail.sum())
    num_blocks = math.ceil(1.2 * needed)
    perm = rng.permutation(num_blocks).astype(np.int32)
    at = n_pre
    tables = np.full((len(ctx), n_pre + n_mid + max(1, int(tail.max()))), -1, dtype=np.int32)
    b = 0
    for size in sizes:
        mid = perm[at: at + n_mid]
        at += n_mid
        for _ in range(size):
            tables[b, :n_pre] = perm[:n_pre]
            tables[b, n_pre: n_pre + n_mid] = mid
            tables[b, n_pre + n_mid: n_pre + n_mid + tail[b]] = perm[at: at + tail[b]]
            at += int(tail[b])
            b += 1
    starts = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    return SimpleNamespace(ctx=ctx.astype(np.int32), chunk=chunk.astype(np.int32), tables=tables,
                           num_blocks=num_blocks, starts=starts)


def _values(c, s, seed):
    gen = torch.Generator(device=DEVICE).manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=gen, dtype=torch.bfloat16, device=DEVICE)

    pool = (s.num_blocks, c["hkv"], BLOCK, c["d"])
    rows = int(s.chunk.sum()) if c["kind"] == "extend" else len(s.ctx)
    k, v, q = normal(*pool), normal(*pool), normal(rows, c["hq"], c["d"])
    new = [normal(len(s.ctx), c["hkv"], c["d"]) for _ in range(2)] if c["kind"] == "append" else []
    return k, v, q, new


def prepare(c, seed):
    s = _structure(c, seed)
    k, v, q, new = _values(c, s, seed)
    state = {"kind": c["kind"], "new": new}
    if c["kind"] == "extend":
        state.update(pool=binding.kv_pool_create(s.num_blocks, BLOCK, c["hkv"], c["d"], k, v), q=q,
                     q_start=torch.from_numpy(np.concatenate([[0], np.cumsum(s.chunk)]).astype(np.int32)).to(DEVICE),
                     total=int(s.chunk.sum()), tables=torch.from_numpy(s.tables).to(DEVICE),
                     stride=s.tables.shape[1], ctx=torch.from_numpy(s.ctx).to(DEVICE), batch=len(s.ctx), hq=c["hq"],
                     scale=1.0 / math.sqrt(c["d"]), max_ctx=int(s.ctx.max()), max_chunk=int(s.chunk.max()),
                     out=torch.zeros_like(q))
        return state
    w = SimpleNamespace(batch=len(s.ctx), num_q_heads=c["hq"], num_kv_heads=c["hkv"], head_dim=c["d"],
                        num_blocks=s.num_blocks, context_lens=s.ctx, block_tables=s.tables,
                        scale=1.0 / math.sqrt(c["d"]), partition_size=c["partition"],
                        max_context_len=int(s.ctx.max()), q=q.view(torch.int16).cpu().numpy().view(np.uint16))
    kw = {}
    if c["prefix_partition"]:
        kw.update(prefix_len=c["prefix"], prefix_partition_size=c["prefix_partition"])
        if c["mid"]:
            kw.update(group_start=s.starts, group_len=c["mid"])
    batch = PagedBatch(w, DEVICE, k_pool=k, v_pool=v, schedule=c["schedule"], **kw)
    state.update(batch=batch, out=batch.out.view(torch.bfloat16), k=k, v=v)
    return state


def run(state):
    kind = state["kind"]
    if kind == "extend":
        x = state
        binding.paged_attn_extend(x["pool"], x["q"], x["q_start"], x["total"], x["tables"], x["stride"], x["ctx"],
                                  x["batch"], x["hq"], x["scale"], x["max_ctx"], x["max_chunk"], x["out"])
        return {"out": x["out"]}
    b = state["batch"]
    if kind == "step":
        b.run()
    elif kind == "append":
        b.decode_append(*state["new"])
        if b.needs_reduce:
            b.reduce()
        return {"out": state["out"], "k": state["k"], "v": state["v"]}
    else:
        binding.paged_attn_decode_noalloc(b.pool, b.q, b.bt, b.bt_stride, b.ctx, b.batch, b.hq, b.w.scale,
                                          b.max_ctx, b.partition_size, b.out)
    return {"out": state["out"]}


# --------------------------------------------------------------------------
# the same in 64 bits
# --------------------------------------------------------------------------

def exact(c, seed):
    s = _structure(c, seed)
    k, v, q, new = _values(c, s, seed)
    hq, hkv, d = c["hq"], c["hkv"], c["d"]
    group, scale = hq // hkv, 1.0 / math.sqrt(d)
    if new:
        last = s.ctx.astype(np.int64) - 1
        block = torch.from_numpy(s.tables[np.arange(len(last)), last // BLOCK].astype(np.int64)).to(DEVICE)
        row = torch.from_numpy(last % BLOCK).to(DEVICE)
        k[block, :, row] = new[0]
        v[block, :, row] = new[1]
    out = torch.empty(q.shape, dtype=torch.float64, device=DEVICE)
    at = 0
    for b, n in enumerate(s.ctx.tolist()):
        ids = torch.from_numpy(s.tables[b, : (n + BLOCK - 1) // BLOCK].astype(np.int64)).to(DEVICE)
        rows = int(s.chunk[b]) if c["kind"] == "extend" else 1
        qb = q[at: at + rows].double().reshape(rows, hkv, group, d)
        seen = torch.arange(n, device=DEVICE)[None, :] <= torch.arange(n - rows, n, device=DEVICE)[:, None]
        for g in range(hkv):
            kg = k[ids, g].reshape(-1, d)[:n].double()
            vg = v[ids, g].reshape(-1, d)[:n].double()
            for lo in range(0, rows, 1024):
                qg = qb[lo: lo + 1024, g].reshape(-1, d)
                x = (qg @ kg.t() * scale).reshape(-1, group, n)
                x = torch.softmax(x.masked_fill(~seen[lo: lo + 1024, None, :], -math.inf), dim=-1)
                out[at + lo: at + min(rows, lo + 1024), g * group: (g + 1) * group] = \
                    (x.reshape(-1, n) @ vg).reshape(-1, group, d)
        at += rows
    return {"out": out, "k": k, "v": v} if new else {"out": out}
