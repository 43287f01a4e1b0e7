"""The matrix-core decode at the edges of its tiles, for every geometry it
takes (head_dim 64 and 128, four and eight query heads per KV head) and for
negative and zero scales: contexts of 0 and 1 tokens, around one block, around
one round of the four wavefronts, around the 64 block ids read at a time, and
an item's masked last block on each wavefront.  Poison past every context;
outputs against the oracle under the parity gate."""
from dataclasses import replace

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import compare, decode_workload  # noqa: E402
from workloads import duplicate_shared_blocks, f32_to_bf16_bits, logical_case, page_case  # noqa: E402

CTX = [0, 1, 15, 16, 17, 33, 48, 63, 64, 65, 81, 127, 1009, 1023, 1024, 1025, 1041, 2064, 2100]


@pytest.mark.parametrize("scale", [None, -0.2, 0.0])
@pytest.mark.parametrize("S", [0, 64, 1040])
@pytest.mark.parametrize("d,hq,hkv", [(64, 8, 2), (64, 24, 3), (128, 12, 3), (128, 8, 1)])
def test_tile_edges(d, hq, hkv, S, scale):
    from paper_2510_14126_amd.device import PagedBatch
    print(f"[gpu case] tile edges D={d} Hq={hq} Hkv={hkv} S={S} scale={scale}", flush=True)
    w = page_case(logical_case(400 + d + hq, len(CTX), hq, hkv, d, CTX, scale=scale), 401, poison=True)
    ref = decode_workload(w)[0]
    outs = []
    for shared in (False, True):           # both cache policies (and ring depths)
        pb = PagedBatch(w, "cuda:0", partition_size=S)
        if shared:
            from paper_2510_14126_amd import binding
            binding.kv_pool_retain(pb.pool, [int(w.block_tables[-1, 0])])
        pb.out.fill_(0x7FC0)               # NaN bits: every row must be written
        pb.run()
        torch.cuda.synchronize()
        outs.append(pb.out_bits())
        pb.close()
    rep = compare(outs[0], ref)
    assert rep.passed, f"{rep}"
    assert np.array_equal(outs[0], outs[1])


@pytest.mark.parametrize("d,hq,hkv", [(64, 8, 2), (64, 24, 3), (128, 12, 3), (128, 8, 1)])
def test_fused_append_in_every_row(d, hq, hkv):
    """The appended token in each row of a block, as the last row of a whole
    block and as the first of a new one, and past 64 blocks."""
    from oracle import append_kv
    from paper_2510_14126_amd.device import PagedBatch
    ctx = list(range(1, 18)) + [64, 65, 1024, 1025, 1040]
    print(f"[gpu case] fused append D={d} Hq={hq} Hkv={hkv}", flush=True)
    w = page_case(logical_case(420 + d + hq, len(ctx), hq, hkv, d, ctx), 421, poison=True)
    rng = np.random.default_rng(422)
    new = [f32_to_bf16_bits(rng.standard_normal((len(ctx), hkv, d), dtype=np.float32)) for _ in range(2)]
    for b, n in enumerate(ctx):            # what the slot holds beforehand is never used
        w.k_pool[w.block_tables[b, (n - 1) // 16], :, (n - 1) % 16] = 0x7FC0
        w.v_pool[w.block_tables[b, (n - 1) // 16], :, (n - 1) % 16] = 0x7FC0
    for S in (0, 512):
        pb = PagedBatch(w, "cuda:0", partition_size=S)
        pb.decode_append(*(torch.from_numpy(x.view(np.int16)).cuda() for x in new))
        if pb.needs_reduce:
            pb.reduce()
        torch.cuda.synchronize()
        out, k, v = pb.out_bits(), pb.k.cpu().numpy().view(np.uint16), pb.v.cpu().numpy().view(np.uint16)
        pb.close()
        wk, wv = append_kv(w.k_pool, w.v_pool, w.block_tables, w.context_lens, new[0], new[1])
        assert np.array_equal(k, wk) and np.array_equal(v, wv)
        rep = compare(out, decode_workload(replace(w, k_pool=wk, v_pool=wv))[0])
        assert rep.passed, f"S={S}: {rep}"


def wide_batch(hkv, group, n, shared, lens, spare=0):
    """len(lens) sequences of up to n blocks over a shuffled pool, the first `shared`
    blocks in every table (and `spare` blocks in none), as a workload and its
    device pools."""
    from types import SimpleNamespace
    d, batch = 128, len(lens)
    nb = shared + batch * (n - shared) + spare
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    k, v = (torch.randn((nb, hkv, 16, d), generator=gen, dtype=torch.bfloat16, device="cuda:0") for _ in range(2))
    perm = np.random.default_rng(6).permutation(nb).astype(np.int32)
    tables = np.empty((batch, n), np.int32)
    tables[:, :shared] = perm[:shared]
    tables[:, shared:] = perm[shared: shared + batch * (n - shared)].reshape(batch, -1)
    hq = group * hkv
    w = SimpleNamespace(batch=batch, num_q_heads=hq, num_kv_heads=hkv, head_dim=d, num_blocks=nb, block_size=16,
                        context_lens=np.asarray(lens, np.int32), block_tables=tables, scale=d ** -0.5,
                        partition_size=512, max_context_len=16 * n,
                        q=f32_to_bf16_bits(np.random.default_rng(7).standard_normal((batch, hq, d), dtype=np.float32)))
    return w, k, v


def test_sharing_changes_the_cache_policy_and_no_bit():
    """The plain decode streams its tiles while the pool holds no shared block
    and loads them with the default policy from the first one on (which also
    lets neighbours share a workgroup): both give the same bits, and what the
    oracle gives."""
    from paper_2510_14126_amd import binding
    from paper_2510_14126_amd.device import PagedBatch
    print("[gpu case] cache policy: no block known as shared, then ten", flush=True)
    n = 1050
    w, k, v = wide_batch(8, 4, n, 10, [16 * n, 16 * n - 5, 9000, 33])
    pb = PagedBatch(w, "cuda:0", k_pool=k, v_pool=v, register_blocks=False)
    assert binding.kv_pool_num_shared(pb.pool) == 0
    pb.run()
    torch.cuda.synchronize()
    streamed = pb.out_bits().copy()
    w.k_pool, w.v_pool = (x.view(torch.int16).cpu().numpy().view(np.uint16) for x in (k, v))
    assert compare(streamed, decode_workload(w)[0]).passed
    pb.register_placement()
    assert binding.kv_pool_num_shared(pb.pool) == 10
    pb.out.fill_(0x7FC0)
    pb.run()
    torch.cuda.synchronize()
    assert np.array_equal(streamed, pb.out_bits())
    pb.close()


@pytest.mark.parametrize("schedule", [False, True])
@pytest.mark.parametrize("group", [4, 8])
def test_other_sequences_in_the_pool_do_not_slow_a_shared_batch(group, schedule):
    """64 sequences over a shared 2048-token prefix, in a pool that holds nothing
    else and in one whose references are otherwise to private blocks (1.1 GB of
    them).  The call reads the same tiles either way, so it takes the same time
    (runs differ by 1%); with streaming loads, which the many private references
    once switched on, each shared tile left the caches between its readers and
    the step took 1.3 (eight heads) to 1.65 times as long."""
    from paper_2510_14126_amd import binding
    from paper_2510_14126_amd.device import PagedBatch
    print(f"[gpu case] shared batch in a mostly private pool, group {group}, work list {schedule}", flush=True)
    shared, n, spare = 128, 160, 17000
    w, k, v = wide_batch(8, group, n, shared, np.linspace(2112, 2560, 64).round(), spare)
    us = []
    for private in (False, True):
        pb = PagedBatch(w, "cuda:0", k_pool=k, v_pool=v, schedule=schedule)
        if private:
            binding.kv_pool_claim(pb.pool, [i for i in range(w.num_blocks)
                                            if binding.kv_pool_refcount(pb.pool, i) == 0])
        us.append(median_us(pb.run))
        pb.close()
    assert us[1] <= 1.15 * us[0], us


@pytest.mark.parametrize("group", [4, 8])
def test_few_shared_blocks_keep_the_streaming_loads(group):
    """64 sequences of 3000..4100 tokens with a work list, 1.3% of whose
    references are to a shared block: the same tiles with the pool told of the
    sharing and without.  At most a tenth of the call's blocks can be shared, so
    both stream their tiles: the same bits and the same time (runs differ by 1%);
    with the default policy the told pool took 1.12 times as long.  The
    sequences of a second call are few against the same references: the same
    bits under the default policy, and what the oracle gives."""
    from types import SimpleNamespace
    from paper_2510_14126_amd import binding
    from paper_2510_14126_amd.device import PagedBatch
    print(f"[gpu case] few shared blocks and a work list, group {group}", flush=True)
    n, shared = 257, 3
    w, k, v = wide_batch(8, group, n, shared, np.linspace(3000, 16 * n, 64).round())
    us, outs = [], []
    for told in (False, True):
        pb = PagedBatch(w, "cuda:0", k_pool=k, v_pool=v, register_blocks=told, schedule=True)
        assert binding.kv_pool_num_shared(pb.pool) == (shared if told else 0)
        us.append(median_us(pb.run))
        outs.append(pb.out_bits())
        pb.close()
    few = SimpleNamespace(**{**vars(w), "batch": 5, "context_lens": w.context_lens[:5],
                             "block_tables": w.block_tables[:5], "q": w.q[:5]})
    pb = PagedBatch(few, "cuda:0", k_pool=k, v_pool=v, schedule=True)
    pb.run()
    torch.cuda.synchronize()
    assert np.array_equal(outs[0], outs[1])
    assert np.array_equal(outs[0][:5], pb.out_bits())
    pb.close()
    few.k_pool, few.v_pool = (x.view(torch.int16).cpu().numpy().view(np.uint16) for x in (k, v))
    assert compare(outs[0][:5], decode_workload(few)[0]).passed
    print(f"[gpu case] told of no sharing {us[0]:.1f} us, told {us[1]:.1f} us", flush=True)
    assert us[1] <= 1.06 * us[0], us


@pytest.mark.parametrize("S", [16, 64, 176, 1024])
@pytest.mark.parametrize("d,hq,hkv", [(64, 8, 2), (128, 12, 3), (128, 8, 1)])
def test_pairs_of_sequences_over_shared_blocks(d, hq, hkv, S):
    """Neighbouring sequences whose partitions hold the same blocks (four query
    heads: computed together) give the same bits as over private copies: shared
    prefixes that end inside a partition, an odd batch, contexts that end
    inside, at and one past the shared tokens, and the fused append."""
    prefix = 1056
    ctx = [prefix, prefix + 1, 1500, 1500, 1088, 3000, prefix + 16, 2112, 1100]
    print(f"[gpu case] pairs over shared blocks D={d} Hq={hq} Hkv={hkv} S={S}", flush=True)
    w = page_case(logical_case(440 + d + hq, len(ctx), hq, hkv, d, ctx, prefix_len=prefix), 441, poison=True)
    w.context_lens[2] = 700                # ends inside the shared tokens
    own = duplicate_shared_blocks(w)
    assert compare(run_step(w, S), decode_workload(w)[0]).passed
    for schedule in (False, True):
        assert np.array_equal(run_step(w, S, schedule), run_step(own, S, schedule))
    # the appended token: sequences 0 and 2 end in shared blocks and are left out
    rng = np.random.default_rng(442)
    new = [torch.from_numpy(f32_to_bf16_bits(rng.standard_normal((len(ctx), hkv, d), dtype=np.float32))
                            .view(np.int16)).cuda() for _ in range(2)]
    w.context_lens[[0, 2]] = 0
    own.context_lens[[0, 2]] = 0
    assert np.array_equal(run_step(w, S, new=new), run_step(own, S, new=new))


def run_step(w, S, schedule=False, new=None):
    from paper_2510_14126_amd.device import PagedBatch
    pb = PagedBatch(w, "cuda:0", partition_size=S, schedule=schedule)
    pb.out.fill_(0x7FC0)
    pb.decode_append(*new) if new else pb.decode()
    if pb.needs_reduce:
        pb.reduce()
    torch.cuda.synchronize()
    out = pb.out_bits()
    pb.close()
    return out


@pytest.mark.parametrize("append", [False, True])
@pytest.mark.parametrize("group", [4, 8])
def test_long_contexts_over_shared_blocks(group, append):
    """Both sides of the line from which one wavefront merges an item's rows
    (32 partitions of 512 tokens and 16384 workgroups in the grid: 64 sequences
    under a max_context_len of 16384, or 63): the same bits for the sequences
    that both batches hold, and what the oracle gives."""
    from types import SimpleNamespace
    from paper_2510_14126_amd.device import PagedBatch
    print(f"[gpu case] long contexts over shared blocks, group {group}, append {append}", flush=True)
    lens = [16384, 16383, 513, 3100, 0, 512, 1] + list(range(40, 40 + 57))
    if append:
        lens[4] = 17
    shared = 0 if append else 32                 # an appended block belongs to its sequence
    w, k, v = wide_batch(8, group, 1024, shared, lens)
    new = [torch.randn((64, 8, 128), dtype=torch.bfloat16, device="cuda:0") for _ in range(2)]
    outs = []
    for batch in (64, 63):
        x = SimpleNamespace(**{**vars(w), "batch": batch, "context_lens": w.context_lens[:batch],
                               "block_tables": w.block_tables[:batch], "q": w.q[:batch]})
        pb = PagedBatch(x, "cuda:0", k_pool=k.clone(), v_pool=v.clone(), register_blocks=False)
        one_shared_block(pb)
        pb.out.fill_(0x7FC0)
        pb.decode_append(*(t[:batch].contiguous() for t in new)) if append else pb.decode()
        pb.reduce()
        torch.cuda.synchronize()
        outs.append(pb.out_bits()[:63])
        w.k_pool, w.v_pool = (t.view(torch.int16).cpu().numpy().view(np.uint16) for t in (pb.k, pb.v))
        pb.close()
    assert np.array_equal(outs[0], outs[1])
    w.batch = 63
    for name in ("q", "context_lens", "block_tables"):
        setattr(w, name, getattr(w, name)[:63])
    rep = compare(outs[0], decode_workload(w)[0])
    assert rep.passed, f"{rep}"


def one_shared_block(pb):
    """A pool that knows one shared block: the default cache policy."""
    from paper_2510_14126_amd import binding
    ids = binding.kv_pool_alloc(pb.pool, 1)
    binding.kv_pool_retain(pb.pool, ids)


@pytest.mark.parametrize("group", [4, 8])
def test_head64_items_keep_up_with_their_gather(group):
    """256 sequences of 256 tokens at D = 64 against the same tiles read with no
    arithmetic, in the same launch shape: 1.14 times as long measured, 1.34 with
    a ring of four tiles, whose loads past an item's end cost that much on
    items of four tiles per wavefront."""
    from types import SimpleNamespace
    from paper_2510_14126_amd.device import PagedBatch
    print(f"[gpu case] D=64 decode against its gather, group {group}", flush=True)
    batch, hkv, d, n = 256, 8, 64, 16
    k, v = (torch.randn((batch * n, hkv, 16, d), dtype=torch.bfloat16, device="cuda:0") for _ in range(2))
    w = SimpleNamespace(batch=batch, num_q_heads=group * hkv, num_kv_heads=hkv, head_dim=d, num_blocks=batch * n,
                        context_lens=np.full(batch, 16 * n, np.int32), scale=0.125, partition_size=0,
                        block_tables=np.random.default_rng(8).permutation(batch * n).reshape(batch, n).astype(np.int32),
                        max_context_len=16 * n,
                        q=f32_to_bf16_bits(np.random.default_rng(9).standard_normal((batch, group * hkv, d),
                                                                                    dtype=np.float32)))
    pb = PagedBatch(w, "cuda:0", k_pool=k, v_pool=v)
    spans = torch.from_numpy(pb.tile_spans()).cuda()
    sink = torch.empty(len(spans) * hkv * 4, dtype=torch.int32, device="cuda:0")
    decode = median_us(pb.decode)
    gather = median_us(lambda: pb.gather_tiles(spans, len(spans), sink))
    pb.close()
    assert decode <= 1.24 * gather, (decode, gather)


@pytest.mark.parametrize("group", [4, 8])
def test_head64_lone_workgroups_keep_up_with_their_gather(group):
    """128 workgroups of 8192 tokens at D = 64, each with a CU to itself, against
    the same tiles read with no arithmetic: 1.31 times as long measured, 1.47
    with a ring of two tiles."""
    from types import SimpleNamespace
    from paper_2510_14126_amd.device import PagedBatch
    print(f"[gpu case] D=64 long items on an idle GPU against their gather, group {group}", flush=True)
    batch, hkv, d, n = 16, 8, 64, 512
    k, v = (torch.randn((batch * n, hkv, 16, d), dtype=torch.bfloat16, device="cuda:0") for _ in range(2))
    w = SimpleNamespace(batch=batch, num_q_heads=group * hkv, num_kv_heads=hkv, head_dim=d, num_blocks=batch * n,
                        context_lens=np.full(batch, 16 * n, np.int32), scale=0.125, partition_size=0,
                        block_tables=np.random.default_rng(8).permutation(batch * n).reshape(batch, n).astype(np.int32),
                        max_context_len=16 * n,
                        q=f32_to_bf16_bits(np.random.default_rng(9).standard_normal((batch, group * hkv, d),
                                                                                    dtype=np.float32)))
    pb = PagedBatch(w, "cuda:0", k_pool=k, v_pool=v)
    spans = torch.from_numpy(pb.tile_spans()).cuda()
    sink = torch.empty(len(spans) * hkv * 4, dtype=torch.int32, device="cuda:0")
    decode = median_us(pb.decode)
    gather = median_us(lambda: pb.gather_tiles(spans, len(spans), sink))
    print(f"[gpu case] decode {decode:.2f} us, gather {gather:.2f} us", flush=True)
    pb.close()
    assert decode <= 1.39 * gather, (decode, gather)


@pytest.mark.parametrize("S", [0, 512, 1024])
@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("hq,hkv", [(8, 2), (24, 3)])
def test_head64_ring_depths_agree(hq, hkv, shared, S):
    """At D = 64 the ring holds four tiles in up to 256 workgroups of long items,
    else two; a wavefront takes its blocks in the same order either way, so a
    batch has the same bits alone and as the first rows of one whose grid is
    larger, and what the oracle gives."""
    from paper_2510_14126_amd.device import PagedBatch
    print(f"[gpu case] D=64 ring depths Hq={hq} Hkv={hkv} S={S} shared={shared}", flush=True)
    ctx = [0, 1, 16, 17, 63, 65, 511, 513, 1023, 1025, 1041, 2064, 2100]
    copies = 1 + 256 // (hkv * len(ctx))
    w = page_case(logical_case(440 + hq, len(ctx), hq, hkv, 64, ctx), 441, poison=True)
    rep = lambda x: np.concatenate([x] * copies)
    many = replace(w, batch=copies * len(ctx), q=rep(w.q), block_tables=rep(w.block_tables),
                   context_lens=rep(w.context_lens))
    outs = []
    for case in (w, many):
        pb = PagedBatch(case, "cuda:0", partition_size=S, register_blocks=False)
        parts = -(-max(ctx) // S) if S else 1
        assert (parts * case.batch * hkv <= 256) == (case is w)
        if shared:
            one_shared_block(pb)
        pb.run()
        torch.cuda.synchronize()
        outs.append(pb.out_bits()[: len(ctx)])
        pb.close()
    report = compare(outs[0], decode_workload(w)[0])
    assert report.passed, f"{report}"
    assert np.array_equal(outs[0], outs[1])


def median_us(call):
    """Median time of one call, in microseconds."""
    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    times = []
    for _ in range(8):                      # the first warms up
        a.record()
        for _ in range(20):
            call()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 1e3 / 20)
    return sorted(times[1:])[3]
