"""The two forms of the pass over shared tokens, on both sides of the rule
that chooses between them: query rows around one and two 32-row tiles (and
past 64), partitions of one block to 1024 tokens with odd block counts,
contexts that end inside the shared tokens, groups, and negative and zero
scales.  Poison past every context; outputs against the oracle under the
parity gate, and the full grid against the work list bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import compare, decode_workload  # noqa: E402
from workloads import group_starts, grouped_case, logical_case, page_case  # noqa: E402


def split_form(w, partition_size, prefix_len, prefix_partition_size, group_start=None, group_len=0):
    """The rule of cascade.hip (split_span), restated: whether a step takes the
    form for small grids (tokens split over the wavefronts, 32 rows each)."""
    group = w.num_q_heads // w.num_kv_heads

    def tiles(rows):
        return -(-rows // 32)

    runs = -(-prefix_len // prefix_partition_size) * tiles(w.batch * group)
    if group_len:
        runs += (len(group_start) - 1) * tiles(int(np.diff(group_start).max()) * group)
    runs += -(-(w.max_context_len - prefix_len - group_len) // partition_size) * w.batch
    return runs * w.num_kv_heads <= 320 + 20 * (max(min(prefix_len, prefix_partition_size), group_len) // 32)


def outputs(w, schedule, **kw):
    from paper_2510_14126_amd.device import PagedBatch
    pb = PagedBatch(w, "cuda:0", schedule=schedule, **kw)
    pb.out.fill_(0x7FC0)                   # NaN bits: every row must be written
    pb.run()
    torch.cuda.synchronize()
    out = pb.out_bits()
    pb.close()
    return out


def check(w, what, **kw):
    print(f"[gpu case] shared span {what}", flush=True)
    out = outputs(w, True, **kw)
    assert np.array_equal(out, outputs(w, False, **kw)), "the work list changed bits"
    rep = compare(out, decode_workload(w)[0])
    assert rep.passed, f"{what}: {rep}"


@pytest.mark.parametrize("prefix,pps", [(16, 16), (48, 1024), (80, 32), (544, 528), (1040, 1024)])
@pytest.mark.parametrize("hq,hkv,batch,split", [(4, 1, 1, True), (4, 1, 8, True), (12, 3, 9, True), (28, 7, 17, True),
                                                (8, 1, 4, True), (64, 8, 5, True), (32, 8, 90, False),
                                                (64, 8, 56, False)])
def test_prefix_tiles(hq, hkv, batch, split, prefix, pps):
    rng = np.random.default_rng(700 + batch)
    ctx = prefix + rng.integers(1, 70, size=batch)
    w = page_case(logical_case(701 + batch, batch, hq, hkv, 128, ctx, prefix_len=prefix), 702, poison=True)
    if batch > 3:                          # contexts that end inside the shared tokens
        w.context_lens[2] = 5
        w.context_lens[1] = 0
        w.context_lens[3] = prefix - 1
    kw = dict(partition_size=64, prefix_len=prefix, prefix_partition_size=pps)
    assert split_form(w, **kw) == split
    check(w, f"Hq={hq} Hkv={hkv} batch={batch} prefix={prefix}/{pps}", **kw)


@pytest.mark.parametrize("scale", [-0.15, 0.0])
@pytest.mark.parametrize("batch", [6, 90])
def test_scale_sign(batch, scale):
    ctx = 96 + np.arange(batch) % 37
    w = page_case(logical_case(720, batch, 32, 8, 128, ctx, prefix_len=96, scale=scale), 721, poison=True)
    w.context_lens[2] = 40
    check(w, f"scale {scale} batch={batch}", partition_size=64, prefix_len=96, prefix_partition_size=48)


@pytest.mark.parametrize("sizes", [[1], [8, 1, 16, 9], [5] * 20])
@pytest.mark.parametrize("hq,hkv,mid", [(4, 1, 16), (28, 7, 144), (32, 8, 1024)])
def test_group_tiles(hq, hkv, mid, sizes):
    suffix = 1 + np.arange(sum(sizes)) * 7 % 50
    w = grouped_case(730 + hq, hq, hkv, 128, 64, sizes, mid, suffix)
    check(w, f"groups Hq={hq} Hkv={hkv} sizes={sizes[:4]} mid={mid}", partition_size=32, prefix_len=64,
          prefix_partition_size=48, group_start=group_starts(w), group_len=mid)
