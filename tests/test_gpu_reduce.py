"""The cross-split merge at the edges of its groups of partitions (eight per
wavefront, eight wavefronts, 64 log-sum-exps per round), with NaN in every
slot that no partition wrote, against the same merge in float64.  Tolerance:
rounding to nearest with bf16's eight significant bits is off by at most 2^-8
of the value (half a unit in the last place, 2^-7, of the smallest
significand), plus 1e-5 of the row's largest value for the fp32 sums."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import bf16_to_f64  # noqa: E402


@pytest.mark.parametrize("stride", [1, 7, 8, 9, 16, 63, 64, 65, 130])
@pytest.mark.parametrize("d", [64, 128])
def test_reduce_group_edges(d, stride):
    from paper_2510_14126_amd import binding
    print(f"[gpu case] reduce D={d} partitions={stride}", flush=True)
    S, hq = 32, 4
    parts = sorted({0, 1, min(2, stride), max(stride - 1, 0), stride, (stride + 1) // 2})
    ctx = np.array([max(0, p * S - (i % S if p else 0)) for i, p in enumerate(parts)], np.int32)
    assert [-(-int(n) // S) for n in ctx] == parts
    rng = np.random.default_rng(500 + stride)
    o = np.full((len(parts), hq, stride, d), np.nan, np.float32)
    lse = np.full((len(parts), hq, stride), np.nan, np.float32)
    ref = np.zeros((len(parts), hq, d))
    for b, p in enumerate(parts):
        o[b, :, :p] = rng.standard_normal((hq, p, d))
        lse[b, :, :p] = 3 * rng.standard_normal((hq, p))
        if p > 2:
            lse[b, 0, 1] = -np.inf          # a partition in which a row attended to nothing
        if p:
            w = np.exp(lse[b, :, :p].astype(np.float64) - lse[b, :, :p].max(axis=1, keepdims=True))
            ref[b] = (w[:, :, None] * o[b, :, :p]).sum(axis=1) / w.sum(axis=1)[:, None]
    out = torch.full((len(parts), hq, d), 0x7FC0, dtype=torch.int16, device="cuda:0")
    binding.paged_attn_reduce(torch.from_numpy(o).cuda(), torch.from_numpy(lse).cuda(),
                              torch.from_numpy(ctx).cuda(), len(parts), hq, d, S, stride, out)
    torch.cuda.synchronize()
    got = bf16_to_f64(out.cpu().numpy().view(np.uint16))
    assert np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-5 * np.abs(ref).max(axis=2, keepdims=True))


def reduce_us(rows_b, hq, d, S, stride, ctx):
    """Median time of one merge call, in microseconds."""
    from paper_2510_14126_amd import binding
    o = torch.zeros((rows_b, hq, stride, d), device="cuda:0")
    lse = torch.zeros((rows_b, hq, stride), device="cuda:0")
    lens = torch.full((rows_b,), ctx, dtype=torch.int32, device="cuda:0")
    out = torch.empty((rows_b, hq, d), dtype=torch.int16, device="cuda:0")
    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    times = []
    for _ in range(8):                      # the first warms up
        a.record()
        for _ in range(20):
            binding.paged_attn_reduce(o, lse, lens, rows_b, hq, d, S, stride, out)
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 1e3 / 20)
    return sorted(times[1:])[3]


def test_slots_that_no_partition_wrote_are_not_read():
    """8192 rows of one partition each take about as long in buffers for 64
    partitions (a loose max_context_len) as in buffers for one: 4.7 against 3.5
    us measured, at most 10 us if every row moved the 64 log-sum-exps besides
    its 512 + 256 bytes (12 MB at 2 TB/s, and the launch).  Reading all 64 rows is
    268 MB, over 33 us at the nominal 8 TB/s."""
    print("[gpu case] reduce: 8192 rows, one partition, buffers for 64 and for one", flush=True)
    tight = reduce_us(128, 64, 128, 512, 1, 500)
    loose = reduce_us(128, 64, 128, 512, 64, 500)
    assert loose <= tight + 10.0, (loose, tight)


@pytest.mark.parametrize("prefix", [0, 8])
@pytest.mark.parametrize("rows_b", [4, 8, 9, 40])
@pytest.mark.parametrize("stride", [8, 9, 65, 130])
def test_reduce_forms(rows_b, stride, prefix):
    """Both sides of the lines between the kernel's forms (64 heads: 512 | 576
    rows; early loads of up to 4 MB that may be in vain; streaming loads beyond
    32 MB of partials) give the float64 merge, with NaN in every slot that no
    partition wrote and sequences of none, some and all partitions after those
    that all have."""
    from paper_2510_14126_amd import binding
    print(f"[gpu case] reduce forms rows={64 * rows_b} partitions={stride} prefix={prefix}", flush=True)
    S, hq, d = 16, 64, 128
    parts = np.array([max(prefix, (0, 1, stride, stride // 2)[i % 4]) for i in range(rows_b)])
    rng = np.random.default_rng(520 + stride)
    o = np.full((rows_b, hq, stride, d), np.nan, np.float32)
    lse = np.full((rows_b, hq, stride), np.nan, np.float32)
    ref = np.zeros((rows_b, hq, d))
    for b, p in enumerate(parts):
        if p:
            o[b, :, :p] = rng.standard_normal((hq, p, d), dtype=np.float32)
            lse[b, :, :p] = 3 * rng.standard_normal((hq, p))
            w = np.exp(lse[b, :, :p].astype(np.float64) - lse[b, :, :p].max(axis=1, keepdims=True))
            ref[b] = (w[:, None, :] @ o[b, :, :p].astype(np.float64))[:, 0] / w.sum(axis=1)[:, None]
    out = torch.full((rows_b, hq, d), 0x7FC0, dtype=torch.int16, device="cuda:0")
    args = [torch.from_numpy(o).cuda(), torch.from_numpy(lse).cuda(),
            torch.from_numpy((parts * S).astype(np.int32)).cuda(), rows_b, hq, d, S]
    if prefix:
        binding.paged_attn_reduce_cascade(*args, prefix * S, S, stride, out)
    else:
        binding.paged_attn_reduce(*args, stride, out)
    torch.cuda.synchronize()
    got = bf16_to_f64(out.cpu().numpy().view(np.uint16))
    assert np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-5 * np.abs(ref).max(axis=2, keepdims=True))
