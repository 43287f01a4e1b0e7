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
