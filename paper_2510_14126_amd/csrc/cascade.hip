// One-launch shared-prefix (cascade) step: some workgroups run the
// shared-prefix pass (matrix-core tiles over all query rows) and, with a
// second level, the pass over each group's shared tokens (tiles over the
// group's rows), in one of two forms (split_span); the others run the
// per-sequence decode over the tokens after what is shared.  All write
// disjoint (o, lse) partials, so they need no synchronisation.  Shared and
// per-sequence work alternate in runs of num_kv_heads workgroups (with a phase
// flip every 8 runs, see below), so every CU holds some of each at once: the
// L2-fed prefix work overlaps the HBM-fed per-sequence work instead of
// preceding it, and workgroup i still serves KV head
// i % num_kv_heads, which keeps each head on one XCD (the dispatcher deals
// workgroups to the XCDs round-robin).
#include "decode_body.h"
#include "mfma_body.h"
#include "shared_body.h"
#include "shared_rows_body.h"

namespace pa {
namespace {

constexpr int kMax(int a, int b) { return a > b ? a : b; }
template <int G, bool SPLIT>
constexpr int cascade_lds() { return kMax(SPLIT ? shared::kLdsBytes : mfma::kPrefixLdsBytes, decode::lds_bytes<128, G, true>()); }

// Tiles in flight per wavefront of the per-sequence half: two for the short
// tails of the G = 4 stages, three for the 512-token items of G = 8.  (Four
// and four: 64-call generator step 25.0 -> 25.6 us, fixer iteration 50.0 ->
// 51.3 us, long-context step 1503 -> 1509 us; three and two: 25.6, 50.6 and
// 1501 us.)
template <int G>
constexpr int cascade_nbuf() { return G == 4 ? 2 : 3; }

template <int G, bool TRACE, bool APPEND, bool SPLIT>
__global__ void __launch_bounds__(64 * mfma::kWaves) __attribute__((amdgpu_waves_per_eu(2, 8)))
cascade_kernel(const PrefixParams pp, const DecodeParams dp, int prefix_runs, int group_runs,
               int decode_runs) {
  __shared__ __attribute__((aligned(16))) uint8_t smem[cascade_lds<G, SPLIT>()];
  lds_u8_t* lds = (lds_u8_t*)smem;
  // Run r = blockIdx / Hkv: while both kinds remain, even runs are shared
  // runs (the prefix partitions, then the groups) and odd runs decode runs;
  // then the longer kind continues alone.
  const int hkv = dp.num_kv_heads;
  const int run = blockIdx.x / hkv;
  const int g = blockIdx.x - run * hkv;
  const int shared_runs = prefix_runs + group_runs;
  const int both = min(shared_runs, decode_runs);
  bool shared;
  int idx;
  if ((SPLIT ? 1 : 3) * shared_runs >= decode_runs) {
    // Many shared runs: all of them first; consecutive ones reach every shader
    // engine.  Rows form, from a third of the decode runs on: 2% faster than
    // interleaving on the fixer batch with its request groups.  Split form, whose
    // runs are twice as many and shorter, from as many as decode runs on: with a
    // third, 51.2 -> 54.7 us on the same batch.
    shared = run < shared_runs;
    idx = shared ? run : run - shared_runs;
  } else if (run < 2 * both) {
    // Alternate, flipping the phase every 8 runs.  Each XCD hands its
    // workgroups to its four shader engines in a fixed cycle and waits for
    // the next engine in the cycle to have room, so a plain alternation would
    // put every shared run on two engines of each XCD and every decode run on
    // the other two (measured: dispatch then stalls on the engines that hold
    // the longest items while the others sit half empty).
    const int blk = run >> 3, w = run & 7;
    shared = ((w ^ blk) & 1) == 0;
    idx = (blk << 2) + (w >> 1);
  } else {
    shared = shared_runs > decode_runs;
    idx = both + (run - 2 * both);
  }
  if (shared) {
    if constexpr (SPLIT) {
      if (idx < prefix_runs)
        shared::prefix_body<G, TRACE>(pp, idx * hkv + g, lds);
      else
        shared::group_body<G, TRACE>(pp, (idx - prefix_runs) * hkv + g, lds);
    } else {
      if (idx < prefix_runs)
        mfma::prefix_mfma_body<G, TRACE>(pp, idx * hkv + g, lds);
      else
        mfma::group_mfma_body<G, TRACE>(pp, (idx - prefix_runs) * hkv + g, lds);
    }
    return;
  }
  const int wg = idx * hkv + g;
  decode::decode_body<128, G, cascade_nbuf<G>(), TRACE, /*STREAM=*/true, APPEND>(dp, wg, lds);
}

}  // namespace

namespace {

// Whether the shared spans go to shared_body.h (32 rows per workgroup, tokens
// split over the wavefronts) or to shared_rows_body.h (64 rows, 16 per
// wavefront).  The first form's chain per workgroup is four times shorter,
// the second has half the workgroups and reads from L2.  While the grid is
// small the chain is the step: the split form is taken up to a number of
// workgroups that grows with the chain.  Whole step, 32 query heads over 8,
// rows / split form: 2048-token prefix in 512-token partitions, batch 2 21.7
// / 11.0 us, 16 19.4 / 12.3, 48 (576 workgroups) 23.1 / 19.3, 64 (768) 23.8 /
// 24.9; request groups with 1024-token partitions, 8 requests 36.5 / 22.1, 24
// (896) 45.2 / 40.5, 32 (1192) 50.4 / 51.2; one KV head, 128 sequences over
// 4096 tokens (512) 23.6 / 21.4, 256 (1024) 31.3 / 36.1; 32 sequences of
// 8K-32K tokens (1856) 55.0 / 55.5.  Every launch of a step (plain, over a
// work list, with the fused append, traced) decides alike: the rule does not
// look at the work list.
bool split_span(const PrefixParams& pp, const DecodeParams& dp, int group) {
  const int64_t prefix_tiles = ((int64_t)pp.batch * group + kSharedTileRows - 1) / kSharedTileRows;
  const int64_t group_tiles = ((int64_t)pp.max_group_size * group + kSharedTileRows - 1) / kSharedTileRows;
  const int64_t runs = pp.prefix_parts * prefix_tiles + (pp.num_groups > 0 ? pp.num_groups * group_tiles : 0) +
                       (int64_t)dp.num_parts * dp.batch;
  const int prefix_tokens = pp.prefix_len < pp.part_tokens ? pp.prefix_len : pp.part_tokens;
  const int chain = (prefix_tokens > pp.group_len ? prefix_tokens : pp.group_len) / 32;   // block pairs
  return runs * pp.num_kv_heads <= 320 + 20 * chain;
}

template <int G, bool SPLIT>
hipError_t launch_t(const PrefixParams& pp, const DecodeParams& dp, bool trace, hipStream_t stream) {
  // Every kind of work is whole runs of num_kv_heads workgroups (the KV head
  // is the fastest index of all).
  constexpr int64_t kTileRows = SPLIT ? kSharedTileRows : kSharedRowsPerWg;
  const int64_t prefix_runs = pp.prefix_parts * (((int64_t)pp.batch * G + kTileRows - 1) / kTileRows);
  const int64_t group_runs =
      pp.num_groups > 0 ? pp.num_groups * (((int64_t)pp.max_group_size * G + kTileRows - 1) / kTileRows) : 0;
  const int64_t decode_runs = decode_items(dp);
  const int64_t grid = (prefix_runs + group_runs + decode_runs) * dp.num_kv_heads;
  if (grid == 0) return hipSuccess;
  if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(64 * mfma::kWaves), 0, stream, pp, dp,
                       (int)prefix_runs, (int)group_runs, (int)decode_runs);
  };
  // The trace kernels have no fused append.
  if (trace)
    go(cascade_kernel<G, true, false, SPLIT>);
  else if (dp.k_new != nullptr)
    go(cascade_kernel<G, false, true, SPLIT>);
  else
    go(cascade_kernel<G, false, false, SPLIT>);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_cascade(const PrefixParams& pp, const DecodeParams& dp, int group, bool trace,
                          hipStream_t stream) {
  if (pp.num_kv_heads != dp.num_kv_heads) return hipErrorInvalidValue;
  const bool split = split_span(pp, dp, group);
  if (group == 4) return split ? launch_t<4, true>(pp, dp, trace, stream) : launch_t<4, false>(pp, dp, trace, stream);
  if (group == 8) return split ? launch_t<8, true>(pp, dp, trace, stream) : launch_t<8, false>(pp, dp, trace, stream);
  return hipErrorInvalidValue;
}

}  // namespace pa
