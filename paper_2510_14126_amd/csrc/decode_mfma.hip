// Split-KV paged decode attention on MFMA tiles: kernel entry points.  The
// algorithm lives in decode_body.h; the shared-prefix cascade runs it inside
// its own kernel (cascade.hip).
#include "decode_body.h"

namespace pa {
namespace {

using mfma::kWaves;

// Tiles kept in flight per wavefront (DEEP: see deep_ring).  With every tile read once from memory
// (STREAM) at D = 128, three tiles and two wavefronts per SIMD: 256 sequences
// of 64..8192 tokens take 238 us, against 251 us with two tiles and three
// wavefronts.  Where sequences share blocks the tiles come from L2, the items
// are short of latency hiding, not of bandwidth, and two tiles (154 VGPRs:
// three wavefronts per SIMD) win: 64 sequences over a shared 2048-token
// prefix 47.7 -> 42.6 us.  At D = 64 a tile is half the bytes, and the loads
// past an item's end, NBUF - 1 per wavefront, weigh more than the depth gains:
// four / three / two tiles, whole step, 48 sequences of 61..4093 tokens 29.0 /
// 28.6 / 28.2 us, 256 of 256 27.8 / 25.3 / 23.2, 64 over a shared 2048-token
// prefix 24.6 / 23.3 / 21.5, 256 of 64..8192 in 512-token partitions 413 / 397 /
// 383 (VALU kernel 407), in one partition 391 / 394 / 386.
template <int D, bool STREAM, bool DEEP>
constexpr int nbuf() { return DEEP ? 4 : D == 128 && STREAM ? 3 : 2; }

template <int D, int G, bool TRACE, bool STREAM, bool APPEND, bool ONE_MERGE, bool DEEP>
__global__ void __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(2, ONE_MERGE && G == 8 ? 2 : 8)))
decode_mfma_kernel(const DecodeParams p) {
  __shared__ __attribute__((aligned(16))) uint8_t smem[decode::lds_bytes<D, G, STREAM>()];
  decode::decode_body<D, G, nbuf<D, STREAM, DEEP>(), TRACE, STREAM, APPEND, ONE_MERGE>(p, blockIdx.x, (lds_u8_t*)smem);
}

// Whether one wavefront merges and stores an item's rows, and at G = 8 two
// wavefronts per SIMD run instead of three: for long contexts with the default
// cache policy (D = 128), where the stores of many items that end at once, all
// four wavefronts of each, hold up the loads of the others.  Whole step, four /
// one storing wavefronts (G = 8: three / two per SIMD), G = 8: 128 sequences of
// 8K-32K tokens over 4096 shared ones 1698 / 1677 us, 64 of 8K-32K 1029 / 1018, in
// 1024-token partitions 992 / 975, 64 of 4K-16K (16384 workgroups) 508 / 498; G = 4:
// 1582 / 1561, 974 / 969, 949 / 948, 479 / 476.  The other side: 128 of up to 8K in
// 16 partitions, G = 8, 464 / 474, in 32 of 256 tokens 492 / 496, 8 of 8K-32K (4096
// workgroups) 131.4 / 132.4, short contexts over shared blocks 42 / 46; streaming
// 910 / 916.
bool one_merge(const DecodeParams& p) {
  return p.head_dim == 128 && p.part_tokens >= 512 && p.num_parts >= 32 &&
         (int64_t)p.num_parts * p.batch * p.num_kv_heads >= 16384;
}

// Whether the wavefronts keep four tiles in flight at D = 64: where every
// workgroup has a CU to itself and an item is long, a wavefront's own round trips
// are its time, and the loads past its end are few.  Whole step, two / four
// tiles, four heads per KV head: 3 sequences of 12.7K-20.8K tokens on one KV head
// in 2048-token partitions (33 workgroups) 21.6 / 19.8 us; 16 of 8K, 128 workgroups of
// 2048 tokens 24.5 / 22.2, 256 of 512 11.0 / 10.7.  The other side: 288 workgroups of
// 2048 tokens 32.0 / 35.4, 128 of 256 tokens 7.8 / 8.0; with the default cache policy
// (half of the tokens shared) 256 of 512 tokens 9.0 / 9.3, 224 of 1024 the same.
constexpr int64_t kDeepMaxWorkgroups = 256;   // one per CU
bool deep_ring(const DecodeParams& p, int64_t grid) {
  return p.head_dim == 64 && grid <= kDeepMaxWorkgroups && p.part_tokens >= (p.stream_tiles ? 512 : 1024);
}

// The trace kernel keeps the default cache policy (the hint changes no
// index) and has no fused append.
template <int D, int G>
hipError_t launch_t(const DecodeParams& p, bool trace, hipStream_t stream) {
  const int64_t grid = decode_items(p) * p.num_kv_heads;
  if (grid == 0) return hipSuccess;
  const bool append = p.k_new != nullptr;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(64 * kWaves), 0, stream, p);
  };
  constexpr bool kDeep = D == 64, kOneMerge = D == 128;
  const bool deep = deep_ring(p, grid);
  if (trace)
    go(decode_mfma_kernel<D, G, true, false, false, false, false>);
  else if (p.stream_tiles && append)
    go(deep ? decode_mfma_kernel<D, G, false, true, true, false, kDeep>
            : decode_mfma_kernel<D, G, false, true, true, false, false>);
  else if (p.stream_tiles)
    go(deep ? decode_mfma_kernel<D, G, false, true, false, false, kDeep>
            : decode_mfma_kernel<D, G, false, true, false, false, false>);
  else if (append)
    go(one_merge(p) ? decode_mfma_kernel<D, G, false, false, true, kOneMerge, false>
       : deep       ? decode_mfma_kernel<D, G, false, false, true, false, kDeep>
                    : decode_mfma_kernel<D, G, false, false, true, false, false>);
  else
    go(one_merge(p) ? decode_mfma_kernel<D, G, false, false, false, kOneMerge, false>
       : deep       ? decode_mfma_kernel<D, G, false, false, false, false, kDeep>
                    : decode_mfma_kernel<D, G, false, false, false, false, false>);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_decode_mfma(const DecodeParams& p, bool trace, hipStream_t stream) {
  const int group = p.num_q_heads / p.num_kv_heads;
  if (p.head_dim == 128 && group == 4) return launch_t<128, 4>(p, trace, stream);
  if (p.head_dim == 128 && group == 8) return launch_t<128, 8>(p, trace, stream);
  if (p.head_dim == 64 && group == 4) return launch_t<64, 4>(p, trace, stream);
  if (p.head_dim == 64 && group == 8) return launch_t<64, 8>(p, trace, stream);
  return hipErrorInvalidValue;
}

}  // namespace pa
