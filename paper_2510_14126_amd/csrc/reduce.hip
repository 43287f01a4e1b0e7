// Cross-split reduce: merge split-KV partials into the bf16 output.
//
// For sequence b and query head h the decode kernels left, per partition p,
// the partition-normalised output o_p and its log-sum-exp lse_p (natural
// log): first the partitions of a prefix shared by the whole batch (if any),
// then ceil((ctx_b - prefix) / S) partitions of the rest.  With M = max lse_p:
//     w_p = exp(lse_p - M),   out = sum_p w_p o_p / sum_p w_p,
// which is exactly softmax attention over the whole context (zeros when
// every w_p is 0).  NW wavefronts per (b, h).  Lane q loads lse_q (64
// partitions per round); the partitions' o rows are dealt to the wavefronts
// in groups of kGroup, each group loaded together.  Lane l owns output dims
// (D/64)*l .. and adds its wavefront's partitions in order (weights broadcast
// from the lane that computed them), then the wavefronts' sums are added in
// order through LDS, so the result is deterministic and P_b = 1 reproduces o_0
// bit for bit.
//
// What bounds it: the round trips to memory (context length, then partials)
// while rows are few, the bytes of the partials that exist while they are many.
// A buffer sized for a long max_context_len holds many slots that no partition
// wrote, so o rows are loaded after the context length says which exist, except
// where the call is so small that the rest costs nothing (PRE, launch_t).  Large
// buffers are read with the streaming hint (STREAM, kStreamBytes).
// (Loading every slot's row with the length, whatever the call: 128 sequences
// of 500 tokens under a bound of 32768, 64 heads, whole step 193 us, now 153;
// 256 of 64..8192 in 512-token partitions 320, now 308.)
#include "kernels.h"
#include "pa_device.h"

#include <algorithm>

namespace pa {
namespace {

constexpr int kGroup = 8;   // partitions whose o rows a wavefront loads together

template <int D, int NW, bool PRE, bool STREAM>
__global__ void __launch_bounds__(64 * NW) reduce_kernel(const ReduceParams p) {
  constexpr int DPL = D / 64;
  const int lane = threadIdx.x & 63;
  const int wave = wave_uniform(threadIdx.x >> 6);
  const int bh = blockIdx.x;
  const int b = bh / p.num_q_heads;
  const float* lse = p.part_lse + (size_t)bh * p.part_stride;
  const float* po = p.part_o + (size_t)bh * p.part_stride * D + DPL * lane;

  // o rows of partitions first .. first+kGroup-1 (clamped to `lastq`; what
  // lies past P_b, also lse, may hold anything and is never used)
  float v[kGroup][DPL];
  auto load_group = [&](int first, int lastq) {
#pragma unroll
    for (int k = 0; k < kGroup; ++k) {
      const int q = min(first + k, lastq);
#pragma unroll
      for (int d = 0; d < DPL; ++d) {
        const float* x = po + (size_t)q * D + d;
        v[k][d] = STREAM ? __builtin_nontemporal_load(x) : *x;
      }
    }
  };
  const float x0 = lane < p.part_stride ? lse[lane] : 0.f;
  if constexpr (PRE) load_group(wave * kGroup, p.part_stride - 1);

  int n = p.context_lens[b] - p.prefix_len;
  n = n < 0 ? 0 : n;
  int pb = p.prefix_parts + n / p.part_tokens + (n % p.part_tokens != 0);
  pb = pb > p.part_stride ? p.part_stride : pb;
  if constexpr (!PRE) {
    if (wave * kGroup < pb) load_group(wave * kGroup, pb - 1);
  }
  const float l0 = lane < pb ? x0 : -__builtin_inff();

  float mx = l0;
  for (int c0 = 64; c0 < pb; c0 += 64)
    mx = fmaxf(mx, c0 + lane < pb ? lse[c0 + lane] : -__builtin_inff());
  mx = group_max4(row_max16(mx));
  const float mref = (mx == -__builtin_inff()) ? 0.f : mx;

  float wsum = 0.f, o[DPL];
#pragma unroll
  for (int d = 0; d < DPL; ++d) o[d] = 0.f;
  for (int c0 = 0; c0 < pb; c0 += 64) {
    const float x = c0 == 0 ? l0 : (c0 + lane < pb ? lse[c0 + lane] : 0.f);
    const int wl = __float_as_int(fast_exp2((x - mref) * kLog2e));   // w of partition c0 + lane
    const int cnt = min(64, pb - c0);
    for (int j0 = wave * kGroup; j0 < cnt; j0 += NW * kGroup) {
      if (c0 + j0 > wave * kGroup) load_group(c0 + j0, pb - 1);
#pragma unroll
      for (int k = 0; k < kGroup; ++k) {
        if (j0 + k < cnt) {
          const float w = __int_as_float(__builtin_amdgcn_readlane(wl, j0 + k));
          wsum += w;
#pragma unroll
          for (int d = 0; d < DPL; ++d) o[d] = fmaf(w, v[k][d], o[d]);
        }
      }
    }
  }
  if constexpr (NW > 1) {
    __shared__ float so[NW][D], sw[NW];
#pragma unroll
    for (int d = 0; d < DPL; ++d) so[wave][DPL * lane + d] = o[d];
    if (lane == 0) sw[wave] = wsum;
    __syncthreads();
    if (wave != 0) return;
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      wsum += sw[w];
#pragma unroll
      for (int d = 0; d < DPL; ++d) o[d] += so[w][DPL * lane + d];
    }
  }
  const float inv = wsum > 0.f ? 1.0f / wsum : 0.f;
  uint16_t* orow = p.out + (size_t)bh * D;
  if constexpr (DPL == 2)
    *reinterpret_cast<uint32_t*>(orow + 2 * lane) = bf16_rne(o[0] * inv) | (bf16_rne(o[1] * inv) << 16);
  else
    orow[lane] = (uint16_t)bf16_rne(o[0] * inv);
}

// The eight-wavefront form is for calls of few rows: up to kWideRows of them
// their wavefronts fit the GPU at once.  Whole step, one / eight wavefronts: one
// sequence of 59 partitions, 64 rows, 26.6 / 24.2 us, 256 rows of 59 88.7 / 86.6,
// 512 171.6 / 169.9; 1024 333.4 / 333.2, 2048 666 / 667, and with short contexts
// under a bound of 64 partitions 1024 rows 27.1 / 27.9, 8192 153 / 162.
constexpr int64_t kWideRows = 512;
// Most bytes of o rows that a call may load in vain before the context lengths
// arrive.  Up to 4 MB they cost less than the round trip they save; whole step,
// with / without the early loads: 64 rows of 59 partitions 23.6 / 24.2 us, 128 rows
// 45.0 / 45.5, 2048 of five 30.9 / 31.1; 64 and 128 rows of one partition under a
// bound of 64 (2 and 4 MB) the same, 256 (8 MB) 12.9 / 12.4, 2048 of one under a
// bound of six (5 MB) 18.4 / 17.9, of eight (7 MB) 20.2 / 18.8.
constexpr int64_t kPreloadBytes = (int64_t)4 << 20;

// Size of the partial buffer from which its rows are loaded with the streaming
// hint: more than the eight 4 MB L2s hold.  The decode left those rows dirty in the
// caches and nobody reads them again; with default loads they stay, and their
// write-back takes bandwidth from the next decode.  128 sequences of 8K-32K tokens
// (268 MB), whole step, default / streaming, one batch again and again 1441 / 1417
// us, two batches in turn 1500 / 1433; 256 of 64..8192 in 512-token partitions (67
// MB) 308.6 / 307.4.  In 5 MB it costs: 64 over a shared 2048-token prefix, three
// batches in turn, 23.8 / 24.1.
constexpr int64_t kStreamBytes = (int64_t)32 << 20;

template <int D, int NW>
void launch_nw(const ReduceParams& p, bool pre, hipStream_t stream) {
  const int64_t rows = (int64_t)p.batch * p.num_q_heads;
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3((unsigned)rows), dim3(64 * NW), 0, stream, p); };
  const bool nt = rows * p.part_stride * D * (int64_t)sizeof(float) > kStreamBytes;
  if (pre && nt)
    go(reduce_kernel<D, NW, true, true>);
  else if (pre)
    go(reduce_kernel<D, NW, true, false>);
  else if (nt)
    go(reduce_kernel<D, NW, false, true>);
  else
    go(reduce_kernel<D, NW, false, false>);
}

template <int D>
void launch_t(const ReduceParams& p, hipStream_t stream) {
  constexpr int kWide = 8;
  const int64_t rows = (int64_t)p.batch * p.num_q_heads;
  const bool wide = p.part_stride > kGroup && rows <= kWideRows;
  // slots loaded early, less those that every sequence (of at least one token) has
  const int early = std::min(p.part_stride, kGroup * (wide ? kWide : 1));
  const int vain = std::max(early - std::max(p.prefix_parts, 1), 0);
  const bool pre = rows * vain * D * (int64_t)sizeof(float) <= kPreloadBytes;
  if (wide)
    launch_nw<D, kWide>(p, pre, stream);
  else
    launch_nw<D, 1>(p, pre, stream);
}

}  // namespace

hipError_t launch_reduce(const ReduceParams& p, int head_dim, hipStream_t stream) {
  if (head_dim == 128)
    launch_t<128>(p, stream);
  else if (head_dim == 64)
    launch_t<64>(p, stream);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace pa
