// Attention of many query rows over a token span that they share, on 32x32
// MFMA tiles (gfx950, head_dim 128): the prefix that every sequence of the
// batch shares, and the tokens that a group of sequences shares after it.
//
// For KV head g the rows are (sequence, head) pairs: row R of the span is
// sequence seq0 + R / G, head g*G + R % G.  One workgroup owns
// kSharedTileRows rows (the columns of one 32x32 tile) and one partition of
// the span; its wavefronts take the partition's blocks two at a time (a stage
// of 32 tokens), round-robin, and merge through LDS at the end.  All
// workgroups of a KV head read the same blocks, so each comes from HBM once
// and from that XCD's L2 afterwards.  Every row writes its (o, lse) partial,
// lse = -inf when it attended to nothing.
//
// Lanes: h = lane >> 5, n = lane & 31.  v_mfma_f32_32x32x16_bf16 takes A row n
// / B column n at contraction indices 8h .. 8h+7 and leaves in register r of
// its result row 8(r/4) + 4h + r%4 of column n.
//  * K tiles are read in whole 256-byte token rows and put in LDS (k_off); S^T
//    = K Q^T takes A row i from the token that makes register r = 8m + e of
//    lane (h, n) the score of token 2e + h of block m for row n (a_row).
//  * V tiles are read in whole rows too, eight bytes per lane: lane (h, c)
//    holds dims 4c .. 4c+3 of tokens 2u + h (u = 0..7) of a block.  O += P V
//    takes k = 8h + e for token 2e + h, which makes the scores above exactly
//    the A operand and element j of the lane's own V registers the B operand
//    of output column c = dim 4c + j (four v_perm_b32 per MFMA): neither P nor
//    V moves between lanes.  Each probability reaches the matrix core as a
//    bf16 pair, high part and rounded remainder (about 2^-17 relative), two
//    MFMAs per PV step; the row sum adds the fp32 values.
// The running max, the lazy rescale and the scale are as in decode_body.h.
//
// What bounds it: the dependent chain of a stage (loads, LDS, QK^T, softmax,
// PV).  Splitting the partition's tokens over the wavefronts instead of its
// rows makes the chain four times shorter: three sequences over a 768-token
// prefix, one partition, 27.7 -> 12.4 us a step.  extend_body.h uses the same
// routine for small chunks.  Both sides of the choice are measured at
// split_span (cascade.hip) and at launch_t (extend.hip).
#pragma once

#include "kernels.h"
#include "mfma_body.h"
#include "pa_device.h"

namespace pa {
namespace shared {

using mfma::bf16x8_t;
using mfma::floatx16_t;
using mfma::floatx4_t;
using mfma::kLazyRescale;
using mfma::kWaves;
using mfma::lds_floatx4_t;
using mfma::lds_u32x4_t;
using mfma::pack_bf16;
using mfma::u32x4_t;

constexpr int kD = 128;
constexpr int kRows = kSharedTileRows;
static_assert(kRows == 32, "the columns of a 32x32 tile");
constexpr int kStageBytes = 2 * 16 * kD * 2;          // the K rows of a stage
constexpr int kSwapBytes = 4 * 1024;                  // one wavefront's outputs for another at the merge
constexpr int kMergeBytes = kWaves * (kWaves - 1) * kSwapBytes;
constexpr int kStatOffset = kMergeBytes > kWaves * kStageBytes ? kMergeBytes : kWaves * kStageBytes;
constexpr int kLdsBytes = kStatOffset + 3 * kWaves * kRows * 4;   // maxima, sums, one value per row

// LDS byte offset of 16-byte chunk c of row r (0..31, block r / 16) of a
// staged K tile pair: chunk c at position c ^ (r % 16).  Writers fill whole
// rows; eight consecutive reading lanes (rows a_row(n), eight consecutive
// ones in some order) touch positions that differ modulo eight.
__device__ __forceinline__ int k_off(int r, int c) { return r * (2 * kD) + ((c ^ (r & 15)) << 4); }

// Row of the staged pair that supplies A row i: i = 8a + 4h + b is token
// 2(4(a%2) + b) + h of block a/2.
__device__ __forceinline__ int a_row(int i) {
  const int a = i >> 3, h = (i >> 2) & 1, b = i & 3;
  return 16 * (a >> 1) + 2 * (4 * (a & 1) + b) + h;
}

// One value per row, from the lane (h, n) that holds it as column n, to the lanes
// that hold the row's outputs: rows 8a + 4h + b in out[4a + b].  rowv: 32 floats
// of LDS of the wavefront's own.
__device__ __forceinline__ void per_row(lds_f32_t* rowv, int h, int n, float x, float (&out)[16]) {
  if (h == 0) rowv[n] = x;
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const floatx4_t y = *reinterpret_cast<const lds_floatx4_t*>(rowv + 8 * a + 4 * h);
#pragma unroll
    for (int e = 0; e < 4; ++e) out[4 * a + e] = y[e];
  }
  __builtin_amdgcn_wave_barrier();
}

// Running-max step before a stage's probabilities: xmax is the lane's largest
// unmasked score of column n.  The test needs no cross-lane reduction: any lane
// above its row's max + kLazyRescale triggers the rescale.
__device__ __forceinline__ void raise_max(float xmax, float& m, float& neg, float& l, floatx16_t (&o)[4],
                                          lds_f32_t* rowv, int h, int n) {
  if (__builtin_amdgcn_ballot_w64(xmax > m + kLazyRescale) != 0) {
    float x = xmax, y = xmax;
    swap32(x, y);
    const float bm = fmaxf(x, y);
    const float mn = bm > m + kLazyRescale ? bm : m;
    // 1 for rows that keep their max (or have attended to nothing yet)
    const float alpha = mn == -__builtin_inff() ? 1.f : fast_exp2(m - mn);
    l *= alpha;
    if (__builtin_amdgcn_ballot_w64(m != -__builtin_inff()) != 0) {
      float ar[16];
      per_row(rowv, h, n, alpha, ar);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[j][r] *= ar[r];
    }
    m = mn;
    neg = mn == -__builtin_inff() ? 0.f : -mn;
  }
}

// The rows of one tile against nblk blocks, on all wavefronts of the workgroup.
//   q_row    query row (128 bf16) of column n
//   desc(base, i)  buffer descriptor of the tile at block i (i < nblk) of the
//            pool that starts at base (this KV head's tiles)
//   vis(i)   tokens of block i that column n sees (may exceed 16 or be
//            negative)
//   seen(i)  called once per block by the wavefront that loads it
//   stats(mx, lt)  maximum (log2 units) and sum of column n's row, once per
//            workgroup on wavefront 0 (both half wavefronts hold them)
//   put(row, c, acc)  dims 4c .. 4c+3 of the normalised output of a tile row
// A block that column n does not see, or a token past its vis, gets weight 0:
// its V must be finite or read as zero.
template <typename Desc, typename Vis, typename Seen, typename Stats, typename Put>
__device__ __forceinline__ void tile_core(const uint16_t* q_row, const uint16_t* kbase, const uint16_t* vbase,
                                          int nblk, float scale_log2, lds_u8_t* smem, Desc&& desc, Vis&& vis,
                                          Seen&& seen, Stats&& stats, Put&& put) {
  const int lane = threadIdx.x & 63;
  const int wave = wave_uniform(threadIdx.x >> 6);
  const int h = lane >> 5;
  const int n = lane & 31;

  // A negative scale goes into the sign of Q (bf16 negation is exact, and so
  // is the negation of every score).  A scale of zero becomes the smallest
  // normal number, so that masked scores stay -inf times it (scores below
  // 2^100 still weigh exactly the same).
  const uint32_t qflip = scale_log2 < 0.f ? 0x80008000u : 0u;
  const float scale = scale_log2 == 0.f ? 1.1754944e-38f : fabsf(scale_log2);
  u32x4_t qb[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const uint4 w = *reinterpret_cast<const uint4*>(q_row + (2 * s + h) * 8);
    qb[s] = u32x4_t{w.x ^ qflip, w.y ^ qflip, w.z ^ qflip, w.w ^ qflip};
  }

  const int nstage = (nblk + 1) >> 1;
  // Past the last block the descriptor is empty: the loads return zeros.
  const __amdgpu_buffer_rsrc_t none =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(kbase), 0, 0, kBufferDescWord3);
  const int krow = lane >> 4, kchunk = lane & 15;      // rows 4u + krow
  const int k_lane = (krow * kD + kchunk * 8) * 2;
  const int v_lane = (h * kD + n * 4) * 2;             // rows 2u + h, dims 4n ..
  u32x4_t rk[2][4];
  uint2 rv[2][8];
  auto load_k = [&](int s) {
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const __amdgpu_buffer_rsrc_t d = 2 * s + m < nblk ? desc(kbase, 2 * s + m) : none;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        rk[m][u] = __builtin_bit_cast(u32x4_t,
                                      __builtin_amdgcn_raw_buffer_load_b128(d, k_lane + u * 4 * kD * 2, 0, 0));
    }
  };
  auto load_v = [&](int s) {
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const __amdgpu_buffer_rsrc_t d = 2 * s + m < nblk ? desc(vbase, 2 * s + m) : none;
#pragma unroll
      for (int u = 0; u < 8; ++u)
        rv[m][u] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(d, v_lane + u * 2 * kD * 2, 0, 0));
    }
  };

  lds_u8_t* stage = smem + wave * kStageBytes;
  lds_f32_t* sm = reinterpret_cast<lds_f32_t*>(smem + kStatOffset);   // [kWaves][32]
  lds_f32_t* sl = sm + kWaves * kRows;                                 // [kWaves][32]
  lds_f32_t* rowv = sl + kWaves * kRows + wave * kRows;

  float m = -__builtin_inff(), neg = 0.f, l = 0.f;
  floatx16_t o[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[j][i] = 0.f;

  const int arow = a_row(n);
  load_k(wave);
  load_v(wave);
  for (int s = wave; s < nstage; s += kWaves) {
    // K through LDS; its registers take the next stage at once.
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int u = 0; u < 4; ++u)
        *reinterpret_cast<lds_u32x4_t*>(stage + k_off(16 * mb + 4 * u + krow, kchunk)) = rk[mb][u];
    load_k(s + kWaves);
    floatx16_t a;
#pragma unroll
    for (int i = 0; i < 16; ++i) a[i] = 0.f;
#pragma unroll
    for (int c = 0; c < 8; ++c)
      a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
          __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const lds_u32x4_t*>(stage + k_off(arow, 2 * c + h))),
          __builtin_bit_cast(bf16x8_t, qb[c]), a, 0, 0, 0);

    // Register r = 8 mb + e is token 2e + h of block 2s + mb.
    int see[2];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
      see[mb] = 2 * s + mb < nblk ? vis(2 * s + mb) : 0;
      if (2 * s + mb < nblk) seen(2 * s + mb);
    }
    if (__builtin_amdgcn_ballot_w64(min(see[0], see[1]) < 16) != 0) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (2 * (r & 7) + h >= see[r >> 3]) a[r] = -__builtin_inff();
    }

    float mx = a[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, a[r]);
    raise_max(mx * scale, m, neg, l, o, rowv, h, n);

    u32x4_t hi[2], lo[2];
    float sum[2];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        float pf[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          pf[i] = fast_exp2(fmaf(a[8 * mb + e + i], scale, neg));
        }
        const uint32_t hp = pack_bf16(pf[0], pf[1]);
        hi[mb][e / 2] = hp;
        lo[mb][e / 2] = pack_bf16(pf[0] - bf16_lo(hp), pf[1] - bf16_hi(hp));
        const float s2 = pf[0] + pf[1];
        sum[mb] = e == 0 ? s2 : sum[mb] + s2;
      }
    l += sum[0] + sum[1];

#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
      u32x4_t vb[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const uint2 v0 = rv[mb][2 * w], v1 = rv[mb][2 * w + 1];
          vb[j][w] = j < 2 ? __builtin_amdgcn_perm(v1.x, v0.x, sel) : __builtin_amdgcn_perm(v1.y, v0.y, sel);
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
        o[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, hi[mb]),
                                                       __builtin_bit_cast(bf16x8_t, vb[j]), o[j], 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        o[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, lo[mb]),
                                                       __builtin_bit_cast(bf16x8_t, vb[j]), o[j], 0, 0, 0);
    }
    load_v(s + kWaves);
  }

  // Merge.  Row n's maximum and sum over the wavefronts, then each wavefront
  // scales its outputs to the common maximum and the final sum; wavefront d
  // adds up rows 8d + 4h + b (b = 0..3), four dims per lane and row.
  {
    float x = l, y = l;
    swap32(x, y);
    if (h == 0) {
      sm[wave * kRows + n] = m;
      sl[wave * kRows + n] = x + y;
    }
  }
  __syncthreads();
  float mx = sm[n];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) mx = fmaxf(mx, sm[w * kRows + n]);
  const float mref = mx == -__builtin_inff() ? 0.f : mx;
  float lt = 0.f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) lt = fmaf(sl[w * kRows + n], fast_exp2(sm[w * kRows + n] - mref), lt);
  const float inv = lt > 0.f ? 1.0f / lt : 0.f;
  if (wave == 0) stats(mx, lt);
  float f[16];
  per_row(rowv, h, n, fast_exp2(m - mref) * inv, f);
  auto piece = [&](int d, int b) {   // the lane's dims of row 8d + 4h + b, normalised
    return floatx4_t{o[0][4 * d + b] * f[4 * d + b], o[1][4 * d + b] * f[4 * d + b],
                     o[2][4 * d + b] * f[4 * d + b], o[3][4 * d + b] * f[4 * d + b]};
  };
  auto slot = [&](int dst, int src) {   // outputs of wavefront src for wavefront dst
    return smem + (dst * (kWaves - 1) + (src > dst ? src - 1 : src)) * kSwapBytes + lane * 16;
  };
#pragma unroll
  for (int d = 0; d < kWaves; ++d)
    if (d != wave) {
#pragma unroll
      for (int b = 0; b < 4; ++b) *reinterpret_cast<lds_floatx4_t*>(slot(d, wave) + b * 1024) = piece(d, b);
    }
  __syncthreads();
#pragma unroll
  for (int d = 0; d < kWaves; ++d)
    if (d == wave) {
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        floatx4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kWaves; ++w)
          acc += w == d ? piece(d, b) : *reinterpret_cast<const lds_floatx4_t*>(slot(d, w) + b * 1024);
        put(8 * d + 4 * h + b, n, acc);
      }
    }
}

// Rows and tokens of one workgroup: rows row0 .. row0 + 31 of the span's rows
// 0 .. total_rows-1; tokens start .. end-1 (whole blocks), whose block ids
// begin at bt; the result goes to partial slot `part`; the walk over the
// blocks starts at block `rot`.
struct Span {
  int seq0, total_rows, row0;
  int start, end;
  const int32_t* bt;
  int part;
  int rot;
};

template <int G, bool TRACE>
__device__ __forceinline__ void span_body(const PrefixParams& p, int g, const Span& sp, lds_u8_t* smem,
                                          int32_t* trace) {
  const int lane = threadIdx.x & 63;
  const int n = lane & 31;
  const int nblk = (sp.end - sp.start) >> 4;    // 1 .. 64 for every launched span
  const int raw = lane < nblk ? sp.bt[lane] : 0;
  const int idc = min(max(raw, 0), p.num_blocks - 1);

  // Column n is row R = row0 + n.  A column without a row repeats the first
  // one's query, sees everything and is not written.
  const int R = sp.row0 + n;
  const bool has_row = R < sp.total_rows;
  const int bR = has_row ? sp.seq0 + R / G : sp.seq0;
  const size_t q_index = (size_t)bR * p.num_q_heads + g * G + (has_row ? R % G : 0);
  int lim = p.context_lens[bR];
  lim = !has_row ? 0x7fffffff : (lim < 0 ? 0 : (lim > p.max_ctx ? p.max_ctx : lim));

  constexpr size_t kTileElems = 16 * kD;
  const size_t blk_stride = (size_t)p.num_kv_heads * kTileElems;
  auto block_of = [&](int i) { const int j = i + sp.rot; return j >= nblk ? j - nblk : j; };
  tile_core(
      p.q + q_index * kD, p.k_pool + (size_t)g * kTileElems, p.v_pool + (size_t)g * kTileElems, nblk,
      p.scale_log2, smem,
      [&](const uint16_t* base, int i) {
        const size_t id = (size_t)__builtin_amdgcn_readlane(idc, block_of(i));
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base + id * blk_stride), 0,
                                                 (int)(kTileElems * 2), kBufferDescWord3);
      },
      [&](int i) { return lim - (sp.start + 16 * block_of(i)); },
      [&](int i) {
        if constexpr (TRACE) {
          // slot = the block's position in the span (not in the walk)
          const int b = block_of(i);
          const int id = __builtin_amdgcn_readlane(raw, b);
          if (lane == 0) {
            int32_t* tr = trace + 3 * b;
            tr[0] = (sp.start >> 4) + b;
            tr[1] = id;
            tr[2] = 16;
          }
        }
      },
      [&](float mx, float lt) {
        if (lane < kRows && has_row)
          p.part_lse[q_index * p.part_stride + sp.part] = lt > 0.f ? (mx + log2f(lt)) * kLn2 : -__builtin_inff();
      },
      [&](int r, int c, const floatx4_t& acc) {
        const int row = sp.row0 + r;
        if (row < sp.total_rows) {
          const size_t at = ((size_t)(sp.seq0 + row / G) * p.num_q_heads + g * G + row % G) * p.part_stride + sp.part;
          store_partial4(p.part_o + at * kD + 4 * c, acc[0], acc[1], acc[2], acc[3]);
        }
      });
}

// The batch-wide prefix: partition `part` of the prefix against row tile
// `tile` of all B*G query rows of KV head g.
template <int G, bool TRACE>
__device__ __forceinline__ void prefix_body(const PrefixParams& p, int wg_index, lds_u8_t* smem) {
  const int total_rows = p.batch * G;
  const int tiles = (total_rows + kRows - 1) / kRows;
  int wg = wg_index;
  const int g = wg % p.num_kv_heads;
  wg /= p.num_kv_heads;
  const int tile = wg % tiles;
  const int part = wg / tiles;
  Span sp;
  sp.seq0 = 0;
  sp.total_rows = total_rows;
  sp.row0 = tile * kRows;
  sp.start = part * p.part_tokens;
  sp.end = min(p.prefix_len, sp.start + p.part_tokens);
  sp.bt = p.block_tables + (sp.start >> 4);
  sp.part = part;
  // The workgroups of a KV head walk the partition from evenly spread
  // starting blocks, so at any moment they read different blocks instead of
  // all queueing on the L2 lines of the same one.
  const int nblk = (sp.end - sp.start) >> 4;
  sp.rot = (int)(((int64_t)tile * nblk) / tiles) % nblk;
  int32_t* tr = nullptr;
  if constexpr (TRACE) {
    // one trace per kSharedRowsPerWg rows: its tiles read the same blocks
    const int groups = (total_rows + kSharedRowsPerWg - 1) / kSharedRowsPerWg;
    const int grp = sp.row0 / kSharedRowsPerWg;
    tr = p.trace_prefix + (((size_t)part * groups + grp) * p.num_kv_heads + g) * p.prefix_trace_tiles * 3;
  }
  span_body<G, TRACE>(p, g, sp, smem, tr);
}

// The second level: row tile `tile` of group k's rows (its sequences x G heads
// of KV head g) against the group_len tokens the group shares after the
// prefix, one partition written to slot prefix_parts.
template <int G, bool TRACE>
__device__ __forceinline__ void group_body(const PrefixParams& p, int wg_index, lds_u8_t* smem) {
  int wg = wg_index;
  const int g = wg % p.num_kv_heads;
  wg /= p.num_kv_heads;
  const int tiles = (p.max_group_size * G + kRows - 1) / kRows;
  const int tile = wg % tiles;
  const int k = wg / tiles;
  // device data: clamped into the batch and the stated bound
  int s0 = p.group_start[k];
  s0 = s0 < 0 ? 0 : (s0 > p.batch ? p.batch : s0);
  int s1 = p.group_start[k + 1];
  s1 = s1 < s0 ? s0 : (s1 > p.batch ? p.batch : s1);
  s1 = min(s1, s0 + p.max_group_size);
  Span sp;
  sp.seq0 = s0;
  sp.total_rows = (s1 - s0) * G;
  sp.row0 = tile * kRows;
  if (sp.row0 >= sp.total_rows) return;        // whole workgroup: no rows here
  sp.start = p.prefix_len;
  sp.end = p.prefix_len + p.group_len;
  sp.bt = p.block_tables + (size_t)s0 * p.bt_stride + (sp.start >> 4);
  sp.part = p.prefix_parts;
  sp.rot = 0;
  int32_t* tr = nullptr;
  if constexpr (TRACE)
    tr = p.trace_group + ((size_t)k * p.num_kv_heads + g) * p.group_trace_tiles * 3;
  span_body<G, TRACE>(p, g, sp, smem, tr);
}

}  // namespace shared
}  // namespace pa
