// Causal attention of a chunk of new tokens over its sequence's paged context
// (extend / chunked prefill) on 32x32 MFMA tiles (gfx950, head_dim 128).
//
// For KV head g, the (chunk token i, head j) pairs of sequence b form rows
// R = i*G + j; row R sees the tokens 0 .. n - L + i (n: context with the chunk,
// L: chunk length).  One workgroup owns kExtendRowsPerWg rows, 32 per
// wavefront, and streams the sequence's blocks once through LDS for all of
// them, a stage of two blocks (32 tokens) at a time: each wavefront loads one
// quarter (four token rows of K and of V) of each block into registers one
// stage ahead and publishes it to LDS.  The stream stops at the workgroup's
// last visible token; rows past it are read as zeros (buffer bounds).
//
// Lanes: h = lane >> 5, n = lane & 31.  v_mfma_f32_32x32x16_bf16 takes A row n
// / B column n at contraction indices 8h .. 8h+7 and leaves in register r of
// its result row 8(r/4) + 4h + r%4 of column n.
//  * S^T = K Q^T: A = K rows (token i of the stage in row i, dims 16s + 8h ..
//    in step s), B = Q^T with query row n of the wavefront in column n.  Lane
//    (h, n) receives the scores of tokens 8a + 4h + b (register 4a + b).
//  * O += P V: for block m of the stage the contraction index k = 8h + e
//    stands for token 16m + 8(e/4) + 4h + e%4, which makes the scores above
//    exactly the A operand (P never moves between lanes); the B operand comes
//    from the staged V through transposing reads (ds_read_b64_tr_b16: lane i
//    of a 16-lane group receives element i%4 of the 8-byte chunks addressed by
//    lanes 4k + i/4 of its group, k = 0..3).  Each probability reaches the
//    matrix core as a bf16 pair, high part and rounded remainder (about 2^-17
//    relative), two MFMAs per PV step; the row sum adds the fp32 values.
//
// What bounds it.  On this card a 16x16x32 MFMA keeps the VALU port of its
// SIMD from the other wavefront for about 8 of its 16 cycles, a 32x32x16 one
// for about 10 of its 32, so the larger tile leaves the softmax room: 24
// MFMAs and about 115 VALU instructions per wavefront and stage.  The prefill
// of 93 sequences (55k chunk tokens over 2.4k-3.3k contexts, four heads per KV
// head) takes 20% fewer cycles than with 16x16 tiles and the unpipelined loop
// (5.2e7 against 6.6e7 GPU cycles summed over the XCDs; 3.52 -> 3.18-3.35 ms, 660
// -> 694-732 TFLOP/s of causal flops, 1.5 times that on the matrix cores), and runs
// at 1.99 instead of 2.35 GHz, drawing 1.36 kW either way: the card's 1.4 kW limit
// holds it (a 16384^3 library matrix product reaches 1340-1350 TFLOP/s here, at 1.82
// GHz and 1.37 kW).  Two tiles per wavefront at one
// wavefront per SIMD, which halve the LDS reads, measured 4.5 ms; the low
// parts formed by v_dot2 instead of unpack and subtract 3.32 against 3.15 ms;
// raised priority during the MFMAs 3.21 against 3.15 ms.
//
// The loop is software-pipelined by one stage: iteration j computes the scores
// of stage j+1, the probabilities of stage j and their PV, all in one
// straight-line block, then tests the running max for stage j+1 (the only
// branch: lazy rescale, rare).
#pragma once

#include "kernels.h"
#include "mfma_body.h"
#include "pa_device.h"
#include "shared_body.h"

namespace pa {
namespace extend {

using mfma::bf16x8_t;
using mfma::floatx16_t;
using mfma::kWaves;
using mfma::lds_short4_t;
using mfma::lds_u32x4_t;
using mfma::pack_bf16;
using mfma::u32x4_t;
using shared::k_off;     // K rows of a stage; lane (h, n) reads row n, chunk 2s + h
using shared::per_row;
using shared::raise_max;

typedef int i32x2_t __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) i32x2_t lds_i32x2_t;

constexpr int kD = 128;
constexpr int kRows = 32;                          // query rows per wavefront
static_assert(kRows * kWaves == kExtendRowsPerWg, "one 32-row tile per wavefront");
constexpr int kTokens = 32;                        // per stage: two blocks
constexpr int kSlots = 3;                          // LDS stages: one written, K of one and V of one read
constexpr int kStageBytes = 2 * kTokens * kD * 2;  // K rows, then V rows
constexpr int kVOffset = kTokens * kD * 2;
constexpr int kIdOffset = kSlots * kStageBytes;    // block ids
constexpr int kRowOffset = kIdOffset + kExtendMaxTokens / 16 * 4;   // one value per row, per wavefront
constexpr int kLdsBytes = kRowOffset + kWaves * kRows * 4;

template <bool B> struct BoolTag { static constexpr bool value = B; };

// LDS byte offset of 16-byte chunk c of token row r in a staged V tile: eight
// 32-byte windows (dims 16w .. 16w+15) per row, window w at position
// w ^ 2(r % 4).  The transposing reads of a half wavefront take windows 2j and
// 2j+1 of four consecutive rows: eight different positions, all 64 banks.
__device__ __forceinline__ int v_off(int r, int c) {
  return r * (2 * kD) + (((c >> 1) ^ ((r & 3) << 1)) << 5) + ((c & 1) << 4);
}

// Sequence b's chunk: its first row in q and out, its length, and the
// position of its first token.  Device data, clamped into the buffers.
struct Chunk {
  int start, len, first;
};
__device__ __forceinline__ Chunk chunk_of(const ExtendParams& p, int b) {
  int ctx = p.context_lens[b];
  ctx = ctx < 0 ? 0 : (ctx > p.max_ctx ? p.max_ctx : ctx);
  int qs = p.q_start[b];
  int L = p.q_start[b + 1] - qs;
  qs = qs < 0 ? 0 : qs;
  L = L < 0 ? 0 : (L > ctx ? ctx : (L > p.max_chunk ? p.max_chunk : L));
  L = qs + L > p.total_q ? (p.total_q > qs ? p.total_q - qs : 0) : L;
  return {qs, L, ctx - L};
}

template <int G>
__device__ __forceinline__ void extend_body(const ExtendParams& p, int wg_index, lds_u8_t* smem) {
  const int lane = threadIdx.x & 63;
  const int wave = wave_uniform(threadIdx.x >> 6);
  const int h = lane >> 5;
  const int n = lane & 31;

  int wg = wg_index;
  const int g = wg % p.num_kv_heads;
  wg /= p.num_kv_heads;
  const int grp = wg % p.groups;
  const int b = wg / p.groups;

  const Chunk c = chunk_of(p, b);
  const int rows = c.len * G;
  if (grp * kExtendRowsPerWg >= rows) return;            // whole workgroup: no rows here
  const int row0 = grp * kExtendRowsPerWg + kRows * wave;   // this wavefront's first row
  const int first = c.first;
  const int qs = c.start;

  // Tokens the workgroup needs: up to its last row's position.
  const int last_row = min(rows, (grp + 1) * kExtendRowsPerWg) - 1;
  const int vis_max = first + last_row / G + 1;
  const int nblk = (vis_max + 15) >> 4;

  // Block ids of the stream, clamped into the pool, staged once in LDS (at
  // most kExtendMaxTokens / 16 of them).
  lds_i32_t* ids = reinterpret_cast<lds_i32_t*>(smem + kIdOffset);
  {
    const int32_t* bt = p.block_tables + (size_t)b * p.bt_stride;
    for (int j = threadIdx.x; j < nblk + (nblk & 1); j += 64 * kWaves)   // whole pairs
      ids[j] = j < nblk ? min(max(bt[j], 0), p.num_blocks - 1) : 0;
    __syncthreads();
  }

  // Column n is row R = row0 + n: chunk token R / G, query head g*G + R % G.
  // A negative scale goes into the sign of Q (bf16 negation is exact, and so
  // is the negation of every score).
  const uint32_t qflip = p.scale_log2 < 0.f ? 0x80008000u : 0u;
  const float scale = fabsf(p.scale_log2);
  u32x4_t qb[8];
  int lim;   // tokens column n sees
  {
    const int R = row0 + n;
    const bool ok = R < rows;
    const int i = ok ? R / G : 0;
    const uint16_t* qrow = p.q + ((size_t)(qs + i) * p.num_q_heads + g * G + R % G) * kD;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const uint4 w = ok ? *reinterpret_cast<const uint4*>(qrow + (2 * s + h) * 8) : make_uint4(0, 0, 0, 0);
      qb[s] = u32x4_t{w.x ^ qflip, w.y ^ qflip, w.z ^ qflip, w.w ^ qflip};
    }
    lim = ok ? first + i + 1 : 0;
  }

  constexpr size_t kTileElems = 16 * kD;
  const size_t blk_stride = (size_t)p.num_kv_heads * kTileElems;
  const uint16_t* kbase = p.k_pool + (size_t)g * kTileElems;
  const uint16_t* vbase = p.v_pool + (size_t)g * kTileElems;
  // This wavefront's quarter of a block: token row 4*wave + lane / 16, chunk lane % 16.
  const int srow = 4 * wave + (lane >> 4);
  const int schunk = lane & 15;
  const int share_off = (srow * kD + schunk * 8) * 2;
  u32x4_t rk[2], rv[2];
  // Block ids of stage j (read from LDS a stage before they are needed);
  // stages past the stream repeat its last pair and load nothing.
  const int npair = (nblk + 1) >> 1;
  auto stage_ids = [&](int j) { return *reinterpret_cast<const lds_i32x2_t*>(ids + 2 * min(j, npair - 1)); };
  auto load = [&](int j, i32x2_t id2) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int bytes = wave_uniform(max(0, min(16, vis_max - 16 * (2 * j + e))) * (kD * 2));
      const size_t id = (size_t)__builtin_amdgcn_readfirstlane(id2[e]);
      const __amdgpu_buffer_rsrc_t dk = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<uint16_t*>(kbase + id * blk_stride), 0, bytes, kBufferDescWord3);
      const __amdgpu_buffer_rsrc_t dv = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<uint16_t*>(vbase + id * blk_stride), 0, bytes, kBufferDescWord3);
      rk[e] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(dk, share_off, 0, 0));
      rv[e] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(dv, share_off, 0, 0));
    }
  };
  const int wk = k_off(srow, schunk);       // + 16 rows for the stage's second block
  const int wv = v_off(srow, schunk);
  auto publish = [&](int slot) {
    lds_u8_t* st = smem + slot * kStageBytes;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      *reinterpret_cast<lds_u32x4_t*>(st + e * 16 * kD * 2 + wk) = rk[e];
      *reinterpret_cast<lds_u32x4_t*>(st + kVOffset + e * 16 * kD * 2 + wv) = rv[e];
    }
  };

  // Scores of the stage in `slot`.
  int ka[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) ka[s] = k_off(n, 2 * s + h);
  auto scores = [&](int slot) {
    const lds_u8_t* st = smem + slot * kStageBytes;
    floatx16_t a;
#pragma unroll
    for (int i = 0; i < 16; ++i) a[i] = 0.f;
#pragma unroll
    for (int s = 0; s < 8; ++s)
      a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
          __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const lds_u32x4_t*>(st + ka[s])),
          __builtin_bit_cast(bf16x8_t, qb[s]), a, 0, 0, 0);
    return a;
  };
  // Transposing reads: lane i = lane % 16 of group (h, f = bit 4 of lane)
  // addresses row 4h + i/4 (+ 8, + 16m), dims 32j + 16f + 4(i%4) .. +3.
  const int vr = 4 * h + ((lane & 15) >> 2);
  const int vf = (lane >> 4) & 1;
  int va[2][4];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      va[u][j] = kVOffset + v_off(vr + 8 * u, 2 * (2 * j + vf)) + ((lane & 3) << 3);

  float m = -__builtin_inff(), neg = 0.f, l = 0.f;
  floatx16_t o[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[j][i] = 0.f;

  lds_f32_t* rowv = reinterpret_cast<lds_f32_t*>(smem + kRowOffset) + wave * kRows;

  // Running-max test of a stage whose first token is t0, before its
  // probabilities are formed.
  auto raise = [&](auto tail, const floatx16_t& a, int t0) {
    constexpr bool TAIL = decltype(tail)::value;
    float mx = -__builtin_inff();   // the lane's largest unmasked raw score
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (!TAIL || t0 + 8 * (r >> 2) + 4 * h + (r & 3) < lim) mx = fmaxf(mx, a[r]);
    // NaN (no rescale) when all are masked and the scale is 0
    raise_max(mx * scale, m, neg, l, o, rowv, h, n);
  };

  // Probabilities of stage j (raw scores a, first token t0) and their PV.
  auto attend = [&](auto tail, const floatx16_t& a, int t0, int slot) {
    constexpr bool TAIL = decltype(tail)::value;
    u32x4_t hi[2], lo[2];
    float sum[2];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        float pf[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int r = 8 * mb + e + i;     // token 16mb + 8((e+i)/4) + 4h + (e+i)%4
          float ex = fmaf(a[r], scale, neg);
          if (TAIL && t0 + 8 * (r >> 2) + 4 * h + (r & 3) >= lim) ex = -__builtin_inff();
          pf[i] = fast_exp2(ex);
        }
        hi[mb][e / 2] = pack_bf16(pf[0], pf[1]);
        lo[mb][e / 2] = pack_bf16(pf[0] - bf16_lo(hi[mb][e / 2]), pf[1] - bf16_hi(hi[mb][e / 2]));
        const float s2 = pf[0] + pf[1];
        sum[mb] = e == 0 ? s2 : sum[mb] + s2;
      }
    }
    l += sum[0] + sum[1];
    const lds_u8_t* st = smem + slot * kStageBytes;
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
      u32x4_t vb[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint2 b0 = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                                       (lds_short4_t*)(st + mb * 16 * kD * 2 + va[0][j])));
        const uint2 b1 = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                                       (lds_short4_t*)(st + mb * 16 * kD * 2 + va[1][j])));
        vb[j] = u32x4_t{b0.x, b0.y, b1.x, b1.y};
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
  };

  const int nit = (nblk + 1) >> 1;
  // Stages wholly visible to every row of the workgroup (its first row sees
  // the fewest tokens) need no masks.
  const int min_lim = min(first + grp * kExtendRowsPerWg / G + 1, vis_max);
  const int nvis = min(min_lim / kTokens, nit);

  // Stages 0 and 1 into LDS, stage 2 into registers.
  load(0, stage_ids(0));
  publish(0);
  load(1, stage_ids(1));
  publish(1);
  load(2, stage_ids(2));
  i32x2_t idn = stage_ids(3);
  __syncthreads();
  floatx16_t s = scores(0);
  raise(BoolTag<true>{}, s, 0);

  // Iteration j: stage j+2 from the registers to its slot, stage j+3 into the
  // registers, the scores of stage j+1, the probabilities and PV of stage j.
  // Every slot is read only between the barriers that follow its writing and
  // precede its next writing: iteration j reads K of slot j+1 and V of slot j
  // and writes slot j+2 (modulo 3).
  auto stream = [&](auto tail, int jb, int je) {
    for (int j0 = jb; j0 < je; j0 += kSlots) {
#pragma unroll
      for (int u = 0; u < kSlots; ++u) {
        const int j = j0 + u;
        if (j < je) {                                // uniform over the workgroup
          const floatx16_t next = scores((u + 1) % kSlots);
          publish((u + 2) % kSlots);
          load(j + 3, idn);
          idn = stage_ids(j + 4);
          attend(tail, s, j * kTokens, u);
          if (j + 1 < nit) raise(tail, next, (j + 1) * kTokens);
          s = next;
          __syncthreads();
        }
      }
    }
  };
  // The unmasked loop also tests stage j+1 unmasked; it runs whole rounds of
  // slots, so that both loops find stage j in slot j % 3.
  const int nfast = max(nvis - 1, 0) / kSlots * kSlots;
  stream(BoolTag<false>{}, 0, nfast);
  stream(BoolTag<true>{}, nfast, nit);

  // Normalise, transpose through LDS (the stages are free: every wavefront is
  // past the last barrier) and write bf16 rows in 16-byte pieces.
  float lx = l, ly = l;
  swap32(lx, ly);
  const float lcol = lx + ly;
  float inv[16];
  per_row(rowv, h, n, lcol > 0.f ? 1.0f / lcol : 0.f, inv);
  lds_u8_t* tile = smem + wave * (kRows * kD * 2);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = 8 * (r >> 2) + 4 * h + (r & 3);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      *reinterpret_cast<__attribute__((address_space(3))) uint16_t*>(tile + row * (kD * 2) + (32 * j + n) * 2) =
          (uint16_t)bf16_rne(o[j][r] * inv[r]);
  }
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int row = 4 * i + (lane >> 4);
    const int R = row0 + row;
    const u32x4_t x = *reinterpret_cast<const lds_u32x4_t*>(tile + row * (kD * 2) + (lane & 15) * 16);
    if (R < rows)
      *reinterpret_cast<u32x4_t*>(p.out + ((size_t)(qs + R / G) * p.num_q_heads + g * G + R % G) * kD +
                                  (lane & 15) * 8) = x;
  }
}

// The form for small grids: 32 rows per workgroup with the tokens split over
// the wavefronts (shared_body.h), a chain four times shorter per workgroup.
constexpr int kSplitIdOffset = shared::kLdsBytes;
constexpr int kSplitLdsBytes = kSplitIdOffset + kExtendMaxTokens / 16 * 4;

template <int G>
__device__ __forceinline__ void extend_split_body(const ExtendParams& p, int wg_index, lds_u8_t* smem) {
  constexpr int kTile = shared::kRows;
  const int n = threadIdx.x & 31;
  int wg = wg_index;
  const int g = wg % p.num_kv_heads;
  wg /= p.num_kv_heads;
  const int tile = wg % p.groups;
  const int b = wg / p.groups;
  const Chunk c = chunk_of(p, b);
  const int rows = c.len * G;
  const int row0 = tile * kTile;
  if (row0 >= rows) return;                                // whole workgroup: no rows here
  const int vis_max = c.first + (min(rows, row0 + kTile) - 1) / G + 1;   // tokens the tile needs
  const int nblk = (vis_max + 15) >> 4;

  lds_i32_t* ids = reinterpret_cast<lds_i32_t*>(smem + kSplitIdOffset);
  {
    const int32_t* bt = p.block_tables + (size_t)b * p.bt_stride;
    for (int j = threadIdx.x; j < nblk; j += 64 * kWaves)
      ids[j] = min(max(bt[j], 0), p.num_blocks - 1);
    __syncthreads();
  }

  // A column without a row repeats the tile's first, sees everything and is
  // not written.
  const bool has_row = row0 + n < rows;
  const int R = has_row ? row0 + n : row0;
  const int lim = has_row ? c.first + R / G + 1 : 0x7fffffff;
  constexpr size_t kTileElems = 16 * kD;
  const size_t blk_stride = (size_t)p.num_kv_heads * kTileElems;
  shared::tile_core(
      p.q + ((size_t)(c.start + R / G) * p.num_q_heads + g * G + R % G) * kD, p.k_pool + (size_t)g * kTileElems,
      p.v_pool + (size_t)g * kTileElems, nblk, p.scale_log2, smem,
      [&](const uint16_t* base, int i) {   // rows past the last visible token are read as zeros
        const size_t id = (size_t)__builtin_amdgcn_readfirstlane(ids[i]);
        const int bytes = wave_uniform(min(16, vis_max - 16 * i) * (kD * 2));
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base + id * blk_stride), 0, bytes,
                                                 kBufferDescWord3);
      },
      [&](int i) { return lim - 16 * i; }, [](int) {}, [](float, float) {},
      [&](int r, int col, const mfma::floatx4_t& acc) {
        const int row = row0 + r;
        if (row < rows)
          *reinterpret_cast<uint2*>(p.out + ((size_t)(c.start + row / G) * p.num_q_heads + g * G + row % G) * kD +
                                    4 * col) =
              make_uint2(bf16_rne(acc[0]) | (bf16_rne(acc[1]) << 16), bf16_rne(acc[2]) | (bf16_rne(acc[3]) << 16));
      });
}

}  // namespace extend
}  // namespace pa
