// Split-KV paged decode attention on MFMA tiles (gfx950): head_dim 64 or 128,
// four or eight query heads per KV head.
//
// One workgroup handles one work item (partition p, sequence b, KV head g):
// the G query heads g*G .. g*G+G-1 that share KV head g attend to the tokens
// [p*S, min((p+1)*S, ctx_b)) of sequence b.  Its wavefronts take the
// partition's 16-token KV blocks round-robin, each keeping its own
// online-softmax state, and merge through LDS at the end.  Each wavefront
// keeps NBUF tiles in a register ring, so the next NBUF-1 blocks stream in
// while one is being computed.
//
//  * Both tiles of a block are read from the pool in row order: each 16-lane
//    group takes one whole token row, so a load instruction reads four whole
//    rows of contiguous memory and the vector L1 sees one access per 64
//    bytes.  (Reading the MFMA operand layout straight from the pool would
//    put 16 different rows in every 16-lane group, about one L1 access per
//    lane, and the L1 becomes the limit when the tiles come from L2.)  Lane
//    (q, n) = (lane >> 4, lane & 15) then holds tokens 4u+q (u = 0..3), dims
//    (D/16)*n .. of both tiles.
//  * S^T = K Q^T with v_mfma_f32_16x16x32_bf16: A = K rows (16 tokens x 32
//    dims per instruction) read back from an LDS copy of the K tile
//    (stage_off: XOR-swizzled rows, so writes and reads spread over the
//    banks); B = Q^T with query row n % G in column n.  A row i is token
//    4(i%4) + i/4, so lane (q, n) receives the scores of tokens 4r+q
//    (r = 0..3) for query row n % G.
//  * O += P V with v_mfma_f32_16x16x16bf16_1k, one per D/16 output dims: the
//    contraction index k = 4q+e stands for token 4e+q, which makes the
//    scores above exactly the A operand (P never moves between lanes), and
//    output column n of instruction j is dim (D/16)*n + j, which makes the B
//    operand V[token 4e+q][dim (D/16)*n + j] element j of the lane's own V
//    registers (two v_perm_b32 per instruction; V never goes through LDS).
//  * Each probability reaches the matrix core as a bf16 pair p = hi + lo,
//    hi = bf16(p), lo = bf16(p - hi) (the difference is exact in fp32), which
//    carries it to about 2^-17 relative; the row sum adds the fp32 values.
//    The 16 columns hold only G query rows, so both parts ride in one MFMA:
//    columns with bit G of n clear carry the high parts (O rows 0 .. G-1),
//    those with it set the low parts (O rows G .. 2G-1), and the two are
//    added once, at the end.  (With G = 4, columns 8..15 repeat columns 0..7.)
//
// Measured against the kernels this one took the place of (VALU dot products
// for G = 4 and for D = 64, two MFMAs per PV step for G = 8 at D = 128; whole
// step, one MI355X): 64 sequences over a shared 2048-token prefix without the
// cascade 70 -> 42.6 us, 48 sequences of 61..4093 tokens at D = 64 40.7 -> 28.2
// us, 4 of 100..300 tokens 6.8 -> 4.8 us, 256 of 64..8192 tokens 239 -> 237
// us (6.6 TB/s, what the same tiles take without arithmetic).  The VALU form
// issued about 250 instructions per block, this one about 100.
//
// The online softmax keeps one running max per query row, replicated over its
// lanes, and rescales the accumulator only when a block raises the max by
// more than kLazyRescale (log2 units): probabilities stay <= 2^8, the rescale
// branch is wave-uniform and rare.  The scale is applied inside the exponent's
// FMA; a negative scale rides on the sign of Q.  Tail rows are removed by
// select (probability 0, V zero), so stale or NaN data past the context never
// reaches the result.
#pragma once

#include "kernels.h"
#include "mfma_body.h"
#include "pa_device.h"

namespace pa {
namespace decode {

using mfma::bf16x8_t;
using mfma::column_value;
using mfma::floatx2_t;
using mfma::floatx4_t;
using mfma::k_arow;
using mfma::kLazyRescale;
using mfma::kWaves;
using mfma::lds_floatx2_t;
using mfma::lds_floatx4_t;
using mfma::lds_u32x4_t;
using mfma::pack_bf16;
using mfma::short4_t;
using mfma::u32x4_t;

typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) u32x2_t lds_u32x2_t;

// Tile ring of a wavefront: D / 32 dwords per lane and token row.
template <int D>
struct KvTile {
  static constexpr int VW = D / 32;
  uint32_t k[4][VW];   // [u]: token 4u+q, dims (D/16)*n ..
  uint32_t v[4][VW];
};

// Dims (D/16)*n .. of token rows 4u+q of one K or V tile, through a buffer
// descriptor built from the wave-uniform tile address (scalar registers) and
// the lane's fixed byte offset: no per-tile vector address math, and the
// descriptor bounds every access to the tile.  `bytes` = 0 turns the loads
// into no-ops that return zeros but still count as issued, so every path
// through the prefetch ring issues the same loads.  AUX: the loads' cache
// policy (kLoadDefault or kLoadStreaming).
template <int D, int AUX>
__device__ __forceinline__ void load_rows(uint32_t (&dst)[4][D / 32], const uint16_t* tile,
                                          uint32_t lane_off, int bytes) {
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(tile), 0, bytes, kBufferDescWord3);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int off = (int)lane_off + u * 4 * D * 2;
    if constexpr (D == 128) {
      const auto x = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, AUX);
      dst[u][0] = x[0]; dst[u][1] = x[1]; dst[u][2] = x[2]; dst[u][3] = x[3];
    } else {
      const auto x = __builtin_amdgcn_raw_buffer_load_b64(rsrc, off, 0, AUX);
      dst[u][0] = x[0]; dst[u][1] = x[1];
    }
  }
}

// LDS byte offset of 16-byte chunk c of token row r in a staged K tile: rows
// of 2D bytes, chunk c at position c ^ swz(r).  Writers fill whole rows;
// A-operand readers (lane (q, n): row k_arow(n), chunk 4s+q) touch distinct
// positions within every eight consecutive lanes.  At D = 64 a row has eight
// chunks and spans all 32 banks once, so swz takes eight values: the rows
// k_arow(0..7) = 0, 4, 8, 12, 1, 5, 9, 13 (and those of lanes 8..15) map to
// eight different ones.
template <int D>
__device__ __forceinline__ int stage_off(int r, int c) {
  if constexpr (D == 128) return mfma::k_stage(r, c);
  return r * (2 * D) + ((c ^ ((r >> 2) | ((r & 1) << 2))) << 4);
}

// Softmax state of the wavefront's G query rows and its share of the output.
template <int D>
struct WaveState {
  float m;                 // running max of query row n % G (log2 units)
  float neg;               // -m, or 0 while m is -inf
  float l;                 // this lane's share of the row sum (tokens 4r+q of each block)
  floatx4_t o[D / 16];     // [j]: O[rows 4q+r][dim (D/16)*n + j]
};

// One 16-token block.  valid: tokens of the block that exist (TAIL: fewer
// than 16 may); lo: 1 in the columns that carry the low parts, else 0.
template <int D, int G, bool TAIL>
__device__ __forceinline__ void process_tile(WaveState<D>& S, const KvTile<D>& T, const uint4 (&qb)[D / 32],
                                             lds_u8_t* stage, int valid, int q, int n, float lo,
                                             float scale_log2) {
  constexpr int VW = D / 32;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    if constexpr (D == 128) {
      *reinterpret_cast<lds_u32x4_t*>(stage + stage_off<D>(4 * u + q, n)) =
          u32x4_t{T.k[u][0], T.k[u][1], T.k[u][2], T.k[u][3]};
    } else {
      *reinterpret_cast<lds_u32x2_t*>(stage + stage_off<D>(4 * u + q, n >> 1) + ((n & 1) << 3)) =
          u32x2_t{T.k[u][0], T.k[u][1]};
    }
  }
  u32x4_t ka[D / 32];
#pragma unroll
  for (int s = 0; s < D / 32; ++s)
    ka[s] = *reinterpret_cast<const lds_u32x4_t*>(stage + stage_off<D>(k_arow(n), 4 * s + q));

  // Two independent accumulation chains, summed at the end.
  const floatx4_t z = {0.f, 0.f, 0.f, 0.f};
  floatx4_t st[2];
#pragma unroll
  for (int s = 0; s < D / 32; ++s)
    st[s & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, ka[s]),
                                                        __builtin_bit_cast(bf16x8_t, qb[s]),
                                                        s < 2 ? z : st[s & 1], 0, 0, 0);
  const floatx4_t raw = st[0] + st[1];

  // The rescale test needs no cross-lane reduction: any lane above its row's
  // max + kLazyRescale triggers it; only then is the block's row max formed.
  float mx = -__builtin_inff();
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (!TAIL || 4 * r + q < valid) mx = fmaxf(mx, raw[r]);
  const float xmax = mx * scale_log2;   // NaN when every token is masked and the scale is 0
  if (__builtin_amdgcn_ballot_w64(xmax > S.m + kLazyRescale) != 0) {
    const float bm = group_max4(xmax);
    const float mn = bm > S.m + kLazyRescale ? bm : S.m;
    // 1 for rows that keep their max (or have attended to nothing yet)
    const float alpha = mn == -__builtin_inff() ? 1.f : fast_exp2(S.m - mn);
    S.l *= alpha;
    // Accumulator rows are indexed by lane group: row 4q+r takes alpha of
    // column 4q+r, held by lane 4q+r.  Before the first tile it is all zeros.
    if (__builtin_amdgcn_ballot_w64(S.m != -__builtin_inff()) != 0) {
      float ar[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) ar[r] = column_value(alpha, q, r);
#pragma unroll
      for (int j = 0; j < D / 16; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) S.o[j][r] *= ar[r];
    }
    S.m = mn;
    S.neg = mn == -__builtin_inff() ? 0.f : -mn;
  }

  // Probabilities: lanes of the high columns keep bf16(p), those of the low
  // columns bf16(p - bf16(p)).
  float p[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float e = fmaf(raw[r], scale_log2, S.neg);
    if (TAIL && 4 * r + q >= valid) e = -__builtin_inff();
    p[r] = fast_exp2(e);
  }
  S.l += (p[0] + p[1]) + (p[2] + p[3]);
  const uint32_t h01 = pack_bf16(p[0], p[1]), h23 = pack_bf16(p[2], p[3]);
  const uint32_t w01 = pack_bf16(fmaf(-lo, bf16_lo(h01), p[0]), fmaf(-lo, bf16_hi(h01), p[1]));
  const uint32_t w23 = pack_bf16(fmaf(-lo, bf16_lo(h23), p[2]), fmaf(-lo, bf16_hi(h23), p[3]));
  const short4_t pa = __builtin_bit_cast(short4_t, make_uint2(w01, w23));

  // PV: instruction j takes B = V[token 4e+q][dim (D/16)*n + j], e = 0..3:
  // bf16 j of the lane's slice in each of its four rows.  Tail rows become
  // zero.
  uint32_t vw[4][VW];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int w = 0; w < VW; ++w) vw[u][w] = TAIL && 4 * u + q >= valid ? 0u : T.v[u][w];
#pragma unroll
  for (int j = 0; j < D / 16; ++j) {
    const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;
    const uint32_t b0 = __builtin_amdgcn_perm(vw[1][j >> 1], vw[0][j >> 1], sel);
    const uint32_t b1 = __builtin_amdgcn_perm(vw[3][j >> 1], vw[2][j >> 1], sel);
    S.o[j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pa, __builtin_bit_cast(short4_t, make_uint2(b0, b1)),
                                                       S.o[j], 0, 0, 0);
  }
}

// Whether a workgroup may take a second sequence's rows in the columns that
// four query heads leave idle: where sequences may share blocks.
template <int G, bool STREAM>
constexpr bool pairs() { return G == 4 && !STREAM; }

// LDS of one work item: a staged K tile per wavefront, reused by the merge
// ([wave][rows] maxima and sums, then [wave][rows][D] outputs).
template <int D, int G, bool STREAM>
constexpr int lds_bytes() {
  constexpr int rows = pairs<G, STREAM>() ? 2 * G : G;
  const int stage = kWaves * 16 * D * 2;
  const int merge = (2 * kWaves * rows + kWaves * rows * D) * 4;
  return stage > merge ? stage : merge;
}

// One work item (partition, sequence, KV head) = workgroup `wg_index`;
// `smem` points at lds_bytes<D, G, STREAM>() bytes of LDS.  STREAM: load the
// tiles as streaming data (kLoadStreaming); it changes caching, never the
// results.
//
// Pairs: with four query heads, columns 8..15 of a tile are idle.  Where blocks
// may be shared (!STREAM), the workgroups of sequences 2k and 2k+1 compare the
// partition's block ids of both; if both contexts hold the whole partition and
// every id is equal, one of them computes both sequences' rows at the cost of
// one, and the other leaves.  Columns do not affect each other, so the
// partials have the same bits either way.  (64 sequences over a shared
// 2048-token prefix, 512-token partitions, no cascade: 42.7 -> 33.6 us a step;
// with the even sequence always computing, no change: half of the shader
// engines had all the work.)
template <int D, int G, int NBUF, bool TRACE, bool STREAM, bool APPEND, bool ONE_MERGE = false>
__device__ __forceinline__ void decode_body(const DecodeParams& p, int wg_index, lds_u8_t* smem) {
  constexpr int VW = D / 32;
  constexpr int DPL = D / 16;   // dims per lane and token row
  static_assert(G == 4 || G == 8, "group size");
  static_assert(D == 64 || D == 128, "head dim");
  const int lane = threadIdx.x & 63;
  const int wave = wave_uniform(threadIdx.x >> 6);
  const int q = lane >> 4;
  const int n = lane & 15;

  int g, b, part;
  decode_item(p, wg_index, g, b, part);

  const int start = p.token_offset + part * p.part_tokens;
  const int j0 = start >> 4;
  const int h0 = g * G;
  const int32_t* bt = p.block_tables + (size_t)b * p.bt_stride + j0;
  // The first 64 block ids and the query rows are loaded before the context
  // length arrives (j0 < bt_stride for every launched partition).
  const int raw_first = lane < min(64, p.bt_stride - j0) ? bt[lane] : 0;
  constexpr bool PAIR = pairs<G, STREAM>();
  const int b2 = (b ^ 1) < p.batch ? b ^ 1 : b;   // the sequence to pair with
  int raw_second = 0;
  if constexpr (PAIR) {
    const int32_t* bt2 = p.block_tables + (size_t)b2 * p.bt_stride + j0;
    raw_second = lane < min(64, p.bt_stride - j0) ? bt2[lane] : 0;
  }

  // Q^T operand: column n holds query row n % G (PAIR: columns 8..15 those of
  // b2); dims 32s + 8q .. +8.  bf16 negation is exact, and so is the negation
  // of every score.
  const uint32_t qflip = p.scale_log2 < 0.f ? 0x80008000u : 0u;
  const float scale_abs = fabsf(p.scale_log2);
  uint4 qb[D / 32];
  {
    const int bq = PAIR && n >= 8 ? b2 : b;
    const uint16_t* qrow = p.q + ((size_t)bq * p.num_q_heads + h0 + (n & (G - 1))) * D;
#pragma unroll
    for (int s = 0; s < D / 32; ++s) {
      uint4 w = *reinterpret_cast<const uint4*>(qrow + (4 * s + q) * 8);
      w.x ^= qflip; w.y ^= qflip; w.z ^= qflip; w.w ^= qflip;
      qb[s] = w;
    }
  }

  int ctx = p.context_lens[b];
  ctx = ctx < 0 ? 0 : (ctx > p.max_ctx ? p.max_ctx : ctx);
  const bool split = p.write_partials != 0;
  if (split && start >= ctx) return;  // whole workgroup; the reduce skips this partition
  bool paired = false;
  if constexpr (PAIR) {
    // Tokens both contexts must hold; with the fused append, the new tokens
    // must lie past them.
    const int need = start + p.part_tokens + (APPEND ? 1 : 0);
    const int blocks = p.part_tokens >> 4;
    paired = split && b2 != b && blocks <= 64 && ctx >= need && min(p.context_lens[b2], p.max_ctx) >= need &&
             __builtin_amdgcn_ballot_w64(lane < blocks && raw_first != raw_second) == 0;
    // Whole workgroup: computed with sequence b2.  Which of the two computes
    // alternates, so that every shader engine of an XCD gets some of the work
    // (consecutive sequences go to them in a fixed cycle of four).
    if (paired && (b & 1) != ((b >> 2) & 1)) return;
  }
  const int end = min(ctx, start + p.part_tokens);
  const int nblk = end > start ? (end - start + 15) >> 4 : 0;

  // Fused append: block jnew of this item (-1: none) holds the new token in
  // row rnew; knew / vnew are the lane's slice of its K and V rows.  The lanes
  // of row group rnew % 4 store the rows.
  int jnew = -1, rnew = 0;
  uint32_t knew[VW], vnew[VW];
  if constexpr (APPEND) {
    if (ctx > 0 && ctx - 1 >= start && ctx - 1 < end) {
      jnew = ((ctx - 1) >> 4) - j0;
      rnew = (ctx - 1) & 15;
      const size_t src = ((size_t)b * p.num_kv_heads + g) * D + DPL * n;
#pragma unroll
      for (int w = 0; w < VW; ++w) {
        knew[w] = reinterpret_cast<const uint32_t*>(p.k_new + src)[w];
        vnew[w] = reinterpret_cast<const uint32_t*>(p.v_new + src)[w];
      }
      if (wave == 0 && q == (rnew & 3)) {
        int phys = p.block_tables[(size_t)b * p.bt_stride + ((ctx - 1) >> 4)];
        phys = min(max(phys, 0), p.num_blocks - 1);
        const size_t dst = (((size_t)phys * p.num_kv_heads + g) * 16 + rnew) * D + DPL * n;
#pragma unroll
        for (int w = 0; w < VW; ++w) {
          reinterpret_cast<uint32_t*>(p.k_pool_w + dst)[w] = knew[w];
          reinterpret_cast<uint32_t*>(p.v_pool_w + dst)[w] = vnew[w];
        }
      }
    }
  }

  // One stage per wavefront: its LDS operations execute in order, so a tile's
  // writes come after the previous tile's reads.
  lds_u8_t* stage = smem + wave * (16 * D * 2);
  const float lo = (n & G) ? 1.f : 0.f;

  WaveState<D> S;
  S.m = -__builtin_inff();
  S.neg = 0.f;
  S.l = 0.f;
#pragma unroll
  for (int j = 0; j < DPL; ++j) S.o[j] = floatx4_t{0.f, 0.f, 0.f, 0.f};

  constexpr size_t kTileElems = 16 * D;
  const size_t blk_stride = (size_t)p.num_kv_heads * kTileElems;
  const uint16_t* kbase = p.k_pool + (size_t)g * kTileElems;
  const uint16_t* vbase = p.v_pool + (size_t)g * kTileElems;
  const size_t item = ((size_t)part * p.batch + b) * p.num_kv_heads + g;
  const uint32_t lane_off = (uint32_t)(q * D + DPL * n) * 2u;   // row q (+ 4 rows per u)

  for (int c0 = 0; c0 < nblk; c0 += 64) {
    const int cn = min(64, nblk - c0);
    const int raw = c0 == 0 ? (lane < cn ? raw_first : 0) : (lane < cn ? bt[c0 + lane] : 0);
    const int idc = min(max(raw, 0), p.num_blocks - 1);

    // The item's last block (rows past the context, the appended token) is
    // processed first, masked, by the wavefront whose turn it is, so the main
    // loop over the other blocks holds one unmasked core.  Its loads are
    // issued first; blocks past the others get an empty descriptor.
    const bool last = c0 + 64 >= nblk;
    const int full = last ? cn - 1 : cn;
    const bool owns_last = last && full % kWaves == wave;
    auto load = [&](KvTile<D>& T, int i, bool ok) {
      const size_t id = (size_t)__builtin_amdgcn_readlane(idc, ok ? i : 0);
      const int bytes = ok ? (int)(kTileElems * 2) : 0;
      constexpr int kAux = STREAM ? kLoadStreaming : kLoadDefault;
      load_rows<D, kAux>(T.k, kbase + id * blk_stride, lane_off, bytes);
      load_rows<D, kAux>(T.v, vbase + id * blk_stride, lane_off, bytes);
    };
    auto trace = [&](int i, int valid) {
      if constexpr (TRACE) {
        if (lane == 0) {
          int32_t* tr = p.trace + (item * p.trace_tiles + (c0 + i)) * 3;
          tr[0] = j0 + c0 + i;
          tr[1] = __builtin_amdgcn_readlane(raw, i);
          tr[2] = valid;
          if (PAIR && paired) {   // the same tiles of sequence b2
            int32_t* tr2 = tr + (int64_t)(b2 - b) * p.num_kv_heads * p.trace_tiles * 3;
            tr2[0] = tr[0];
            tr2[1] = tr[1];
            tr2[2] = valid;
          }
        }
      }
    };

    KvTile<D> T[NBUF];
    int i = wave, ld = wave;
    load(T[NBUF - 1], full, owns_last);
#pragma unroll
    for (int s = 0; s < NBUF - 1; ++s) {
      load(T[s], ld, ld < full);
      ld += kWaves;
    }
    if (owns_last) {
      KvTile<D>& L = T[NBUF - 1];
      if constexpr (APPEND) {
        // the new token's rows replace whatever the slot held
        if (c0 + full == jnew) {
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (4 * u + q == rnew) {
#pragma unroll
              for (int w = 0; w < VW; ++w) { L.k[u][w] = knew[w]; L.v[u][w] = vnew[w]; }
            }
        }
      }
      const int valid = end - (start + (c0 + full) * 16);
      process_tile<D, G, true>(S, L, qb, stage, valid, q, n, lo, scale_abs);
      trace(full, valid);
    }
    bool done = i >= full;
    while (!done) {
#pragma unroll
      for (int s = 0; s < NBUF; ++s) {
        if (!done) {
          load(T[(s + NBUF - 1) % NBUF], ld, ld < full);
          ld += kWaves;
          process_tile<D, G, false>(S, T[s], qb, stage, 16, q, n, lo, scale_abs);
          trace(i, 16);
          i += kWaves;
          done = i >= full;
        }
      }
    }
  }

  // Add the low parts' output rows (G .. 2G-1) to the high parts' (0 .. G-1):
  // rows r and r + G sit in lane groups q and q + G/4, one lane swap apart.
  // Swapping the upper half of the dims against the lower one leaves every
  // such pair of lane groups with half the dims each.
  const float lrow = group_sum4(S.l);
  floatx4_t sum[DPL / 2];
#pragma unroll
  for (int j = 0; j < DPL / 2; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float x = S.o[j][r], y = S.o[j + DPL / 2][r];
      if constexpr (G == 8) swap32(x, y); else swap16(x, y);
      sum[j][r] = x + y;
    }
  constexpr int kMergeRows = PAIR ? 2 * G : G;
  const int half = G == 8 ? q >> 1 : q & 1;          // which half of the lane's dims
  const int qrow = G == 8 ? q & 1 : q >> 1;          // merge rows 4 * qrow + r
  const bool keeps = G == 8 || PAIR || q < 2;        // else groups 2 and 3 hold copies

  // Merge the wavefronts through LDS (the staging area is free now).
  __syncthreads();
  lds_f32_t* sm = reinterpret_cast<lds_f32_t*>(smem);       // [kWaves][rows]
  lds_f32_t* sl = sm + kWaves * kMergeRows;                  // [kWaves][rows]
  lds_f32_t* sacc = sl + kWaves * kMergeRows;                // [kWaves][rows][D]
  if (q == 0 && (n & 7) < G && (PAIR || n < 8)) {
    const int r = PAIR && n >= 8 ? n - 8 + G : n;
    sm[wave * kMergeRows + r] = S.m;
    sl[wave * kMergeRows + r] = lrow;
  }
  if (keeps) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      lds_f32_t* row = sacc + (wave * kMergeRows + 4 * qrow + r) * D + DPL * n + (DPL / 2) * half;
      if constexpr (D == 128) {
        *reinterpret_cast<lds_floatx4_t*>(row) = floatx4_t{sum[0][r], sum[1][r], sum[2][r], sum[3][r]};
      } else {
        row[0] = sum[0][r];
        row[1] = sum[1][r];
      }
    }
  }
  __syncthreads();

  // Two output dims of a row per thread, so that one store instruction writes
  // whole partial rows (512 bytes of one row at D = 128; four dims per thread
  // cost the 8K-32K-token step 0.6%).  All wavefronts merge, a few rows each:
  // against one wavefront merging every row, one long sequence's step takes
  // 25.1 instead of 26.4 us and a one-KV-head batch's 55.4 instead of 57.1 us.
  // ONE_MERGE has wavefront 0 do it (decode_mfma.hip, one_merge).
  constexpr int kMergeWaves = ONE_MERGE ? 1 : kWaves;
  constexpr int kRowThreads = D / 2;
  constexpr int kRowsPerPass = 64 * kMergeWaves / kRowThreads;
  const int d = 2 * (threadIdx.x % kRowThreads);
  const int rows = PAIR && paired ? 2 * G : G;
  if (wave >= kMergeWaves) return;
#pragma unroll
  for (int r0 = 0; r0 < kMergeRows; r0 += kRowsPerPass) {
    const int r = r0 + threadIdx.x / kRowThreads;
    if (r >= rows) return;
    float mx = sm[r];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) mx = fmaxf(mx, sm[w * kMergeRows + r]);
    const float mref = (mx == -__builtin_inff()) ? 0.f : mx;
    float lt = 0.f, o0 = 0.f, o1 = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float f = fast_exp2(sm[w * kMergeRows + r] - mref);
      lt = fmaf(sl[w * kMergeRows + r], f, lt);
      const floatx2_t a = *reinterpret_cast<const lds_floatx2_t*>(sacc + (w * kMergeRows + r) * D + d);
      o0 = fmaf(a[0], f, o0);
      o1 = fmaf(a[1], f, o1);
    }
    const float inv = lt > 0.f ? 1.0f / lt : 0.f;
    const size_t orow = (size_t)(PAIR && r >= G ? b2 : b) * p.num_q_heads + h0 + r % G;
    if (!split) {
      *reinterpret_cast<uint32_t*>(p.out + orow * D + d) = bf16_rne(o0 * inv) | (bf16_rne(o1 * inv) << 16);
    } else {
      const size_t row = orow * p.part_stride + p.part_offset + part;
      store_partial2(p.part_o + row * D + d, o0 * inv, o1 * inv);
      if (d == 0) p.part_lse[row] = lt > 0.f ? (mx + log2f(lt)) * kLn2 : -__builtin_inff();
    }
  }
}

}  // namespace decode
}  // namespace pa
