// Attention of many query rows over a token span that they share, on 16x16
// MFMA tiles (gfx950, head_dim 128): the form for grids that fill the GPU.
//
// For KV head g the rows are (sequence, head) pairs: row R of the span is
// sequence seq0 + R / G, head g*G + R % G.  One workgroup owns
// kSharedRowsPerWg rows, 16 per wavefront, and one partition of the span; its
// wavefronts share every block through LDS, so a block crosses from L2 to the
// CU once per 64 rows.  shared_body.h holds the other form, 32 rows per
// workgroup with the tokens split over the wavefronts: a chain four times
// shorter, and twice the workgroups and reads.
//
// The online softmax keeps one running max per query row, replicated over the
// four lane groups, and rescales the accumulator only when a stage raises the
// max by more than kLazyRescale (log2 units): probabilities stay <= 2^8, the
// rescale branch is wave-uniform and rare.  Each probability reaches the
// matrix core as a bf16 pair (high part and the rounded remainder, two MFMAs
// per PV step), which carries it to about 2^-17 relative; the row sum adds the
// fp32 values.
#pragma once

#include "kernels.h"
#include "mfma_body.h"
#include "pa_device.h"

namespace pa {
namespace mfma {

constexpr int kD = 128;

// Online-softmax state of the wavefront's 16 query columns.
struct MfmaState {
  float m;            // running max of query column n (log2 units), same in all groups
  float neg;          // -m, or 0 while m is -inf
  float l;            // this lane's share of the column sum (tokens 4q..4q+3 of each block)
  floatx4_t o[8];     // [j]: O[rows 4q+r][dim 16j + n]
};

// Window position of row r in a staged V tile: v_swz(r) = (r ^ r/4) & 7.
// A transposing read of one window serves each group of 16 lanes from rows
// q, q+4, q+8, q+12, and v_swz puts those four rows at window positions
// that differ modulo 4, i.e. on four different sets of eight banks (a 32-byte
// window covers 8 of the 32 four-byte banks, and windows w and w+4 share
// them): each group's read is free of bank conflicts.
__device__ __forceinline__ int v_swz(int r) { return (r ^ (r >> 2)) & 7; }

// LDS byte offset of 16-byte chunk c (dims 8c .. 8c+7) of token row r in a
// staged V tile: rows of 256 bytes, each of eight 32-byte windows (dims
// 16w .. 16w+15) at window position w ^ v_swz(r).  Writers (16 lanes per
// row) fill whole rows.
__device__ __forceinline__ int v_stage(int r, int c) {
  return r * 256 + ((((c >> 1) ^ v_swz(r)) << 5) | ((c & 1) << 4));
}

// Lane (q, n)'s address in a staged V tile for the transposing read of
// window 0 (XOR j << 5 for window j): row q + 4(n/4), dims 4(n%4) .. +3.  The
// read hands lane n of group q element n%4 of the rows addressed by lanes
// 4k + n/4 of its group, i.e. V[token q + 4k][dim 16j + n] for k = 0..3.
__device__ __forceinline__ int v_tr(int q, int n) {
  const int r = q + 4 * (n >> 2);
  return r * 256 + (v_swz(r) << 5) + ((n & 3) << 3);
}

// One staged block in the shared-span pass: its K tile (k_stage layout) then
// its V tile (v_stage layout).
constexpr int kPrefixKBytes = 16 * kKPitch;
constexpr int kPrefixStageBytes = kPrefixKBytes + 16 * kD * 2;
// The pass streams its blocks in pairs (one LDS stage and one barrier per
// pair) through a ring of kPrefixRing quarter-blocks: the first pair is loaded
// before the loop and each pair's successor while it is published.
constexpr int kPrefixStageBlocks = 2;
constexpr int kPrefixRing = 4;
static_assert(kPrefixRing == 2 * kPrefixStageBlocks, "two pairs of slots");

// NB 16-token blocks (NB even) staged at st + b * kPrefixStageBytes (K in the
// k_stage layout, V in the v_stage layout) against the wavefront's columns.  The
// QK^T of every block comes first (independent MFMA chains); lane (q, n)
// then holds the scores of tokens 4r+q of each block for column n, and one
// online-softmax step covers all NB*16 tokens.  For PV, blocks 2p and 2p+1
// form the contraction index k = 8q + e (token 4e+q of block 2p for e < 4,
// token 4(e-4)+q of block 2p+1 for e >= 4), so the lane's eight
// probabilities are exactly the A operand of one v_mfma_f32_16x16x32_bf16
// per 16 output dims (output column n = dim 16j + n), whose B operand two
// transposing LDS reads deliver straight from the staged V tiles (vtr is
// the lane's v_tr offset).  valid[b]: rows of block b that hold tokens of the
// span (0: an empty block); lim[b]: rows of block b that column n
// may see.  Rows past valid[b] are zeroed in the B operand (their V may be
// anything, NaN included).  scale_log2 >= 0: the scale is applied inside the
// exponent's FMA, and the running-max test uses the lane's largest unmasked
// raw score times the scale (the same value as the largest scaled score,
// since multiplying by a non-negative number keeps the order).
template <bool TAIL, int NB>
__device__ __forceinline__ void tile_core_nb(MfmaState& S, const lds_u8_t* st, int vtr, const uint4 (&qb)[4],
                                             const int (&valid)[NB], const int (&lim)[NB], int q, int n,
                                             float scale_log2) {
  static_assert(NB % 2 == 0, "blocks go in pairs through the PV contraction");
  const floatx4_t z = {0.f, 0.f, 0.f, 0.f};
  // K operands of every block first, then the score MFMAs interleaved over the
  // blocks so that consecutive MFMAs do not depend on each other.
  u32x4_t ka[NB][4];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int c = 0; c < 4; ++c)
      ka[b][c] = *reinterpret_cast<const lds_u32x4_t*>(st + b * kPrefixStageBytes + k_stage(k_arow(n), 4 * c + q));
  __builtin_amdgcn_s_setprio(1);
  floatx4_t a[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b)
    a[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, ka[b][0]),
                                                   __builtin_bit_cast(bf16x8_t, qb[0]), z, 0, 0, 0);
#pragma unroll
  for (int c = 1; c < 4; ++c)
#pragma unroll
    for (int b = 0; b < NB; ++b)
      a[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, ka[b][c]),
                                                     __builtin_bit_cast(bf16x8_t, qb[c]), a[b], 0, 0, 0);
  __builtin_amdgcn_s_setprio(0);

  float mx = -__builtin_inff();   // the lane's largest unmasked raw score
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (!TAIL || 4 * r + q < lim[b]) mx = fmaxf(mx, a[b][r]);
  const float xmax = mx * scale_log2;   // NaN when all are masked and the scale is 0
  if (__builtin_amdgcn_ballot_w64(xmax > S.m + kLazyRescale) != 0) {   // rare
    const float bm = group_max4(xmax);
    const float mn = bm > S.m + kLazyRescale ? bm : S.m;
    // 1 for columns that keep their max (or have attended to nothing yet)
    const float alpha = mn == -__builtin_inff() ? 1.f : fast_exp2(S.m - mn);
    S.l *= alpha;
    S.m = mn;
    S.neg = mn == -__builtin_inff() ? 0.f : -mn;
    float ar[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) ar[r] = column_value(alpha, q, r);
#pragma unroll
    for (int blk = 0; blk < 8; ++blk)
#pragma unroll
      for (int r = 0; r < 4; ++r) S.o[blk][r] *= ar[r];
  }

  // Probabilities as bf16 pairs (the A operands: element e of pa[p] and pl[p]
  // is the high and low part of the weight of score 8p + e, p = hi + lo to about
  // 2^-17 relative); the column sum adds the fp32 values.
  u32x4_t pa[NB / 2], pl[NB / 2];
  float sum = 0.f;
#pragma unroll
  for (int pp = 0; pp < NB / 2; ++pp) {
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      float pf[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        // element e + i is token 4((e+i) % 4) + q of block 2pp + (e+i) / 4
        const int b = 2 * pp + ((e + i) >> 2), r = (e + i) & 3;
        float ex = fmaf(a[b][r], scale_log2, S.neg);
        if (TAIL && 4 * r + q >= lim[b]) ex = -__builtin_inff();
        pf[i] = fast_exp2(ex);
      }
      const uint32_t hi = pack_bf16(pf[0], pf[1]);
      pa[pp][e / 2] = hi;
      pl[pp][e / 2] = pack_bf16(pf[0] - bf16_lo(hi), pf[1] - bf16_hi(hi));
      sum += pf[0] + pf[1];
    }
  }
  S.l += sum;

  // Element e of a block's B words is its token 4e + q.
  uint32_t mlo[NB], mhi[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    mlo[b] = 0xffffffffu;
    mhi[b] = 0xffffffffu;
    if constexpr (TAIL) {
      mlo[b] = (q < valid[b] ? 0xffffu : 0u) | (q + 4 < valid[b] ? 0xffff0000u : 0u);
      mhi[b] = (q + 8 < valid[b] ? 0xffffu : 0u) | (q + 12 < valid[b] ? 0xffff0000u : 0u);
    }
  }
  // The B operands (two transposing reads each) of kPvGroup output columns are
  // read together and their high-part MFMAs issued before the low-part ones, so
  // that no MFMA waits for its own LDS read or for the MFMA just before it; the
  // MFMAs run at raised priority, so that a wavefront in its softmax does not
  // hold them up.  (64-call generator step, one wavefront per SIMD in this pass:
  // groups of 1 / 2 / 4 columns 24.9 / 24.4 / 24.3 us, and with the priority
  // 24.6 / 24.5 / 23.9; before, 25.1.)
  constexpr int kPvGroup = 4;
  __builtin_amdgcn_s_setprio(1);
#pragma unroll
  for (int pp = 0; pp < NB / 2; ++pp) {
    const lds_u8_t* v0 = st + (2 * pp) * kPrefixStageBytes + kPrefixKBytes;
    const lds_u8_t* v1 = v0 + kPrefixStageBytes;
#pragma unroll
    for (int j = 0; j < 8; j += kPvGroup) {
      u32x4_t vb[kPvGroup];
#pragma unroll
      for (int i = 0; i < kPvGroup; ++i) {
        const int off = vtr ^ ((j + i) << 5);
        const uint2 b0 = __builtin_bit_cast(
            uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_t*)(v0 + off)));
        const uint2 b1 = __builtin_bit_cast(
            uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_t*)(v1 + off)));
        vb[i] = u32x4_t{b0.x & mlo[2 * pp], b0.y & mhi[2 * pp], b1.x & mlo[2 * pp + 1],
                        b1.y & mhi[2 * pp + 1]};
      }
#pragma unroll
      for (int i = 0; i < kPvGroup; ++i)
        S.o[j + i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, pa[pp]),
                                                             __builtin_bit_cast(bf16x8_t, vb[i]), S.o[j + i], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < kPvGroup; ++i)
        S.o[j + i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, pl[pp]),
                                                             __builtin_bit_cast(bf16x8_t, vb[i]), S.o[j + i], 0, 0, 0);
    }
  }
  __builtin_amdgcn_s_setprio(0);
}

// Attention over the prefix that every sequence of the batch shares: for KV
// head g the B*G query rows form the columns of dense 16-row tiles (four
// sequences of four heads, or two of eight, per tile).  One workgroup owns
// kWaves adjacent tiles (wavefront w: tile w) and one prefix partition, and
// its wavefronts share every block: each loads one quarter (four token rows
// of K and of V, 2 KiB) into a double-buffered LDS stage, and after a
// barrier every wavefront runs its own tile against the staged blocks, two
// blocks per barrier through tile_core_nb.  A block
// thus crosses from L2 to the CU once per four tiles, and each wavefront owns
// whole query rows, so no cross-wavefront merge is needed.  All workgroups of
// a KV head read the same blocks, so each comes from HBM once and from L2
// afterwards.  Every row writes its (o, lse) partial for the partition,
// lse = -inf when it attended to nothing.
constexpr int kPrefixRowsPerWg = 16 * kWaves;
static_assert(kPrefixRowsPerWg == kSharedRowsPerWg, "the host sizes traces from kSharedRowsPerWg");
constexpr int kPrefixLdsBytes = 2 * kPrefixStageBlocks * kPrefixStageBytes;   // two stages

// Rows and tokens of one shared-span workgroup: rows R = row0 .. (16 per
// wavefront) of span rows 0 .. total_rows-1, row R being sequence seq0 + R / G
// and head g*G + R % G; tokens start .. end-1, whose block ids begin at bt;
// the result goes to partial slot `part`; the walk over the blocks starts at
// block `rot`.
struct SharedSpan {
  int seq0, total_rows, row0;
  int start, end;
  const int32_t* bt;
  int part;
  int rot;
};

template <int G, bool TRACE>
__device__ __forceinline__ void shared_span_body(const PrefixParams& p, int g, const SharedSpan& sp,
                                                 lds_u8_t* smem, int32_t* trace) {
  const int lane = threadIdx.x & 63;
  const int wave = wave_uniform(threadIdx.x >> 6);
  const int q = lane >> 4;
  const int n = lane & 15;

  const int total_rows = sp.total_rows;
  const int row0 = sp.row0 + 16 * wave;   // this wavefront's tile
  const int start = sp.start;
  const int end = sp.end;
  const int part = sp.part;
  const int nblk = (end - start + 15) >> 4;     // 1 .. 64 for every launched span
  const int raw = lane < nblk ? sp.bt[lane] : 0;
  const int idc = min(max(raw, 0), p.num_blocks - 1);

  // Column n is query row R = row0 + n: sequence seq0 + R / G, head g*G + R % G.
  // A negative scale goes into the sign of Q (bf16 negation is exact, and so
  // is the negation of every score): the core needs a non-negative one.
  const uint32_t qflip = p.scale_log2 < 0.f ? 0x80008000u : 0u;
  const float scale_abs = fabsf(p.scale_log2);
  uint4 qb[4];
  int ctx;
  int min_ctx;
  {
    const int R = row0 + n;
    const bool ok = R < total_rows;
    const int bR = ok ? sp.seq0 + R / G : 0;
    const uint16_t* qrow = p.q + ((size_t)bR * p.num_q_heads + g * G + R % G) * kD;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      uint4 w = ok ? *reinterpret_cast<const uint4*>(qrow + (4 * s + q) * 8) : make_uint4(0, 0, 0, 0);
      w.x ^= qflip; w.y ^= qflip; w.z ^= qflip; w.w ^= qflip;
      qb[s] = w;
    }
    int c = ok ? p.context_lens[bR] : 0;
    c = c < 0 ? 0 : (c > p.max_ctx ? p.max_ctx : c);
    ctx = c;
    // shortest context among the tile's columns (decides when to mask)
    min_ctx = __builtin_amdgcn_readfirstlane(-(int)group_max4(row_max16(-(float)c)));
  }

  MfmaState S;
  S.m = -__builtin_inff();
  S.neg = 0.f;
  S.l = 0.f;
#pragma unroll
  for (int blk = 0; blk < 8; ++blk) S.o[blk] = floatx4_t{0.f, 0.f, 0.f, 0.f};

  constexpr size_t kTileElems = 16 * kD;
  const size_t blk_stride = (size_t)p.num_kv_heads * kTileElems;
  // This wavefront's quarter of a tile: token row 4*wave + q, chunk n.
  const int share_off = ((4 * wave + q) * kD + n * 8) * 2;
  const int vtr = v_tr(q, n);
  const uint16_t* kbase = p.k_pool + (size_t)g * kTileElems;
  const uint16_t* vbase = p.v_pool + (size_t)g * kTileElems;

  const int rot = sp.rot;
  auto block_of = [&](int i) { const int j = i + rot; return j >= nblk ? j - nblk : j; };
  auto load = [&](uint4 (&dst)[2], int i) {
    const bool ok = i < nblk;
    const size_t id = (size_t)__builtin_amdgcn_readlane(idc, ok ? block_of(i) : 0);
    const int bytes = ok ? (int)(kTileElems * 2) : 0;
    const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(kbase + id * blk_stride), 0, bytes, kBufferDescWord3);
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(vbase + id * blk_stride), 0, bytes, kBufferDescWord3);
    const auto k = __builtin_amdgcn_raw_buffer_load_b128(rk, share_off, 0, 0);
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(rv, share_off, 0, 0);
    dst[0] = make_uint4(k[0], k[1], k[2], k[3]);
    dst[1] = make_uint4(v[0], v[1], v[2], v[3]);
  };

  // The blocks go in pairs: every wavefront publishes its quarter of both
  // blocks of pair j to one LDS stage (double-buffered), loads the quarters
  // of pair j+1 into the other two ring slots, one barrier, then every
  // wavefront runs its tile against the pair.  The two blocks of a pair need
  // not be adjacent; an odd last block pairs with an empty one (valid = 0).
  constexpr int NB = 2;
  constexpr int kRing = kPrefixRing;
  uint4 ring[kRing][2];
#pragma unroll
  for (int s = 0; s < kRing - 2; ++s) load(ring[s], s);
  const int npair = (nblk + 1) >> 1;
  for (int j0 = 0; j0 < npair; j0 += kRing / 2) {
#pragma unroll
    for (int h = 0; h < kRing / 2; ++h) {
      const int j = j0 + h;
      if (j < npair) {                         // uniform over the workgroup
        lds_u8_t* st = smem + (j & 1) * 2 * kPrefixStageBytes;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          lds_u8_t* sb = st + e * kPrefixStageBytes;
          const int s = 2 * h + e;
          *reinterpret_cast<lds_u32x4_t*>(sb + k_stage(4 * wave + q, n)) =
              u32x4_t{ring[s][0].x, ring[s][0].y, ring[s][0].z, ring[s][0].w};
          *reinterpret_cast<lds_u32x4_t*>(sb + kPrefixKBytes + v_stage(4 * wave + q, n)) =
              u32x4_t{ring[s][1].x, ring[s][1].y, ring[s][1].z, ring[s][1].w};
        }
        load(ring[(2 * h + kRing - 2) % kRing], 2 * j + kRing - 2);
        load(ring[(2 * h + kRing - 1) % kRing], 2 * j + kRing - 1);
        __syncthreads();
        int valid[NB], lim[NB];
        bool fast = true;
#pragma unroll
        for (int s = 0; s < NB; ++s) {
          const int i = NB * j + s;
          const bool has = i < nblk;
          const int tb = has ? start + block_of(i) * 16 : end;
          valid[s] = has ? min(16, end - tb) : 0;
          lim[s] = min(valid[s], max(ctx - tb, 0));
          fast = fast && valid[s] == 16 && min_ctx - tb >= 16;
          if constexpr (TRACE) {
            // slot = the block's position in the span (not in the walk)
            const int bi = has ? block_of(i) : 0;
            const int id = __builtin_amdgcn_readlane(raw, bi);
            if (has && wave == 0 && lane == 0) {
              int32_t* tr = trace + 3 * bi;
              tr[0] = (start >> 4) + bi;
              tr[1] = id;
              tr[2] = valid[s];
            }
          }
        }
        if (fast)
          tile_core_nb<false, NB>(S, st, vtr, qb, valid, lim, q, n, scale_abs);
        else
          tile_core_nb<true, NB>(S, st, vtr, qb, valid, lim, q, n, scale_abs);
      }
    }
  }

  // Normalise per row and write this partition's partials: lane (q, n)
  // holds O[rows 4q+r][dims 16j + n], j = 0..7.
  const float lcol = group_sum4(S.l);
  const float inv = lcol > 0.f ? 1.0f / lcol : 0.f;
  if (q == 0 && row0 + n < total_rows) {
    const int R = row0 + n;
    const size_t row = ((size_t)(sp.seq0 + R / G) * p.num_q_heads + g * G + R % G) * p.part_stride + part;
    p.part_lse[row] = lcol > 0.f ? (S.m + log2f(lcol)) * kLn2 : -__builtin_inff();
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int R = row0 + 4 * q + r;
    const float f = column_value(inv, q, r);
    if (R < total_rows) {
      const size_t row =
          ((size_t)(sp.seq0 + R / G) * p.num_q_heads + g * G + R % G) * p.part_stride + part;
      float* po = p.part_o + row * kD + n;
#pragma unroll
      for (int j = 0; j < 8; ++j) store_partial(po + 16 * j, S.o[j][r] * f);
    }
  }
}

// The batch-wide prefix: partition `part` of the prefix against row group
// `grp` (64 rows) of all B*G query rows of KV head g.
template <int G, bool TRACE>
__device__ __forceinline__ void prefix_mfma_body(const PrefixParams& p, int wg_index, lds_u8_t* smem) {
  const int total_rows = p.batch * G;
  const int groups = (total_rows + kPrefixRowsPerWg - 1) / kPrefixRowsPerWg;
  int wg = wg_index;
  const int g = wg % p.num_kv_heads;
  wg /= p.num_kv_heads;
  const int grp = wg % groups;
  const int part = wg / groups;
  SharedSpan sp;
  sp.seq0 = 0;
  sp.total_rows = total_rows;
  sp.row0 = grp * kPrefixRowsPerWg;
  sp.start = part * p.part_tokens;
  sp.end = min(p.prefix_len, sp.start + p.part_tokens);
  sp.bt = p.block_tables + (sp.start >> 4);
  sp.part = part;
  // The workgroups of a KV head walk the partition from evenly spread
  // starting blocks, so at any moment they read different blocks instead of
  // all queueing on the L2 lines of the same one.
  const int nblk = (sp.end - sp.start + 15) >> 4;
  sp.rot = (int)(((int64_t)grp * nblk) / groups) % nblk;
  int32_t* tr = nullptr;
  if constexpr (TRACE)
    tr = p.trace_prefix + (((size_t)part * groups + grp) * p.num_kv_heads + g) * p.prefix_trace_tiles * 3;
  shared_span_body<G, TRACE>(p, g, sp, smem, tr);
}

// The second level: group k's rows (its sequences x G heads of KV head g,
// at most 64) against the group_len tokens the group shares after the
// prefix, one partition written to slot prefix_parts.
template <int G, bool TRACE>
__device__ __forceinline__ void group_mfma_body(const PrefixParams& p, int wg_index, lds_u8_t* smem) {
  const int g = wg_index % p.num_kv_heads;
  const int k = wg_index / p.num_kv_heads;
  // device data: clamped into the batch and the stated bound
  int s0 = p.group_start[k];
  s0 = s0 < 0 ? 0 : (s0 > p.batch ? p.batch : s0);
  int s1 = p.group_start[k + 1];
  s1 = s1 < s0 ? s0 : (s1 > p.batch ? p.batch : s1);
  s1 = min(s1, s0 + p.max_group_size);
  if (s1 == s0) return;                        // whole workgroup: an empty group
  SharedSpan sp;
  sp.seq0 = s0;
  sp.total_rows = (s1 - s0) * G;
  sp.row0 = 0;
  sp.start = p.prefix_len;
  sp.end = p.prefix_len + p.group_len;
  sp.bt = p.block_tables + (size_t)s0 * p.bt_stride + (sp.start >> 4);
  sp.part = p.prefix_parts;
  sp.rot = 0;
  int32_t* tr = nullptr;
  if constexpr (TRACE)
    tr = p.trace_group + ((size_t)k * p.num_kv_heads + g) * p.group_trace_tiles * 3;
  shared_span_body<G, TRACE>(p, g, sp, smem, tr);
}

}  // namespace mfma
}  // namespace pa
