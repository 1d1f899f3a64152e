// gfx950 kernels for a batch of 2..64 tokens (paper Section 5.3: the rows of W_up / W_down are
// read once for the union of the tokens' active sets), bf16, int8 / int4 or fp32 weights.  What
// follows describes bf16; is_f32 says what differs for fp32.
//
// Every contraction runs on the matrix cores (v_mfma_f32_16x16x32_bf16): LoPA's A x,
// the gate (W_gate x, or B z), the W_up dots of the union rows and the down
// projection.  Token-side operands (x, z, zval) enter as bf16 hi + lo pairs (v - hi
// rounded again): two MFMAs per step whose products are exact in fp32, so the split
// leaves a relative error of about 2^-16 per element, far inside the 1e-3 band of the
// active-set decision.  A 16-row weight tile is the A operand: lane l holds 8
// consecutive bf16 of row l mod 16 and the four lane groups l / 16 hold four
// consecutive 16-byte chunks.  Which k positions a lane group holds does not matter for
// a full reduction as long as both operands use the same ones.  Weights are read row by
// row (up to 256 contiguous bytes of a row per instruction) and reshaped into that
// layout through a wave-private LDS tile (see the streaming core).
//
// One call is three kernels (two for standard gating), one more above 16 tokens:
//   k_split_tokens (more than 16 tokens) the tokens split once into bf16 hi / lo planes
//                  in fragment order, read by the next two kernels;
//   k_lopa_z_mfma  z = A x as two partial sums over halves of the d range;
//   k_gate_up_mfma per segment of at most 64 rows: gate, union of the tokens' active rows,
//                  ascending, W_up dots of the union rows; zval = act * v is left by
//                  quads of entries for the down product (k_gate_up_q4 does the
//                  same for 2..4 tokens on 4x4x4 products, k_gate_up_mfma2 at two
//                  workgroups a CU where d_ff is large);
//   k_down_mfma    Y[tokens][cols] += Z[tokens][entries] D[entries][cols] over the
//                  union rows, segment by segment.
// A wave of the gate kernel multiplies four row tiles over a quarter of the k range, so
// each token fragment it loads (and splits, when it reads fp32 rows) feeds four tiles;
// the loads of the next k steps are in flight while the current ones are multiplied.  All operand loads are
// raw buffer loads: a lane with nothing to load (a row past the segment or the union,
// a token past the batch, a k step past the row) uses an offset beyond the buffer,
// which returns zero without a memory access, so every wave issues the same loads in
// the same order and the load counter waits stay exact.
//
// The down product needs, per lane, 8 entries of one column as the B operand, while a
// row gather gives a lane 8 columns of one entry.  The gathered rows go to LDS as they
// are and come back through gfx950's transposing LDS read (ds_read_b64_tr_b16), which
// exchanges 16-bit elements between the lanes of a 16-lane group: one pair of such
// reads hands every lane its 8 entries of one column.
#include "ffn_device.h"
#include "ffn_internal.h"
#include "ffn_mfma.h"

namespace ffn {
namespace {

constexpr int kTiles = 4;                // 16-row tiles of a gate segment
constexpr int kSegRowsB = 16 * kTiles;   // rows per gate segment (one 64-lane ballot)
constexpr int kParts = kBlock / kWave;   // k parts of a workgroup, one per wave
constexpr int kSegGrid = 256;            // most workgroups of the gate kernel, one per CU
constexpr int kSegGrid2 = 512;           // the same at two workgroups per CU

// k-step range [ks0, ks1) of k part kp out of np for rows of C chunks (4 chunks a step)
__device__ __forceinline__ void kpart(int C, int kp, int np, int* ks0, int* ks1) {
  const int nks = (C + 3) / 4;
  const int per = (nks + np - 1) / np;
  *ks0 = min(nks, kp * per);
  *ks1 = min(nks, *ks0 + per);
}

// ------------------------------------------------------------------ streaming core
// A group of KU consecutive k steps covers 16 RT weight rows x 4 KU chunks.  The group
// is read row by row, LPR = 4 KU lanes per row and 64 / LPR rows per instruction (256
// contiguous bytes per row for KU = 4), streamed past the caches, and reshaped into MFMA
// operands through a wave-private LDS tile: row br of the group sits at br * PITCH, one
// pad chunk per row keeping the operand reads free of bank conflicts.  (Loading the
// operand layout directly reads 64 bytes of each of 16 rows per instruction, which
// streams about 25% slower.)
// Quantized rows (W = WI8 / WI4): a loaded 16-byte chunk holds R8 = 2 or 4 of the tile's
// 8-element chunks, so a row takes 4 KU / R8 lanes; the codes are converted to bf16 as
// they go to the tile, which keeps the bf16 layout.
template <int RT, int KU, class W = WBf16>
struct WStage {
  static constexpr int R8 = W::EPC / tile_elems<W>();  // tile chunks per loaded chunk
  static constexpr int LPR = 4 * KU / R8;     // lanes per row of a load instruction
  static constexpr int RPI = kWave / LPR;     // rows per load instruction
  static constexpr int NI = (16 * RT + RPI - 1) / RPI;  // load instructions per group
  static constexpr int PITCH = 4 * KU + 1;    // 16-byte (8 bf16) chunks per LDS row
  static constexpr int WORDS = 16 * RT * PITCH;  // uint4 of one wave's tile
};

// Rows of this lane's load instructions: roff[i] = row_of(i RPI + lane / LPR) times the
// row's loaded chunks (C / R8 for rows of C tile chunks), or -1 where row_of gives no row
// (-1) or the lane falls past the tile's 16 RT rows.
template <int RT, int KU, class W = WBf16, class RowOf>
__device__ __forceinline__ void stage_rows(int* roff, int C, RowOf row_of) {  // roff: WStage::NI entries
  using S = WStage<RT, KU, W>;
  const int lane = lane_id();
#pragma unroll
  for (int i = 0; i < S::NI; ++i) {
    const int br = i * S::RPI + lane / S::LPR;
    const int r = br < 16 * RT ? row_of(br) : -1;
    roff[i] = r >= 0 ? r * (C / S::R8) : -1;
  }
}

// Operands of one group: the weight chunks as loaded and, per k step and token tile, the
// token fragment.  Two forms of the token side:
//  - fp32 rows: the 8 fp32 of the chunk (two 16-byte halves) from each of NP partial
//    copies of the token matrix, summed and split into hi / lo when multiplied.  A token
//    matrix is [T][8 C] fp32; partial copy p starts part_bytes * p into its buffer; tn = T.
//  - PRE (pre-split, NP = 1): b[u][nt][0] = the hi and lo fragments of the lane, read from
//    planes [k step][token tile][lane] of uint4 (k_split_tokens); the lo plane starts
//    part_bytes after the hi plane; tn = the planes' token-tile count.
// fp32 weights: one piece instead of two, the chunk's 4 fp32 (one plane when PRE).
// NORM (LoPA's z under RMSNorm): also the gains of the chunk's components.
template <int RT, int NT, int KU, int NP, class W = WBf16, bool NORM = false>
struct Frags {
  uint4 a[WStage<RT, KU, W>::NI];
  uint4 b[KU][NT][NP][is_f32<W>() ? 1 : 2];
  uint4 gain[NORM ? KU : 1][is_f32<W>() ? 1 : 2];
};

// RMSNorm between LoPA's factors inside the gate product: h = inv B (gain . z), inv = 1 /
// sqrt(mean z^2 + eps) one scalar a token, so the product takes gain . z and its rows are scaled
// afterwards.  sq[nt]: the sum of squares of the z components that this lane multiplies (token
// 16 nt + (lane & 15)).  A kernel of its own for the norm had cost 4.5 us and a launch (8B shape, full
// form, 16 tokens: 61.8 -> 58.9 us a call, the gate kernel 30.0 -> 31.1).
template <int NT>
struct ZNorm {
  Buf gain;
  bool has_gain;
  float sq[NT];
};

template <int RT, int NT, int KU, int NP, bool PRE = false, class W = WBf16, bool NORM = false>
__device__ __forceinline__ void load_frags(Frags<RT, NT, KU, NP, W, NORM>& f, const Buf& wb, int C,
                                           const int* roff, const Buf& tb, uint32_t part_bytes, int tn, int ks,
                                           int ks1, const ZNorm<NT>* zn = nullptr) {
  using S = WStage<RT, KU, W>;
  const int lane = lane_id(), m = lane & 15, g = lane >> 4;
  {
    // the lane's loaded chunk gc of the group: tile chunks R8 gc .. R8 gc + R8 - 1
    const int gc = lane % S::LPR, c = 4 * ks / S::R8 + gc;
    const bool cv = ks + (gc * S::R8 >> 2) < ks1 && c < C / S::R8;
#pragma unroll
    for (int i = 0; i < S::NI; ++i)
      f.a[i] = ldb_nt(wb, (cv && roff[i] >= 0) ? 16u * (uint32_t)(roff[i] + c) : kOOB);
  }
  if constexpr (PRE) {
    static_assert(NP == 1, "pre-split tokens have one copy");
#pragma unroll
    for (int u = 0; u < KU; ++u)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const uint32_t off = ks + u < ks1 ? 16u * ((uint32_t)((ks + u) * tn + nt) * kWave + lane) : kOOB;
        f.b[u][nt][0][0] = ldb(tb, off);
        if constexpr (!is_f32<W>()) f.b[u][nt][0][1] = ldb(tb, off + part_bytes);
      }
    return;
  }
  const int T = tn;
#pragma unroll
  for (int u = 0; u < KU; ++u) {
    const int c = 4 * (ks + u) + g;
    const bool cv = ks + u < ks1 && c < C;
    if constexpr (NORM) {
      const uint32_t off = cv && zn->has_gain ? tok_bytes<W>() * (uint32_t)c : kOOB;
      f.gain[u][0] = ldb(zn->gain, off);
      if constexpr (!is_f32<W>()) f.gain[u][1] = ldb(zn->gain, off + 16);
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int tok = 16 * nt + m;
      const uint32_t off = (cv && tok < T) ? tok_bytes<W>() * (uint32_t)(tok * C + c) : kOOB;
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        f.b[u][nt][p][0] = ldb(tb, off + p * part_bytes);
        if constexpr (!is_f32<W>()) f.b[u][nt][p][1] = ldb(tb, off + p * part_bytes + 16);
      }
    }
  }
}

// tile: this wave's LDS tile (Stage::WORDS uint4).  Every row tile is multiplied: one
// past the rows in use was loaded as zeros and only adds zeros to an accumulator that
// is never read.
// The token fragment of one k step and token tile from fp32 rows: the NP copies of the
// lane's 8 values summed, then split into hi / lo.
template <int NP>
__device__ __forceinline__ void sum_copies(const uint4 (&b)[NP][2], float (&v)[8]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint4 q = b[0][h];
    v[4 * h] = __uint_as_float(q.x);
    v[4 * h + 1] = __uint_as_float(q.y);
    v[4 * h + 2] = __uint_as_float(q.z);
    v[4 * h + 3] = __uint_as_float(q.w);
  }
#pragma unroll
  for (int p = 1; p < NP; ++p)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint4 q = b[p][h];
      v[4 * h] += __uint_as_float(q.x);
      v[4 * h + 1] += __uint_as_float(q.y);
      v[4 * h + 2] += __uint_as_float(q.z);
      v[4 * h + 3] += __uint_as_float(q.w);
    }
}
// One chunk of z under RMSNorm: its squares into sq, then times the gains.
template <int E, int H>
__device__ __forceinline__ void norm_chunk(float (&v)[E], const uint4 (&gain)[H], bool has_gain, float& sq) {
#pragma unroll
  for (int e = 0; e < E; ++e) sq = fmaf(v[e], v[e], sq);
  if (has_gain) {
#pragma unroll
    for (int h = 0; h < H; ++h) {
      v[4 * h] *= __uint_as_float(gain[h].x);
      v[4 * h + 1] *= __uint_as_float(gain[h].y);
      v[4 * h + 2] *= __uint_as_float(gain[h].z);
      v[4 * h + 3] *= __uint_as_float(gain[h].w);
    }
  }
}

template <int RT, int NT, int KU, int NP, bool PRE = false, class W = WBf16, bool NORM = false>
__device__ __forceinline__ void mma_frags(const Frags<RT, NT, KU, NP, W, NORM>& f, uint4* tile, f32x4_t (&acc)[RT][NT],
                                          ZNorm<NT>* zn = nullptr) {
  using S = WStage<RT, KU, W>;
  const int lane = lane_id(), m = lane & 15, g = lane >> 4;
#pragma unroll
  for (int i = 0; i < S::NI; ++i) {
    const int br = i * S::RPI + lane / S::LPR;
    if constexpr (S::R8 == 1) {
      tile[br * S::PITCH + lane % S::LPR] = f.a[i];
    } else if (br < 16 * RT) {  // lanes past the tile's rows loaded nothing
      put_bf16_chunks<W>(tile + br * S::PITCH + (lane % S::LPR) * S::R8, f.a[i]);
    }
  }
  __builtin_amdgcn_wave_barrier();  // LDS operations of a wave complete in order
  f32x4_t grp[RT][NT];  // fp32 weights: the group's sums
#pragma unroll
  for (int u = 0; u < KU; ++u)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      if constexpr (is_f32<W>()) {
        float v[4];
        v[0] = comp<0>(f.b[u][nt][0][0]);
        v[1] = comp<1>(f.b[u][nt][0][0]);
        v[2] = comp<2>(f.b[u][nt][0][0]);
        v[3] = comp<3>(f.b[u][nt][0][0]);
#pragma unroll
        for (int p = 1; p < NP; ++p) {
          v[0] += comp<0>(f.b[u][nt][p][0]);
          v[1] += comp<1>(f.b[u][nt][p][0]);
          v[2] += comp<2>(f.b[u][nt][p][0]);
          v[3] += comp<3>(f.b[u][nt][p][0]);
        }
        if constexpr (NORM) norm_chunk(v, f.gain[u], zn->has_gain, zn->sq[nt]);
        uint4 a[RT];
        f32x4_t ks[RT];  // the k step's sums
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) a[rt] = tile[(16 * rt + m) * S::PITCH + 4 * u + g];
        // the row tiles inside: no product waits on the one before it
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) ks[rt] = mfma16f(comp<0>(a[rt]), v[0], f32x4_t{0.f, 0.f, 0.f, 0.f});
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) ks[rt] = mfma16f(comp<1>(a[rt]), v[1], ks[rt]);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) ks[rt] = mfma16f(comp<2>(a[rt]), v[2], ks[rt]);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) ks[rt] = mfma16f(comp<3>(a[rt]), v[3], ks[rt]);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) grp[rt][nt] = u == 0 ? ks[rt] : grp[rt][nt] + ks[rt];
        continue;
      } else {
      bf16x8_t hi, lo;
      if constexpr (PRE) {
        hi = bf8(f.b[u][nt][0][0]);
        lo = bf8(f.b[u][nt][0][1]);
      } else {
        float v[8];
        sum_copies<NP>(f.b[u][nt], v);
        if constexpr (NORM) norm_chunk(v, f.gain[u], zn->has_gain, zn->sq[nt]);
        split8(v, hi, lo);
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const bf16x8_t a = bf8(tile[(16 * rt + m) * S::PITCH + 4 * u + g]);
        acc[rt][nt] = mfma16(a, hi, acc[rt][nt]);
        acc[rt][nt] = mfma16(a, lo, acc[rt][nt]);
      }
      }
    }
  if constexpr (is_f32<W>()) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[rt][nt] += grp[rt][nt];
  }
  __builtin_amdgcn_wave_barrier();
}

// acc[rt][nt] += weight tile rt . token tile nt over the k steps [ks0, ks1) (uniform).
// Two register sets alternate: the loads of the next KU steps are issued before the
// current ones are multiplied; loads past ks1 are out of range and read nothing.  A
// pair always multiplies both halves (a group past ks1 adds zeros) and the exit test
// closes the pair, so no load sits on a conditional path: with an exit test between
// the halves the compiler moved the loads next to their use and waited on them there.
template <int RT, int NT, int KU, int NP, bool PRE = false, class W = WBf16, bool NORM = false>
__device__ __forceinline__ void stream_rows(const Buf& wb, int C, const int* roff, uint4* tile, const Buf& tb,
                                            uint32_t part_bytes, int tn, int ks0, int ks1, f32x4_t (&acc)[RT][NT],
                                            ZNorm<NT>* zn = nullptr) {
  if (ks0 >= ks1) return;
  Frags<RT, NT, KU, NP, W, NORM> f0, f1;
  load_frags<RT, NT, KU, NP, PRE, W, NORM>(f0, wb, C, roff, tb, part_bytes, tn, ks0, ks1, zn);
  if (ks0 + KU >= ks1) {  // a single group
    mma_frags<RT, NT, KU, NP, PRE, W, NORM>(f0, tile, acc, zn);
    return;
  }
  for (int ks = ks0;; ks += 2 * KU) {
    load_frags<RT, NT, KU, NP, PRE, W, NORM>(f1, wb, C, roff, tb, part_bytes, tn, ks + KU, ks1, zn);
    issue_barrier();
    mma_frags<RT, NT, KU, NP, PRE, W, NORM>(f0, tile, acc, zn);
    load_frags<RT, NT, KU, NP, PRE, W, NORM>(f0, wb, C, roff, tb, part_bytes, tn, ks + 2 * KU, ks1, zn);
    issue_barrier();
    mma_frags<RT, NT, KU, NP, PRE, W, NORM>(f1, tile, acc, zn);
    if (ks + 2 * KU >= ks1) break;
  }
}

// The token side of a product with rows of C chunks: fp32 rows of x, or (pre) the
// planes written by k_split_tokens for ntt token tiles.
struct TokSrc {
  Buf b;
  uint32_t part;
  int tn;
};
template <class W>
__device__ __forceinline__ TokSrc token_source(bool pre, const float* x, const uint4* xs, int C, int T, int ntt) {
  if (pre) {
    const uint32_t plane = 16u * (uint32_t)((C + 3) / 4) * (uint32_t)ntt * (uint32_t)kWave;
    return TokSrc{make_buf(xs, is_f32<W>() ? plane : 2 * plane), plane, ntt};
  }
  return TokSrc{make_buf(x, tok_bytes<W>() * (uint32_t)T * (uint32_t)C), 0u, T};
}

// ------------------------------------------------------------------ token pre-split
// For batches of more than one token tile every gate workgroup multiplies all tokens
// against its rows.  Read as fp32 rows, a token load instruction touches 16 rows (one per
// token of the tile) and half of each cache line it uses, and every workgroup splits
// every value again.  This kernel writes the split once, in fragment order: entry
// ((ks ntt + nt) 64 + lane) of the hi plane holds the bf16 hi parts of tokens
// 16 nt + (lane & 15), elements 32 ks + 8 (lane >> 4) .. + 7, the lo plane (nks ntt 64
// entries later) their lo parts; zero past the batch and past d.  F32 (fp32 weights): one plane
// of the fp32 values, elements 16 ks + 4 (lane >> 4) .. + 3.
// Values go into the workspace as arithmetic leaves them, without signalling NaNs (the conversions to
// bf16 quiet theirs): one with kZTag's bits would look like a published z to a later call.
__device__ __forceinline__ uint32_t quiet(uint32_t v) { return (v & 0x7FFFFFFFu) > 0x7F800000u ? v | 0x00400000u : v; }
template <bool F32>
__global__ __launch_bounds__(kBlock) void k_split_tokens(const float* __restrict__ x, int C, int T, int nks, int ntt,
                                                         uint4* __restrict__ xs) {
  const int n = nks * ntt * kWave, i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const int lane = i % kWave, fr = i / kWave, nt = fr % ntt, ks = fr / ntt;
  const int tok = 16 * nt + (lane & 15), c = 4 * ks + (lane >> 4);
  if constexpr (F32) {
    uint4 v = tok < T && c < C ? reinterpret_cast<const uint4*>(x)[(size_t)tok * C + c] : make_uint4(0u, 0u, 0u, 0u);
    v.x = quiet(v.x), v.y = quiet(v.y), v.z = quiet(v.z), v.w = quiet(v.w);
    xs[i] = v;
    return;
  }
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (tok < T && c < C) {
    const float4* p = reinterpret_cast<const float4*>(x + 8 * ((size_t)tok * C + c));
    const float4 a = p[0], b = p[1];
    v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w, v[4] = b.x, v[5] = b.y, v[6] = b.z, v[7] = b.w;
  }
  bf16x8_t hi, lo;
  split8(v, hi, lo);
  xs[i] = __builtin_bit_cast(uint4, hi);
  xs[n + i] = __builtin_bit_cast(uint4, lo);
}

// ------------------------------------------------------------------ LoPA z = A x
// Workgroup b: 16-row tile of A over one half (kZParts) of the d range, each of its waves a
// sixteenth of that half, for NT token tiles; with pre-split tokens each group of NT token
// tiles has workgroups of its own (at 64 tokens, r = 512: 256 workgroups instead of 64 that
// each read every token's fragments).  The waves' sums are added in LDS (fixed order) and
// stored as partial copy `part` of z: zp[part][tc][r]; the gate kernel adds the two copies.
constexpr int kZWaves = 16;
constexpr int kZParts = 2;

template <int NT, bool PRE, class W>
__global__ __launch_bounds__(kZWaves * kWave) void k_lopa_z_mfma(const float* __restrict__ x,
                                                                 const uint4* __restrict__ xs, int ntt,
                                                                 const uint4* __restrict__ A, int C, int T, int r,
                                                                 int tc, float* __restrict__ zp, GWork gw,
                                                                 const float* __restrict__ s_a) {
  if (g_precompute(gw)) return;
  __shared__ f32x4_t s_part[kZWaves][NT][kWave];
  const int lane = lane_id(), wave = uniform(threadIdx.x / kWave);
  // blockIdx.x = (tile kZParts + part) ngrp + tg: tg the group of NT token tiles
  const int ngrp = PRE ? ntt / NT : 1;
  const int tg = (int)blockIdx.x % ngrp, tp = (int)blockIdx.x / ngrp;
  const int tile = tp / kZParts, part = tp % kZParts;
  constexpr int KU = NT == 1 ? 4 : NT == 2 ? 2 : 1;
  using S = WStage<1, KU, W>;
  __shared__ uint4 s_stage[kZWaves][S::WORDS];
  int roff[S::NI];
  stage_rows<1, KU, W>(roff, C, [&](int br) { return tile * 16 + br < r ? tile * 16 + br : -1; });
  const Buf ab = make_buf(A, 16u * (uint32_t)r * (uint32_t)(C / S::R8));
  TokSrc tok = token_source<W>(PRE, x, xs, C, T, ntt);
  if constexpr (PRE) {  // the group's first token tile at entry 0 of each k step's row of tiles
    const uint32_t skip = 16u * (uint32_t)(tg * NT * kWave);
    tok.b = make_buf(xs + (size_t)tg * NT * kWave, (is_f32<W>() ? 1 : 2) * tok.part - skip);
  }
  f32x4_t acc[1][NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) acc[0][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  int ks0, ks1;
  kpart(C, part * kZWaves + wave, kZParts * kZWaves, &ks0, &ks1);
  stream_rows<1, NT, KU, 1, PRE, W>(ab, C, roff, s_stage[wave], tok.b, tok.part, tok.tn, ks0, ks1, acc);
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) s_part[wave][nt][lane] = acc[0][nt];
  __syncthreads();
  // thread o: local token o / 16 of the group, row tile * 16 + o % 16 (16 consecutive floats
  // of z a token); that value sits in lane 16 (kk / 4) + tl % 16, element kk % 4, of the
  // group's token tile tl / 16
  const float* sp = reinterpret_cast<const float*>(s_part);
  const int tok0 = 16 * NT * tg;
  for (int o = threadIdx.x; o < 16 * NT * 16; o += kZWaves * kWave) {
    const int tl = o >> 4, kk = o & 15, tok = tok0 + tl;
    const int k = tile * 16 + kk;
    if (k >= r || tok >= T) continue;
    const int nt = tl >> 4, src = ((16 * (kk >> 2) + (tl & 15)) << 2) + (kk & 3);
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < kZWaves; ++w) s += sp[(w * NT + nt) * kWave * 4 + src];
    if constexpr (is_quant<W>()) s *= s_a[k];  // the row's scale
    zp[((size_t)part * tc + tok) * r + k] = s;
  }
}

// One wave's 16 entries: lane m + 16 g holds nz[i] of entry 4 g + i for the tokens m, 16 + m, ...;
// bit 4 g + i of *out is set if any lane of the group holds true.
__device__ __forceinline__ void put_alive(uint16_t* out, const bool (&nz)[4]) {
  uint32_t mask = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint64_t b = __ballot(nz[i]);
#pragma unroll
    for (int g = 0; g < 4; ++g)
      if ((b >> (16 * g)) & 0xffffull) mask |= 1u << (4 * g + i);
  }
  if (lane_id() == 0) *out = (uint16_t)mask;
}

// ------------------------------------------------------------------ gate + union + W_up
// Segments of at most 64 neurons, each workgroup taking every gridDim.x-th one.  Wave w
// multiplies the segment's four row tiles over k part w; the parts are added in LDS,
// wave w owning tile w.  A neuron joins the union if any token activates it (h > t;
// NaN compares false); one ballot orders the union ascending.  The W_up dots of the
// union rows use the same split, and zval = act * v goes to the buffer of the down kernel by
// quads of entries: quad qps seg + k (entries 4 k .. 4 k + 3 of segment seg), token tile nt and
// token 16 nt + m at uint4 ((qps seg + k) ntt + nt) 16 + m, the four values as bf16 hi parts then
// lo parts (fp32 weights: as fp32).  A used quad is written whole (zero past the union), an
// unused one is never read.
// fp32 weights also leave alive[4 seg + k], bit j: entry 16 k + j of the segment has a value other
// than 0 for some token.  The down kernel does not read the W_down rows of the other entries
// (every entry counts as alive in a dense call), as the vector-ALU batch kernels do not.
// LOPA: the gate rows are B [d_ff][r] against z = zp[0] + zp[1]; otherwise W_gate x.
// KU / KUU: k steps per load group of the gate rows / the W_up rows.
// FORM (a FormKind): the paper's full form (`form`): the activation value, SiLU on the
// W_up output and, with kFormLoPA, the fixed term G added to the gate before the union.
template <class W, bool LOPA, bool DENSE, int NT, int KU, int KUU, int FORM>
__device__ __forceinline__ void gate_up_body(const float* __restrict__ x, const float* __restrict__ zp,
                                             const uint4* __restrict__ gate_w, int Cg, const uint4* __restrict__ w_up,
                                             int Cu, int T, int d, int d_ff, int nseg, float t, int slots, int tc,
                                             int32_t* __restrict__ meta, int32_t* __restrict__ seg_count,
                                             int32_t* __restrict__ seg_idx, float* __restrict__ seg_act,
                                             uint4* __restrict__ zf, float* __restrict__ y,
                                             const uint4* __restrict__ xs, int ntt, Form form,
                                             const float* __restrict__ gx, const float* __restrict__ s_g,
                                             const float* __restrict__ s_up, const float* __restrict__ s_down,
                                             uint16_t* __restrict__ alive, int qps) {
  constexpr bool Q = is_quant<W>();
  constexpr int R8 = W::EPC / tile_elems<W>();
  constexpr bool FULL = FORM != kFormDefault, HAS_G = FORM == kFormLoPA;
  constexpr bool PRE = NT > 1;  // tokens pre-split by k_split_tokens
  // the W_up rows of a union of at most two row tiles go as two tiles with twice the k
  // steps a group (one token tile only: the register budget of wider ones is spent)
  constexpr bool NARROW = NT == 1;
  constexpr int STAGE_A = WStage<kTiles, (KU > KUU ? KU : KUU)>::WORDS, STAGE_B = WStage<2, 2 * KUU>::WORDS;
  constexpr int STAGE = NARROW && STAGE_B > STAGE_A ? STAGE_B : STAGE_A;
  __shared__ uint4 s_stage[kParts][STAGE];
  __shared__ f32x4_t s_red[kParts][kTiles][NT][kWave];
  __shared__ float s_act[kSegRowsB][16 * NT];
  __shared__ uint32_t s_mask[kTiles];
  __shared__ int s_list[kSegRowsB];
  __shared__ int s_cnt;
  __shared__ float s_zsq[HAS_G ? kParts : 1][16 * NT];  // sums of z^2 of the waves' k parts

  const int lane = lane_id(), wave = uniform(threadIdx.x / kWave);
  const int m = lane & 15, g = lane >> 4;
  const bool norm = HAS_G && form.rms_eps > 0.f, has_g = HAS_G && form.g_idx;
  clear_output(y, T * d, meta, nseg);
  const TokSrc tok = token_source<W>(PRE, x, xs, Cu, T, ntt);
  const Buf ub = make_buf(w_up, 16u * (uint32_t)d_ff * (uint32_t)(Cu / R8));

  // segments blockIdx.x, blockIdx.x + gridDim.x, ... (the host makes the counts equal)
  const Split segs(d_ff, nseg);
  for (int seg = blockIdx.x; seg < nseg; seg += gridDim.x) {
    if (seg != (int)blockIdx.x) __syncthreads();  // the previous segment's LDS reads are done
    const int row0 = segs.start(seg);
    const int nrows = segs.start(seg + 1) - row0;  // <= kSegRowsB, guaranteed by the host

    f32x4_t acc[kTiles][NT];
#pragma unroll
    for (int rt = 0; rt < kTiles; ++rt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[rt][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    {
      int roff[WStage<kTiles, KU, W>::NI];
      stage_rows<kTiles, KU, W>(roff, Cg, [&](int br) { return br < nrows ? row0 + br : -1; });
      int ks0, ks1;
      kpart(Cg, wave, kParts, &ks0, &ks1);
      const Buf gb = make_buf(gate_w, 16u * (uint32_t)d_ff * (uint32_t)(Cg / R8));
      if constexpr (LOPA) {
        const uint32_t part = tok_bytes<W>() * (uint32_t)tc * (uint32_t)Cg;
        ZNorm<NT> zn;
        if constexpr (HAS_G) {
          zn.has_gain = norm && form.rms_gain;
          zn.gain = make_buf(form.rms_gain, tok_bytes<W>() * (uint32_t)Cg);
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) zn.sq[nt] = 0.f;
        }
        stream_rows<kTiles, NT, KU, 2, false, W, HAS_G>(gb, Cg, roff, s_stage[wave], make_buf(zp, 2 * part), part, T,
                                                        ks0, ks1, acc, &zn);
        if constexpr (HAS_G) {
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            float q = zn.sq[nt];
            q += __shfl_xor(q, 16);
            q += __shfl_xor(q, 32);
            if (lane < 16) s_zsq[wave][16 * nt + lane] = q;
          }
        }
      } else {
        stream_rows<kTiles, NT, KU, 1, PRE, W>(gb, Cg, roff, s_stage[wave], tok.b, tok.part, tok.tn, ks0, ks1, acc);
      }
    }
    // LoPA's fixed term (G x) of the rows and tokens this lane thresholds, written by the z
    // kernel's extra workgroups: loaded after the gate stream (no registers held across
    // it), so that the wait falls after the LDS reduction
    uint32_t gxb[HAS_G ? NT : 1][4] = {};
    if constexpr (HAS_G) {
      const Buf xb = make_buf(gx, 4u * (uint32_t)tc * (uint32_t)d_ff);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int tok = 16 * nt + m, rl = 16 * wave + 4 * g + i;
          gxb[nt][i] = ldb32(xb, has_g && tok < T && rl < nrows ? 4u * ((uint32_t)tok * (uint32_t)d_ff + (uint32_t)(row0 + rl))
                                                        : kOOB);
        }
    }
    // quantized: the row scales of the rows this lane thresholds (likewise after the stream)
    uint32_t sgb[Q ? 4 : 1] = {};
    if constexpr (Q) {
      const Buf qb = make_buf(s_g, 4u * (uint32_t)d_ff);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int rl = 16 * wave + 4 * g + i;
        sgb[i] = ldb32(qb, rl < nrows ? 4u * (uint32_t)(row0 + rl) : kOOB);
      }
    }
#pragma unroll
    for (int rt = 0; rt < kTiles; ++rt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) s_red[wave][rt][nt][lane] = acc[rt][nt];
    __syncthreads();
    {
      // lane holds h of rows 16 wave + 4g + i (i < 4) for tokens 16 nt + m
      f32x4_t h[NT];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        h[nt] = ((s_red[0][wave][nt][lane] + s_red[1][wave][nt][lane]) + s_red[2][wave][nt][lane]) +
                s_red[3][wave][nt][lane];
      float inv[HAS_G ? NT : 1];
      if constexpr (HAS_G) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const int o = 16 * nt + m;
          const float q = ((s_zsq[0][o] + s_zsq[1][o]) + s_zsq[2][o]) + s_zsq[3][o];
          inv[nt] = norm ? 1.f / sqrtf(q / (float)(Cg * tile_elems<W>()) + form.rms_eps) : 1.f;
        }
      }
      uint32_t mask = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int rl = 16 * wave + 4 * g + i;
        bool any = false;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const int tok = 16 * nt + m;
          float hv = h[nt][i];
          if constexpr (Q) hv *= __builtin_bit_cast(float, sgb[i]);
          if constexpr (HAS_G) hv *= inv[nt];
          if constexpr (HAS_G) hv += __builtin_bit_cast(float, gxb[nt][i]);  // h += G x
          const bool on = tok < T && hv > t;
          if (tok < T && rl < nrows) s_act[rl][tok] = on ? (FULL ? gate_value(form.act, hv - t) : hv - t) : 0.f;
          any |= on;
        }
        const uint64_t b = __ballot(any && rl < nrows);
#pragma unroll
        for (int gg = 0; gg < 4; ++gg)
          if ((b >> (16 * gg)) & 0xffffull) mask |= 1u << (4 * gg + i);
      }
      if (lane == 0) s_mask[wave] = mask;
    }
    __syncthreads();
    if (wave == 0) {
      const uint64_t on = (uint64_t)s_mask[0] | ((uint64_t)s_mask[1] << 16) | ((uint64_t)s_mask[2] << 32) |
                          ((uint64_t)s_mask[3] << 48);
      const bool sel = lane < nrows && (DENSE || ((on >> lane) & 1ull));
      const uint64_t b = __ballot(sel);
      const int rank = rank_in_mask(b);
      if (sel) {
        s_list[rank] = lane;
        seg_idx[row0 + rank] = row0 + lane;
      }
      if (lane == 0) {
        s_cnt = __popcll(b);
        seg_count[seg] = __popcll(b);
      }
    }
    __syncthreads();
    const int cnt = uniform(s_cnt);
    for (int o = threadIdx.x; o < cnt * T; o += kBlock) {
      const int tok = o / cnt, e = o - tok * cnt;
      seg_act[(size_t)tok * slots + row0 + e] = s_act[s_list[e]][tok];
    }

    // W_up dots of the union rows: tiles of 16 entries
    const int nut = (cnt + 15) / 16;
#pragma unroll
    for (int rt = 0; rt < kTiles; ++rt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[rt][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (nut > 0) {
      int ks0, ks1;
      kpart(Cu, wave, kParts, &ks0, &ks1);
      auto up_row = [&](int e) { return e < cnt ? row0 + s_list[e] : -1; };
      auto full = [&] {
        int roff[WStage<kTiles, KUU, W>::NI];
        stage_rows<kTiles, KUU, W>(roff, Cu, up_row);
        stream_rows<kTiles, NT, KUU, 1, PRE, W>(ub, Cu, roff, s_stage[wave], tok.b, tok.part, tok.tn, ks0, ks1, acc);
      };
      if constexpr (NARROW) {
        if (nut <= 2) {
          int roff[WStage<2, 2 * KUU, W>::NI];
          stage_rows<2, 2 * KUU, W>(roff, Cu, up_row);
          stream_rows<2, NT, 2 * KUU, 1, false, W>(ub, Cu, roff, s_stage[wave], tok.b, tok.part, tok.tn, ks0, ks1,
                                                   reinterpret_cast<f32x4_t(&)[2][NT]>(acc));
        } else {
          full();
        }
      } else {
        full();
      }
    }
#pragma unroll
    for (int rt = 0; rt < kTiles; ++rt)
      if (rt < nut)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) s_red[wave][rt][nt][lane] = acc[rt][nt];
    __syncthreads();

    // wave w: union entries 16 w .. 16 w + 15, lane m + 16 g the quad of entries 16 w + 4 g ..
    // quantized: the W_up scale of each entry's row, and its W_down scale folded into zval
    float sue[4] = {1.f, 1.f, 1.f, 1.f}, sde[4] = {1.f, 1.f, 1.f, 1.f};
    if constexpr (Q) {
      const Buf ubs = make_buf(s_up, 4u * (uint32_t)d_ff), dbs = make_buf(s_down, 4u * (uint32_t)d_ff);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int e = 16 * wave + 4 * g + i;
        const uint32_t off = e < cnt ? 4u * (uint32_t)(row0 + s_list[e < cnt ? e : 0]) : kOOB;
        sue[i] = __builtin_bit_cast(float, ldb32(ubs, off));
        sde[i] = __builtin_bit_cast(float, ldb32(dbs, off));
      }
    }
    bool nz[4] = {DENSE, DENSE, DENSE, DENSE};  // fp32 weights: the lane's entries, for its tokens
    if (16 * wave + 4 * g < cnt) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int tok = 16 * nt + m;
        f32x4_t v = {0.f, 0.f, 0.f, 0.f};
        if (wave < nut)
          v = ((s_red[0][wave][nt][lane] + s_red[1][wave][nt][lane]) + s_red[2][wave][nt][lane]) +
              s_red[3][wave][nt][lane];
        if (tok < T) {
          uint32_t hw[2] = {0u, 0u}, lw[2] = {0u, 0u};
          f32x4_t zv;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int e = 16 * wave + 4 * g + i;
            const float vu = Q ? v[i] * sue[i] : v[i];
            float zz = e < cnt ? s_act[s_list[e]][tok] * (FULL ? up_value(form.silu_up, vu) : vu) : 0.f;
            if constexpr (Q) zz *= sde[i];
            zv[i] = zz;
            nz[i] |= zz != 0.f;
            const __bf16 hb = (__bf16)zz;
            const __bf16 lb = (__bf16)(zz - (float)hb);
            hw[i >> 1] |= (uint32_t)__builtin_bit_cast(uint16_t, hb) << (16 * (i & 1));
            lw[i >> 1] |= (uint32_t)__builtin_bit_cast(uint16_t, lb) << (16 * (i & 1));
          }
          zf[(((size_t)seg * qps + 4 * wave + g) * ntt + nt) * 16 + m] =
              is_f32<W>() ? __builtin_bit_cast(uint4, zv) : make_uint4(hw[0], hw[1], lw[0], lw[1]);
        }
      }
    }
    if constexpr (is_f32<W>()) put_alive(alive + 4 * seg + wave, nz);
  }
}

#define FFN_GATE_UP_PARAMS                                                                                         \
  const float *__restrict__ x, const float *__restrict__ zp, const uint4 *__restrict__ gate_w, int Cg,             \
      const uint4 *__restrict__ w_up, int Cu, int T, int d, int d_ff, int nseg, float t, int slots, int tc,       \
      int32_t *__restrict__ meta, int32_t *__restrict__ seg_count, int32_t *__restrict__ seg_idx,                  \
      float *__restrict__ seg_act, uint4 *__restrict__ zf, float *__restrict__ y, const uint4 *__restrict__ xs,  \
      int ntt, Form form, const float *__restrict__ gx, const float *__restrict__ s_g,                            \
      const float *__restrict__ s_up, const float *__restrict__ s_down, uint16_t *__restrict__ alive, int qps
#define FFN_GATE_UP_ARGS                                                                                            \
  x, zp, gate_w, Cg, w_up, Cu, T, d, d_ff, nseg, t, slots, tc, meta, seg_count, seg_idx, seg_act, zf, y, xs, ntt, form, \
      gx, s_g, s_up, s_down, alive, qps

// One workgroup per CU: four k steps a group for one token tile (two for LoPA's short
// gate rows and for wider token tiles; one for LoPA's gate rows with four token tiles,
// whose fragments carry both partial copies of z).
template <class W, bool LOPA, bool DENSE, int NT, int FORM>
__global__ __launch_bounds__(kBlock) void k_gate_up_mfma(FFN_GATE_UP_PARAMS) {
  constexpr int KU = NT == 1 ? (LOPA ? 2 : 4) : (LOPA && NT == 4 && !is_f32<W>() ? 1 : 2);
  gate_up_body<W, LOPA, DENSE, NT, KU, NT == 1 ? 4 : 2, FORM>(FFN_GATE_UP_ARGS);
}

// One token tile: two k steps a group, so that two workgroups fit a CU (at most 256
// registers a lane); one workgroup's phase changes (LDS reductions, union) then overlap the
// other's streaming.  LoPA's gate rows keep two k steps a group as in k_gate_up_mfma.
template <class W, bool LOPA, bool DENSE, int FORM>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2))) void k_gate_up_mfma2(
    FFN_GATE_UP_PARAMS) {
  gate_up_body<W, LOPA, DENSE, 1, 2, 2, FORM>(FFN_GATE_UP_ARGS);
}
// ------------------------------------------------------------------ batches of 2 .. 4 tokens
// For at most four tokens the gate and the W_up dots run on v_mfma_f32_4x4x4_16b_bf16 (fp32 rows:
// v_mfma_f32_4x4x1_16b_f32, four a chunk; d 3840, d_ff 14231, LoPA r = 480, 2 / 4 tokens 31.7 /
// 33.3 us on the 16x16x4 kernel -> 21.5 / 27.2 us):
// sixteen independent 4x4x4 products an instruction, in which lane 4b + i holds 4
// consecutive k of row i of block b (A operand), lane 4b + j those of token j (B operand),
// and element i of lane 4b + j receives D[b][i][j].  One load instruction of a quad (four
// rows) gives lane 4b + i the 16-byte chunk b of 16 consecutive chunks of row i: 256
// contiguous bytes a row, already in the A layout (its 8 bf16, or 16 / 32 codes converted
// to bf16, feed 2 / 4 / 8 products), so rows need no reshaping through LDS and a quad of
// union rows is any four rows.  The 16 blocks hold disjoint k ranges of the same 4 x 4
// product and are summed once the quad is done.  The tokens (x, and LoPA's z: the sum of the
// z kernel's two partial copies) sit in LDS, split once per workgroup into bf16 hi + lo in
// the order the lanes read them, so the streams load nothing but weights.  Eight waves a workgroup with four loads in flight each (32 KB a CU) measured
// fastest: at 8B int8 / int4 and four tokens the gate kernel took 22.6 / 22.5 us, against
// 26.1 / 25.9 us with sixteen waves and eight loads, 30.2 / 28.2 us with sixteen and twelve,
// and 33.3 / 28.2 us with four waves and four loads.  Tokens past the batch are zeros (a batch
// of 2 or 3 tokens leaves lanes idle).
// Against the 16x16x32 kernel at four tokens on the 8B shape: standard gating with int8 /
// int4 rows 42.1 / 41.9 -> 32.6 / 32.1 us a call; LoPA (r = 512) with bf16 / int8 / int4 rows
// 38.4 / 34.7 / 34.3 -> 37.7 / 31.8 / 31.5 us.
constexpr int kQ4Waves = 8;       // waves a workgroup (one workgroup a CU: two a SIMD)
constexpr int kQ4Threads = kQ4Waves * kWave;
constexpr int kQ4Depth = 4;       // weight loads in flight a wave
constexpr int kQ4MaxX = 4096;     // elements a token: x (d padded to a whole step) ...
constexpr int kQ4MaxZ = 1024;     // ... and LoPA's z (r padded likewise)
constexpr int kQ4Quads = kSegRowsB / 4;

__device__ __forceinline__ short4_t half4(const uint4& v, int h) {
  return __builtin_bit_cast(short4_t, h ? make_uint2(v.z, v.w) : make_uint2(v.x, v.y));
}
__device__ __forceinline__ f32x4_t mfma4(short4_t a, short4_t b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(a, b, c, 0, 0, 0);
}

// One step of a quad: the weight chunk v (8 elements a 16-byte group J) against the token
// fragment at t: t[f kWave], f < FW / 2 the hi parts, then as many lo parts.  Four accumulators take the
// hi and lo products of the two k halves of each group, so that no product waits on the
// one before it.
// fp32 rows: component c of the chunk in accumulator c (products of one k: 4x4x1).
template <class W>
__device__ __forceinline__ void q4_mma(const uint4& v, const uint4* __restrict__ t, f32x4_t (&acc)[4]) {
  if constexpr (is_f32<W>()) {
    const uint4 b = t[0];
    acc[0] = __builtin_amdgcn_mfma_f32_4x4x1f32(comp<0>(v), comp<0>(b), acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_4x4x1f32(comp<1>(v), comp<1>(b), acc[1], 0, 0, 0);
    acc[2] = __builtin_amdgcn_mfma_f32_4x4x1f32(comp<2>(v), comp<2>(b), acc[2], 0, 0, 0);
    acc[3] = __builtin_amdgcn_mfma_f32_4x4x1f32(comp<3>(v), comp<3>(b), acc[3], 0, 0, 0);
    return;
  } else {
  constexpr int G8 = W::EPC / 8, FW = W::EPC / 4;
  auto one = [&](const uint4& w, const uint4& th, const uint4& tl) {
    acc[0] = mfma4(half4(w, 0), half4(th, 0), acc[0]);
    acc[1] = mfma4(half4(w, 0), half4(tl, 0), acc[1]);
    acc[2] = mfma4(half4(w, 1), half4(th, 1), acc[2]);
    acc[3] = mfma4(half4(w, 1), half4(tl, 1), acc[3]);
  };
  one(bf16_chunk<W, 0>(v), t[0], t[(FW / 2) * kWave]);
  if constexpr (G8 > 1) one(bf16_chunk<W, 1>(v), t[kWave], t[(FW / 2 + 1) * kWave]);
  if constexpr (G8 > 2) {
    one(bf16_chunk<W, 2>(v), t[2 * kWave], t[(FW / 2 + 2) * kWave]);
    one(bf16_chunk<W, 3>(v), t[3 * kWave], t[(FW / 2 + 3) * kWave]);
  }
  }
}

// Items [i0, i1) of a quad stream: item it is step it % ns of quad it / ns; a step is 16
// chunks of a row (C chunks a row, ns = ceil(C / 16) steps).  row_of(q) is this lane's row
// of quad q (row lane & 3 of the quad), or -1.  The weights of item it + kQ4Depth are
// requested when item it has been multiplied; items past i1 load nothing.  deposit(q, s)
// receives the quad's 4 x 4 sums in lanes 0..3 (lane j: s[i] = row i . token j) when the
// stream leaves quad q.  stage() runs once the first loads are out, in every thread.
template <class W, class RowOf, class Stage, class Deposit>
__device__ __forceinline__ void q4_stream(const Buf& wb, int C, int ns, int i0, int i1,
                                          const uint4* __restrict__ tok, RowOf row_of, Stage stage,
                                          Deposit deposit) {
  constexpr int D = kQ4Depth, FW = W::EPC / 4;
  const int lane = lane_id(), b = lane >> 2;
  uint4 wv[D];
  int lq = i0 / ns, ls = i0 - lq * ns;
  int lrow = row_of(lq);
  auto issue = [&](int u, bool live) {
    const int ch = 16 * ls + b;
    wv[u] = ldb_nt(wb, live && lrow >= 0 && ch < C ? 16u * ((uint32_t)lrow * (uint32_t)C + (uint32_t)ch) : kOOB);
    if (live && ++ls == ns) {
      ls = 0;
      lrow = row_of(++lq);
    }
  };
  int cq = i0 / ns, cs = i0 - cq * ns;
#pragma unroll
  for (int u = 0; u < D; ++u) issue(u, i0 + u < i1);
  stage();
  f32x4_t acc[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) acc[a] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  auto flush = [&] {
    f32x4_t s = (acc[0] + acc[1]) + (acc[2] + acc[3]);
#pragma unroll
    for (int o = 4; o < kWave; o <<= 1)
#pragma unroll
      for (int i = 0; i < 4; ++i) s[i] += __shfl_xor(s[i], o);
    deposit(cq, s);
#pragma unroll
    for (int a = 0; a < 4; ++a) acc[a] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  };
  for (int it = i0; it < i1; it += D) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      if (it + u < i1) {
        q4_mma<W>(wv[u], tok + (size_t)cs * FW * kWave + lane, acc);
        if (++cs == ns) {
          flush();
          cs = 0;
          ++cq;
        }
      }
      issue(u, it + u + D < i1);
    }
  }
  if (cs != 0) flush();  // a quad cut by the end of the range
}

// Tokens into LDS: elements [0, K) of rows j < T of src (row stride `stride` floats; with
// copies = 2 the sum of two partial copies `part` floats apart), split into bf16 hi + lo, for lane 4 ((k / EPC) % 16) + j of step k / (16 EPC): part f of a lane's fragment
// (f < FW / 2 hi, then lo) at uint4 (step FW + f) kWave + lane, so that the lanes of a
// wave read 16 consecutive bytes each.  Zeros up to Kp (a whole number of steps) and for
// rows j >= T.  A region of Kp elements takes Kp uint4.  UMAX: the most 8-element units
// a thread takes (4 Kp / 8 <= UMAX kQ4Threads).  The loads are issued by q4_load_tokens and
// the values stored by q4_store_tokens, so that other loads can go out in between.
template <class W, int UMAX>
__device__ __forceinline__ void q4_load_tokens(const float* __restrict__ src, int T, int K, int Kp, int stride,
                                               float4 (&v)[UMAX][2], int copies = 1, uint32_t part = 0) {
  const Buf sb = make_buf(src, 4u * (copies == 2 ? 2u * part : (uint32_t)T * (uint32_t)stride));
  const int nu = 4 * (Kp / 8);
#pragma unroll
  for (int u = 0; u < UMAX; ++u) {
    const int unit = threadIdx.x + u * kQ4Threads, j = unit % 4, k = 8 * (unit / 4);
    const bool ok = unit < nu && j < T && k < K;
    const uint32_t off = ok ? 4u * ((uint32_t)j * (uint32_t)stride + (uint32_t)k) : kOOB;
    const bool ok2 = ok && (W::EPC > 4 || k + 4 < K);  // fp32 rows may end in half a unit
    const uint32_t off2 = ok2 ? off + 16 : kOOB;
    float4 a = __builtin_bit_cast(float4, ldb(sb, off)), c = __builtin_bit_cast(float4, ldb(sb, off2));
    if (copies == 2) {
      const float4 a2 = __builtin_bit_cast(float4, ldb(sb, ok ? off + 4u * part : kOOB));
      const float4 c2 = __builtin_bit_cast(float4, ldb(sb, ok2 ? off2 + 4u * part : kOOB));
      a = make_float4(a.x + a2.x, a.y + a2.y, a.z + a2.z, a.w + a2.w);
      c = make_float4(c.x + c2.x, c.y + c2.y, c.z + c2.z, c.w + c2.w);
    }
    v[u][0] = a;
    v[u][1] = c;
  }
}
template <class W, int UMAX>
__device__ __forceinline__ void q4_store_tokens(const float4 (&v)[UMAX][2], int Kp, uint4* __restrict__ tok) {
  constexpr int EPC = W::EPC, FW = EPC / 4;
  const int nu = 4 * (Kp / 8);
#pragma unroll
  for (int u = 0; u < UMAX; ++u) {
    const int unit = threadIdx.x + u * kQ4Threads, j = unit % 4, k = 8 * (unit / 4);
    if (is_f32<W>() && unit < nu) {  // two chunks of 4
      uint4* p = tok + (size_t)(k / (16 * EPC)) * kWave + 4 * ((k / EPC) % 16) + j;
      p[0] = __builtin_bit_cast(uint4, v[u][0]);
      p[4] = __builtin_bit_cast(uint4, v[u][1]);
    } else if (unit < nu) {
      const float f[8] = {v[u][0].x, v[u][0].y, v[u][0].z, v[u][0].w, v[u][1].x, v[u][1].y, v[u][1].z, v[u][1].w};
      bf16x8_t hi, lo;
      split8(f, hi, lo);
      const int step = k / (16 * EPC), bb = (k / EPC) % 16, grp = (k % EPC) / 8;
      uint4* p = tok + (size_t)step * FW * kWave + 4 * bb + j;
      p[grp * kWave] = __builtin_bit_cast(uint4, hi);
      p[(FW / 2 + grp) * kWave] = __builtin_bit_cast(uint4, lo);
    }
  }
}

// Gate, union and W_up dots of one segment for batches of at most four tokens (the same
// outputs as gate_up_body with one token tile).  Every wave takes an equal share of the
// segment's (quad, step) items, so a quad may be split between waves: each wave leaves its
// partial sums in its own LDS slots and the slots are added in a fixed order.
template <class W, bool LOPA, bool DENSE, int FORM>
__global__ __launch_bounds__(kQ4Threads) void k_gate_up_q4(FFN_GATE_UP_PARAMS) {
  constexpr int EPC = W::EPC, STEP = 16 * EPC;
  constexpr bool Q = is_quant<W>();
  constexpr bool FULL = FORM != kFormDefault, HAS_G = FORM == kFormLoPA;
  constexpr int UX = 4 * kQ4MaxX / 8 / kQ4Threads, UZ = LOPA ? (4 * kQ4MaxZ / 8 + kQ4Threads - 1) / kQ4Threads : 1;
  __shared__ uint4 s_tok[kQ4MaxX + (LOPA ? kQ4MaxZ : 0)];
  // partial sums [wave][quad][token] (element i: row i of the quad) of the gate and W_up
  __shared__ f32x4_t s_pg[kQ4Waves][kQ4Quads][4], s_pu[kQ4Waves][kQ4Quads][4];
  __shared__ float s_act[kSegRowsB][4];
  __shared__ int s_list[kSegRowsB];
  __shared__ int s_cnt;
  __shared__ float s_zsq[HAS_G ? kQ4Waves : 1][4];  // sums of z^2 of the waves' shares
  const bool norm = HAS_G && form.rms_eps > 0.f, has_g = HAS_G && form.g_idx;

  const int lane = lane_id(), wave = uniform(threadIdx.x / kWave);
  for (int j = blockIdx.x * kQ4Threads + threadIdx.x; j < T * d; j += gridDim.x * kQ4Threads) y[j] = 0.f;
  if (blockIdx.x == 0 && threadIdx.x == 0) meta[0] = nseg;
  constexpr int TE = tile_elems<W>();
  const int Cu_ = Cu / (EPC / TE), Cg_ = Cg / (EPC / TE);
  const int nsu = (Cu_ + 15) / 16, Kpx = nsu * STEP, nsg = (Cg_ + 15) / 16, Kpz = LOPA ? nsg * STEP : 0;
  uint4* const tok_g = s_tok + (LOPA ? Kpx : 0);
  const Buf gb = make_buf(gate_w, 16u * (uint32_t)d_ff * (uint32_t)Cg_);
  const Buf ub = make_buf(w_up, 16u * (uint32_t)d_ff * (uint32_t)Cu_);
  auto deposit_g = [&](int q, const f32x4_t& s) {
    if (lane < 4) s_pg[wave][q][lane] = s;
  };
  auto deposit_u = [&](int q, const f32x4_t& s) {
    if (lane < 4) s_pu[wave][q][lane] = s;
  };

  const Split segs(d_ff, nseg);
  bool staged = false;
  for (int seg = blockIdx.x; seg < nseg; seg += gridDim.x) {
    __syncthreads();  // the previous segment's LDS reads are done
    const int row0 = segs.start(seg);
    const int nrows = segs.start(seg + 1) - row0;  // <= kSegRowsB, guaranteed by the host
    for (int o = threadIdx.x; o < kQ4Waves * kQ4Quads * 4; o += kQ4Threads) {
      (&s_pg[0][0][0])[o] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      (&s_pu[0][0][0])[o] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    __syncthreads();
    {
      const int n = ((nrows + 3) / 4) * nsg;
      const int i0 = (int)((int64_t)n * wave / kQ4Waves), i1 = (int)((int64_t)n * (wave + 1) / kQ4Waves);
      auto row_of = [&](int q) {
        const int rl = 4 * q + (lane & 3);
        return rl < nrows ? row0 + rl : -1;
      };
      auto stage = [&] {
        if (staged) return;
        staged = true;
        float4 vx[UX][2];
        q4_load_tokens<W, UX>(x, T, d, Kpx, d, vx);
        float4 vz[UZ][2];
        if constexpr (LOPA) q4_load_tokens<W, UZ>(zp, T, Cg * TE, Kpz, Cg * TE, vz, 2, (uint32_t)(tc * Cg * TE));
        if constexpr (HAS_G) {  // squares and gains of this thread's components of z (token threadIdx.x % 4)
          float4 gn[UZ][2];
          const bool has_gain = norm && form.rms_gain;
          const Buf nb = make_buf(form.rms_gain, 4u * (uint32_t)(Cg * TE));
          float sq = 0.f;
#pragma unroll
          for (int u = 0; u < UZ; ++u) {
            const int k = 8 * (((int)threadIdx.x + u * kQ4Threads) / 4);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              gn[u][h] = __builtin_bit_cast(float4, ldb(nb, has_gain && k + 4 * h < Cg * TE ? 4u * (uint32_t)(k + 4 * h) : kOOB));
              const float4 z = vz[u][h];
              sq = fmaf(z.x, z.x, fmaf(z.y, z.y, fmaf(z.z, z.z, fmaf(z.w, z.w, sq))));
            }
          }
          if (has_gain) {
#pragma unroll
            for (int u = 0; u < UZ; ++u)
#pragma unroll
              for (int h = 0; h < 2; ++h)
                vz[u][h] = make_float4(vz[u][h].x * gn[u][h].x, vz[u][h].y * gn[u][h].y, vz[u][h].z * gn[u][h].z,
                                       vz[u][h].w * gn[u][h].w);
          }
#pragma unroll
          for (int o = 4; o < kWave; o <<= 1) sq += __shfl_xor(sq, o);
          if (lane < 4) s_zsq[wave][lane] = sq;
        }
        q4_store_tokens<W, UX>(vx, Kpx, s_tok);
        if constexpr (LOPA) q4_store_tokens<W, UZ>(vz, Kpz, tok_g);
        __syncthreads();
      };
      if (i0 < i1)
        q4_stream<W>(gb, Cg_, nsg, i0, i1, tok_g, row_of, stage, deposit_g);
      else
        stage();
    }
    // the row scale of the row this lane of wave 0 thresholds
    float sg = 1.f, gxv[4] = {0.f, 0.f, 0.f, 0.f};
    if constexpr (Q)
      if (wave == 0)
        sg = __int_as_float(ldb32(make_buf(s_g, 4u * (uint32_t)d_ff), lane < nrows ? 4u * (uint32_t)(row0 + lane) : kOOB));
    if constexpr (HAS_G)
      if (wave == 0) {
        const Buf xb = make_buf(gx, 4u * (uint32_t)tc * (uint32_t)d_ff);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          gxv[j] = __int_as_float(
              ldb32(xb, has_g && j < T && lane < nrows ? 4u * ((uint32_t)j * (uint32_t)d_ff + (uint32_t)(row0 + lane)) : kOOB));
      }
    __syncthreads();
    if (wave == 0) {
      // lane: row `lane` of the segment
      const int q = lane >> 2, i = lane & 3;
      bool any = false;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float hv = 0.f;
#pragma unroll
        for (int w = 0; w < kQ4Waves; ++w) hv += s_pg[w][q][j][i];
        if constexpr (Q) hv *= sg;
        if constexpr (HAS_G)
          if (norm) {
            float q = 0.f;
#pragma unroll
            for (int w = 0; w < kQ4Waves; ++w) q += s_zsq[w][j];
            hv *= 1.f / sqrtf(q / (float)(Cg * TE) + form.rms_eps);
          }
        if constexpr (HAS_G) hv += gxv[j];
        const bool on = j < T && hv > t;
        if (lane < nrows) s_act[lane][j] = on ? (FULL ? gate_value(form.act, hv - t) : hv - t) : 0.f;
        any |= on;
      }
      const bool sel = lane < nrows && (DENSE || any);
      const uint64_t bm = __ballot(sel);
      const int rank = rank_in_mask(bm);
      if (sel) {
        s_list[rank] = lane;
        seg_idx[row0 + rank] = row0 + lane;
      }
      if (lane == 0) {
        s_cnt = __popcll(bm);
        seg_count[seg] = __popcll(bm);
      }
    }
    __syncthreads();
    const int cnt = uniform(s_cnt);
    for (int o = threadIdx.x; o < cnt * T; o += kQ4Threads) {
      const int tk = o / cnt, e = o - tk * cnt;
      seg_act[(size_t)tk * slots + row0 + e] = s_act[s_list[e]][tk];
    }
    {
      const int n = ((cnt + 3) / 4) * nsu;
      const int i0 = (int)((int64_t)n * wave / kQ4Waves), i1 = (int)((int64_t)n * (wave + 1) / kQ4Waves);
      auto row_of = [&](int q) {
        const int e = 4 * q + (lane & 3);
        return e < cnt ? row0 + s_list[e] : -1;
      };
      if (i0 < i1) q4_stream<W>(ub, Cu_, nsu, i0, i1, s_tok, row_of, [] {}, deposit_u);
    }
    __syncthreads();

    // wave w < 4: union entries 16 w .. 16 w + 15, lane m + 16 g: token m, quad 4 w + g
    const int m = lane & 15, g = lane >> 4;
    float sue[4] = {1.f, 1.f, 1.f, 1.f}, sde[4] = {1.f, 1.f, 1.f, 1.f};
    if constexpr (Q) {
      const Buf ubs = make_buf(s_up, 4u * (uint32_t)d_ff), dbs = make_buf(s_down, 4u * (uint32_t)d_ff);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int e = 16 * (wave & 3) + 4 * g + i;
        const uint32_t off = e < cnt ? 4u * (uint32_t)(row0 + s_list[e < cnt ? e : 0]) : kOOB;
        sue[i] = __int_as_float(ldb32(ubs, off));
        sde[i] = __int_as_float(ldb32(dbs, off));
      }
    }
    bool nz[4] = {DENSE, DENSE, DENSE, DENSE};
    if (wave < 4 && 16 * wave + 4 * g < cnt && m < T) {
      const int qq = 4 * wave + g;  // the quad of entries 16 w + 4 g ..
      f32x4_t v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < kQ4Waves; ++w) v += s_pu[w][qq][m];
      uint32_t hw[2] = {0u, 0u}, lw[2] = {0u, 0u};
      f32x4_t zv;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int e = 16 * wave + 4 * g + i;
        const float vu = Q ? v[i] * sue[i] : v[i];
        float zz = e < cnt ? s_act[s_list[e]][m] * (FULL ? up_value(form.silu_up, vu) : vu) : 0.f;
        if constexpr (Q) zz *= sde[i];
        zv[i] = zz;
        nz[i] |= zz != 0.f;
        const __bf16 hb = (__bf16)zz;
        const __bf16 lb = (__bf16)(zz - (float)hb);
        hw[i >> 1] |= (uint32_t)__builtin_bit_cast(uint16_t, hb) << (16 * (i & 1));
        lw[i >> 1] |= (uint32_t)__builtin_bit_cast(uint16_t, lb) << (16 * (i & 1));
      }
      zf[((size_t)seg * qps + qq) * ntt * 16 + m] =
          is_f32<W>() ? __builtin_bit_cast(uint4, zv) : make_uint4(hw[0], hw[1], lw[0], lw[1]);
    }
    if constexpr (is_f32<W>())
      if (wave < 4) put_alive(alive + 4 * seg + wave, nz);
  }
}

#undef FFN_GATE_UP_PARAMS
#undef FFN_GATE_UP_ARGS

// ------------------------------------------------------------------ down projection
// Workgroup b: column group b % S, row chunk b / S (a balanced share of the segments).
// A wave owns DT 32-column tiles (DT = 4 for one token tile, else 2); a column group
// is CW of them, and wave w takes column slot w % CW and every (4 / CW)-th group of the
// chunk.  The chunk's union entries are packed into groups of 32: each segment's list is
// padded to whole quads of entries and the quads of all segments follow one another, eight a
// group.  (A group had been 32 entries of one segment, where at two to four tokens and 90% a
// segment's 11 - 20 entries left most of it empty: fp32 rows, d 3840, d_ff 14231, 2 / 4 tokens
// 22.6 / 24.5 -> 15.2 / 20.5 us; bf16 rows, 4 tokens 15.3 -> 14.5 us, 64 tokens 0.7 us less.)
// A group's 32 W_down rows are read (64 / 4 DT) rows x 64 DT bytes per instruction, streamed
// past the caches, and written to a wave-private LDS tile; transposing LDS reads
// (ds_read_b64_tr_b16) then hand every lane the 8 entries of one column that the
// matrix-core B operand takes (fp32 weights: see dn_mma).  The packed rows and their zval
// quads are listed in LDS once; the loop reads a group's entries one group ahead, so the
// weight loads of the next group issue without waiting on LDS.  The waves' sums meet in LDS,
// then go to y with one fp32 atomic per token and column (y was cleared by the gate kernel).
constexpr int kDnSlots = 4096;  // most rows of one row chunk
// LDS entries of the packed list: the rows, up to three pad entries a segment (at most kBlock
// segments), and empty entries to the end of the last group
constexpr int kDnList = kDnSlots + 3 * kBlock + 32;

template <int NT, class W = WBf16>
struct DnCfg {
  static constexpr bool F32 = is_f32<W>();
  static constexpr int DT = NT == 1 && !F32 ? 4 : 2;  // 32-column tiles per wave
  static constexpr int CW = NT == 4 ? 1 : 2;  // column slots per workgroup
  static constexpr int WCOLS = 32 * DT * CW;  // columns per workgroup
  static constexpr int R8 = W::EPC / tile_elems<W>();  // tile chunks per loaded chunk
  static constexpr int LPR = 32 * DT / W::EPC;  // lanes per row of a load instruction
  static constexpr int RPI = kWave / LPR;     // rows per load instruction
  static constexpr int NI = 32 / RPI;         // load instructions per group
  // chunks per LDS row: two pad chunks put the 8 rows that a half-wave's transposing
  // reads touch on distinct banks
  static constexpr int PITCH = F32 ? 0 : 4 * DT + 2;
  // the entry of a group that lane `lane` loads with instruction i
  static __device__ __forceinline__ int entry(int i, int lane) {
    return F32 ? 16 * (i >> 2) + 4 * (lane >> 4) + (i & 3) : RPI * i + lane / LPR;
  }
};

template <int NT, class W = WBf16>
struct DnFrags {
  uint4 t[DnCfg<NT, W>::NI];  // W_down chunks as loaded: entry RPI i + lane / LPR, chunk lane % LPR
  u32x4_t z[NT][2];           // zval quads of the token tiles
};

template <int NT, class W = WBf16>
struct DnRows {
  int row[DnCfg<NT, W>::NI];  // neuron of the entry this lane loads, -1 for none
  int zq[2];                  // zval quads of the lane group: entries 4 g .. and 16 + 4 g .., -1 for none
};

// cv: the lane's chunk is one of the row's.  A group past the ngrp listed ones has no entries.
template <int NT, class W>
__device__ __forceinline__ DnRows<NT, W> dn_rows(int group, int ngrp, const int* s_row, const int* s_zq, bool cv) {
  using K = DnCfg<NT, W>;
  const int lane = lane_id();
  const bool has = group < ngrp, ok = cv && has;
  const int g = has ? group : 0;
  DnRows<NT, W> a;
#pragma unroll
  for (int i = 0; i < K::NI; ++i) {
    const int v = s_row[32 * g + K::entry(i, lane)];
    a.row[i] = ok ? v : -1;
  }
  const int z0 = s_zq[8 * g + (lane >> 4)], z1 = s_zq[8 * g + 4 + (lane >> 4)];
  a.zq[0] = has ? z0 : -1;
  a.zq[1] = has ? z1 : -1;
  return a;
}

template <int NT, class W>
__device__ __forceinline__ void dn_issue(DnFrags<NT, W>& f, const DnRows<NT, W>& a, const Buf& db, const Buf& zb,
                                         int C, int ch, int T, int ntt) {
  using K = DnCfg<NT, W>;
  const int lane = lane_id(), m = lane & 15;
#pragma unroll
  for (int i = 0; i < K::NI; ++i) f.t[i] = ldb_nt(db, a.row[i] >= 0 ? 16u * (uint32_t)(a.row[i] * C + ch) : kOOB);
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int h = 0; h < 2; ++h)
      f.z[nt][h] = __builtin_bit_cast(
          u32x4_t, ldb(zb, a.zq[h] >= 0 && 16 * nt + m < T
                               ? 256u * ((uint32_t)a.zq[h] * (uint32_t)ntt + (uint32_t)nt) + 16u * (uint32_t)m
                               : kOOB));
}

// tile: this wave's LDS tile (32 PITCH uint4).  Within each 16-lane group q of the
// transposing read, lane 4a + b addresses 8 bytes (4 columns) of one tile row and lane
// 4b + c receives element c of the chunks of lanes b, 4 + b, 8 + b, 12 + b.  With lane
// 4a + b pointing at entry 4q + a (then 16 + 4q + a), columns 4b .. 4b + 3 of a 16-column
// block, lane n of the group ends with entries 4q .. 4q + 3 (then 16 + 4q ..) of column
// n: the B operand in the entry order of the zval quads (see DnRows).
template <int NT, class W>
__device__ __forceinline__ void dn_mma(const DnFrags<NT, W>& f, uint4* tile,
                                       f32x4_t (&acc)[DnCfg<NT, W>::DT][2][NT]) {
  using K = DnCfg<NT, W>;
  if constexpr (K::F32) {
    // A lane's 16 bytes of entry e are columns 4 n .. 4 n + 3 (n = lane & 15): component c of
    // load i is the B operand of the product over the entries of load i for the columns 4 n + c,
    // so the rows need no reshaping.  Sums of component c go to acc[c / 2][c % 2], the group's
    // own first (see is_f32).
    f32x4_t grp[4][NT];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) grp[c][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto load = [&](auto ic) {
      constexpr int i = decltype(ic)::value;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const float z = __uint_as_float(f.z[nt][i >> 2][i & 3]);
        grp[0][nt] = mfma16f(z, comp<0>(f.t[i]), grp[0][nt]);
        grp[1][nt] = mfma16f(z, comp<1>(f.t[i]), grp[1][nt]);
        grp[2][nt] = mfma16f(z, comp<2>(f.t[i]), grp[2][nt]);
        grp[3][nt] = mfma16f(z, comp<3>(f.t[i]), grp[3][nt]);
      }
    };
    load(Int<0>{}), load(Int<1>{}), load(Int<2>{}), load(Int<3>{});
    load(Int<4>{}), load(Int<5>{}), load(Int<6>{}), load(Int<7>{});
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[c / 2][c % 2][nt] += grp[c][nt];
    return;
  } else {
  constexpr int ROWB = 16 * K::PITCH;  // bytes per tile row
  bf16x8_t zh[NT], zl[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    zh[nt] = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(f.z[nt][0], f.z[nt][1], 0, 1, 4, 5));
    zl[nt] = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(f.z[nt][0], f.z[nt][1], 2, 3, 6, 7));
  }
  const int lane = lane_id();
#pragma unroll
  for (int i = 0; i < K::NI; ++i)  // quantized rows: the codes as bf16, R8 tile chunks a loaded chunk
    put_bf16_chunks<W>(tile + (K::RPI * i + lane / K::LPR) * K::PITCH + (lane % K::LPR) * K::R8, f.t[i]);
  __builtin_amdgcn_wave_barrier();  // LDS operations of a wave complete in order
  const char* src = reinterpret_cast<const char*>(tile) + (4 * (lane >> 4) + ((lane >> 2) & 3)) * ROWB + 8 * (lane & 3);
#pragma unroll
  for (int ct = 0; ct < K::DT; ++ct)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint2 lo = lds_read_tr16(src + 64 * ct + 32 * h);
      const uint2 hi = lds_read_tr16(src + 16 * ROWB + 64 * ct + 32 * h);
      const bf16x8_t b = bf8(make_uint4(lo.x, lo.y, hi.x, hi.y));
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        acc[ct][h][nt] = mfma16(zh[nt], b, acc[ct][h][nt]);
        acc[ct][h][nt] = mfma16(zl[nt], b, acc[ct][h][nt]);
      }
    }
  __builtin_amdgcn_wave_barrier();
  }
}

// C: loaded chunks per row of w_down_t (d / W::EPC); the W_down row scales of quantized
// weights are folded into zval by the gate kernel.
template <int NT, class W>
__global__ __launch_bounds__(kBlock) void k_down_mfma(const int32_t* __restrict__ seg_count,
                                                      const int32_t* __restrict__ seg_idx,
                                                      const uint4* __restrict__ zf, int nseg, int qps, int d_ff,
                                                      int R, int tc,
                                                      const uint4* __restrict__ w_down_t, int C, int d, int T,
                                                      float* __restrict__ y, const uint2* __restrict__ alive) {
  using K = DnCfg<NT, W>;
  constexpr int CW = K::CW, GS = kParts / CW, WCOLS = K::WCOLS;
  const Buf db = make_buf(w_down_t, 16u * (uint32_t)d_ff * (uint32_t)C);
  const int ntt = (tc + 15) / 16;
  const Buf zb = make_buf(zf, 256u * (uint32_t)(nseg * qps) * (uint32_t)ntt);
  // LDS: the waves' tiles and the chunk's packed list during the loop; afterwards the
  // same space holds every wave's sums, [wave][ct][h][nt][lane] as f32x4
  constexpr int STAGE_U4 = kParts * 32 * K::PITCH, IDX_U4 = (kDnList + kDnList / 4 + 3) / 4;
  constexpr int PART_U4 = kParts * K::DT * 2 * NT * kWave;
  constexpr int BIG_U4 = STAGE_U4 + IDX_U4 > PART_U4 ? STAGE_U4 + IDX_U4 : PART_U4;
  __shared__ uint4 s_big[BIG_U4];
  __shared__ uint2 s_alive[K::F32 ? kBlock : 1];  // fp32 weights: a bit an entry whose row is read
  uint4* const s_stage = s_big;
  int* const s_row = reinterpret_cast<int*>(s_big + STAGE_U4);
  int* const s_zq = s_row + kDnList;
  f32x4_t* const s_part = reinterpret_cast<f32x4_t*>(s_big);

  const int S = (d + WCOLS - 1) / WCOLS;
  const int chunk = blockIdx.x / S, cgrp = blockIdx.x % S;
  const Split chunks(nseg, R), segs(d_ff, nseg);
  const int seg_lo = chunks.start(chunk), seg_hi = chunks.start(chunk + 1);
  const int nsc = seg_hi - seg_lo;  // <= kBlock, guaranteed by the host
  const int row_lo = segs.start(seg_lo);
  const int nslot = segs.start(seg_hi) - row_lo;  // <= kDnSlots, guaranteed by the host
  const int tid = threadIdx.x, lane = lane_id(), wave = uniform(tid / kWave);
  const int slot_w = wave % CW, phase = wave / CW;

  // The packed list: wave w takes the chunk's segments w, w + 4, ..., a lane an entry (segments
  // have at most 64 rows), SU of them in flight.  The first ones are requested ahead of the
  // counts' scan.
  constexpr int SU = 8;
  const Buf ib = make_buf(seg_idx + row_lo, 4u * (uint32_t)nslot);
  auto fetch = [&](int (&v)[SU], int s0) {
#pragma unroll
    for (int u = 0; u < SU; ++u) {
      const int sg = s0 + u * kParts, sl = sg < nsc ? sg : 0;
      const int at = segs.start(seg_lo + sl) - row_lo + lane;
      v[u] = ldb32(ib, sg < nsc && at < nslot ? 4u * (uint32_t)at : kOOB);
    }
  };
  int v0[SU];
  // Every wave scans all counts: lane l those of segments 4 l .. 4 l + 3, so that a segment's place
  // in the list comes from a register of the wave that lists it and no wave waits for another (with a
  // scan over the workgroup, two more barriers and 512 empty entries past the last group: LoPA
  // r = 512 on the 8B shape, 4 tokens, int8 30.9 -> 30.4 us a call, int4 30.3 -> 29.8; bf16 70B shape,
  // r = 1024, 8 tokens 130.8 -> 130.4).
  const Buf cb = make_buf(seg_count + seg_lo, 4u * (uint32_t)nsc);
  int c[kParts], first[kParts];  // entries of segment 4 lane + p, its first quad
#pragma unroll
  for (int p = 0; p < kParts; ++p) c[p] = ldb32(cb, kParts * lane + p < nsc ? 4u * (uint32_t)(kParts * lane + p) : kOOB);
  uint2 live = make_uint2(0u, 0u);
  if constexpr (K::F32)
    if (tid < nsc) live = alive[seg_lo + tid];
  fetch(v0, wave);
  int quads = 0;
#pragma unroll
  for (int p = 0; p < kParts; ++p) {
    first[p] = quads;
    quads += (c[p] + 3) >> 2;
  }
  const int upto = wave_inclusive_scan(quads);
  const int nquad = __builtin_amdgcn_readlane(upto, kWave - 1);
  const int ngrp = (nquad + 7) / 8;
  int cw = c[0], fw = first[0];  // of the wave's segments: 4 lane + wave
#pragma unroll
  for (int p = 1; p < kParts; ++p) {
    cw = wave == p ? c[p] : cw;
    fw = wave == p ? first[p] : fw;
  }
  fw += upto - quads;
  for (int o = 4 * nquad + tid; o < 32 * ngrp; o += kBlock) {
    s_row[o] = -1;
    if ((o & 3) == 0) s_zq[o >> 2] = -1;
  }
  if constexpr (K::F32) {
    s_alive[tid] = live;
    __syncthreads();
  }
  for (int s0 = wave;; s0 += kParts * SU) {
#pragma unroll
    for (int u = 0; u < SU; ++u) {
      const int sg = s0 + u * kParts;
      if (sg < nsc) {
        const int n = __builtin_amdgcn_readlane(cw, sg / kParts);
        const int o = 4 * __builtin_amdgcn_readlane(fw, sg / kParts) + lane;
        if (lane < ((n + 3) & ~3)) {
          bool read = lane < n;
          if constexpr (K::F32) read = read && (((lane < 32 ? s_alive[sg].x : s_alive[sg].y) >> (lane & 31)) & 1u);
          s_row[o] = read ? v0[u] : -1;
          if ((lane & 3) == 0) s_zq[o >> 2] = qps * (seg_lo + sg) + (lane >> 2);
        }
      }
    }
    if (s0 + kParts * SU >= nsc) break;
    fetch(v0, s0 + kParts * SU);
  }
  __syncthreads();

  f32x4_t acc[K::DT][2][NT];
#pragma unroll
  for (int ct = 0; ct < K::DT; ++ct)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[ct][h][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // this lane's 16-byte chunk of the wave's columns
  const int ch = (cgrp * WCOLS + slot_w * 32 * K::DT) / W::EPC + lane % K::LPR;
  if (phase < ngrp) {
    // two register sets alternate, one group each per half-iteration; the list entries of group
    // j + 2 GS are read while group j is multiplied.  A pair always multiplies both halves (a
    // group past the last one loads nothing and adds zeros), so no load sits on a conditional
    // path.
    DnFrags<NT, W> f0, f1;
    DnRows<NT, W> a = dn_rows<NT, W>(phase, ngrp, s_row, s_zq, ch < C);
    dn_issue(f0, a, db, zb, C, ch, T, ntt);
    a = dn_rows<NT, W>(phase + GS, ngrp, s_row, s_zq, ch < C);
    for (int j = phase;; j += 2 * GS) {
      dn_issue(f1, a, db, zb, C, ch, T, ntt);
      issue_barrier();
      a = dn_rows<NT, W>(j + 2 * GS, ngrp, s_row, s_zq, ch < C);
      dn_mma(f0, s_stage + wave * 32 * K::PITCH, acc);
      dn_issue(f0, a, db, zb, C, ch, T, ntt);
      issue_barrier();
      a = dn_rows<NT, W>(j + 3 * GS, ngrp, s_row, s_zq, ch < C);
      dn_mma(f1, s_stage + wave * 32 * K::PITCH, acc);
      if (j + 2 * GS >= ngrp) break;
    }
  }
  // lane m + 16 g of wave w holds tokens 16 nt + 4g .. + 3 of column 32 ct + 16 h + m
  // of slot w % CW; the GS waves of a slot are added in a fixed order, then one fp32
  // atomic per token and column goes to y
  __syncthreads();  // every wave is done with its tile and the slot indices
#pragma unroll
  for (int ct = 0; ct < K::DT; ++ct)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) s_part[(((wave * K::DT + ct) * 2 + h) * NT + nt) * kWave + lane] = acc[ct][h][nt];
  __syncthreads();
  constexpr int NE = CW * K::DT * 2 * NT * kWave;
  for (int o = tid; o < NE; o += kBlock) {
    int l = o % kWave, r = o / kWave;  // r = ((slot DT + ct) 2 + h) NT + nt
    const int nt = r % NT;
    int h = (r / NT) % 2, ct = (r / (2 * NT)) % K::DT;
    const int slot = r / (2 * NT * K::DT);
    int cc = 32 * ct + 16 * h + (l & 15);
    if constexpr (K::F32) {
      // 64 consecutive columns of four tokens: thread l takes column l of the slot, component
      // l % 4 of lane l / 4, and 2 ct + h picks the token quad
      const int q = 2 * ct + h;
      cc = l;
      ct = (l >> 1) & 1, h = l & 1;
      l = (l >> 2) + 16 * q;
    }
    const int tok0 = 16 * nt + 4 * (l >> 4);
    const int col = cgrp * WCOLS + slot * 32 * K::DT + cc;
    if (tok0 >= T || col >= d) continue;
    f32x4_t v = s_part[(((slot * K::DT + ct) * 2 + h) * NT + nt) * kWave + l];
#pragma unroll
    for (int p = 1; p < GS; ++p) v += s_part[((((slot + CW * p) * K::DT + ct) * 2 + h) * NT + nt) * kWave + l];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (tok0 + i < T) unsafeAtomicAdd(y + (size_t)(tok0 + i) * d + col, v[i]);
  }
}

// ------------------------------------------------------------------ host side
// fp32 weights: the entries' alive bits, 8 bytes a segment, in the space of seg_zval, which this path
// does not use otherwise (4 d_ff bytes a token, at least 256; segments are of 64 rows, or at most
// 512 of them where d_ff > 8192)
uint16_t* alive_masks(const Workspace& ws) { return reinterpret_cast<uint16_t*>(ws.seg_zval); }
int token_tiles(const Workspace& ws) { return (ws.tc + 15) / 16; }

template <bool F32>
hipError_t split_tokens(const Shape& sh, const float* x, const Workspace& ws, hipStream_t s) {
  const int C = sh.d / (F32 ? 4 : 8), nks = (C + 3) / 4, ntt = token_tiles(ws);
  const int n = nks * ntt * kWave;
  k_split_tokens<F32><<<(n + kBlock - 1) / kBlock, kBlock, 0, s>>>(x, C, sh.T, nks, ntt, ws.xs);
  return hipGetLastError();
}
template <class W, int NT, bool PRE>
hipError_t z_mfma(const Shape& sh, const Form& form, const float* x, const void* lopa_a, const Workspace& ws,
                  hipStream_t s) {
  const int C = sh.d / tile_elems<W>(), ngrp = PRE ? token_tiles(ws) / NT : 1, grid = ((sh.r + 15) / 16) * kZParts * ngrp;
  // with G, extra workgroups write G x for the gate kernel
  const GWork gw{form, x, ws.gx, sh.T, sh.d, sh.d_ff, grid};
  const int g = grid + (form.g_idx ? (g_items(sh.d_ff, sh.T) + kZWaves * kWave - 1) / (kZWaves * kWave) : 0);
  k_lopa_z_mfma<NT, PRE, W><<<g, kZWaves * kWave, 0, s>>>(x, ws.xs, token_tiles(ws), static_cast<const uint4*>(lopa_a),
                                                      C, sh.T, sh.r, ws.tc, ws.z, gw, sh.sc.a);
  return hipGetLastError();
}

// Row-balanced segments: of at most 64 rows where there are more than 128 of those, in multiples of
// the gate kernel's grid so that every workgroup gets the same number; of a smaller d_ff at most 32
// rows, which reach twice the compute units (90%, calls: bf16 d 2560, d_ff 8100, 16 tokens 41.7 -> 36.5
// us; int8 d 2048, d_ff 7000, 16 tokens 31.4 -> 29.0; fp32 d 2048, d_ff 7000, r 256, 16 tokens 42.9 ->
// 37.5; bf16 d 1024, d_ff 4000, 32 tokens 27.3 -> 24.7, 8 tokens 18.6 -> 19.7).  The 4x4x4 kernel, whose
// workgroups each stage all tokens, keeps 64 rows up to half of that d_ff (int8 d 1024, d_ff 4000,
// r 128, 4 tokens 21.5 us against 22.6 with 32).
constexpr int kSmallDff = 128 * kSegRowsB;
int segments_for(int d_ff, int grid, bool q4 = false) {
  const int n = (d_ff + kSegRowsB - 1) / kSegRowsB;
  if (d_ff > kSmallDff) return (n + grid - 1) / grid * grid;
  return q4 && d_ff <= kSmallDff / 2 ? n : (d_ff + 31) / 32;
}
// zval quads a segment has room for: those of its rows.  nseg seg_quads <= 16 batched_segments(d_ff).
int seg_quads(int d_ff, int nseg) { return ((d_ff + nseg - 1) / nseg + 3) / 4; }

// The 4x4x4 kernel takes batches of at most four tokens whose rows (and LoPA's r), padded to
// a whole step, fit its token LDS.
template <class W>
bool q4_fits(const Shape& sh, bool lopa) {
  const int step = 16 * W::EPC;
  return sh.T <= 4 && (sh.d + step - 1) / step * step <= kQ4MaxX && (!lopa || (sh.r + step - 1) / step * step <= kQ4MaxZ);
}

template <class W, bool LOPA, bool DENSE, int NT, int FORM>
hipError_t gate_mfma(const Shape& sh, const Form& form, const float* x, const void* gate_w, const void* w_up, float t,
                     Workspace& ws, float* y, hipStream_t s) {
  const int Cu = sh.d / tile_elems<W>(), Cg = LOPA ? sh.r / tile_elems<W>() : Cu;
  if constexpr (NT == 1)
    if (q4_fits<W>(sh, LOPA)) {
      ws.nseg = segments_for(sh.d_ff, kSegGrid, true);
      return launch_gate_kernel_n(k_gate_up_q4<W, LOPA, DENSE, FORM>, ws.nseg < kSegGrid ? ws.nseg : kSegGrid,
                                  kQ4Threads, s, x,
                                (const float*)ws.z, static_cast<const uint4*>(gate_w), Cg,
                                static_cast<const uint4*>(w_up), Cu, sh.T, sh.d, sh.d_ff, ws.nseg, t, ws.slots, ws.tc,
                                ws.meta, ws.seg_count, ws.seg_idx, ws.seg_act, ws.zf, y, ws.xs, token_tiles(ws), form,
                                (const float*)ws.gx, LOPA ? sh.sc.b : sh.sc.gate, sh.sc.up, sh.sc.down, alive_masks(ws), seg_quads(sh.d_ff, ws.nseg));
    }
  // The two-workgroup kernel (two k steps a load group) takes segments that stay near 64 rows,
  // d_ff >= 24576: halving 8B-shaped bf16 / int8 / int4 segments to 28 rows left the row tiles half empty
  // (int8 / int4 at four tokens, on these kernels: 52.7 / 54.4 us a call, 42.1 / 41.9 us with one
  // workgroup a CU); on the 70B shape LoPA gains too (eight tokens: gate kernel 76.1 -> 71.1 us), where
  // one workgroup a CU walks two segments one after the other.  fp32 rows, twice as long, gain from
  // it at any d_ff (d 3840, d_ff 14231, r 480, 5 / 8 / 16 tokens 73.7 / 83.0 / 90.7 -> 67.8 / 77.5 / 91.1
  // us), and so does a d_ff whose segments are one a workgroup (bf16 d 1024, d_ff 4000, 8 tokens 22.1 ->
  // 18.6; d 4608, d_ff 8000, r 512, 3 tokens 42.1 -> 37.0).
  const bool two = NT == 1 && (is_f32<W>() || sh.d_ff <= kSmallDff || sh.d_ff >= 48 * kSegGrid2);
  const int grid = two ? kSegGrid2 : kSegGrid;
  ws.nseg = segments_for(sh.d_ff, grid);
  const int g = ws.nseg < grid ? ws.nseg : grid;
  auto launch = [&](auto kernel) {
    return launch_gate_kernel(kernel, g, s, x, (const float*)ws.z, static_cast<const uint4*>(gate_w), Cg,
                            static_cast<const uint4*>(w_up), Cu, sh.T, sh.d, sh.d_ff, ws.nseg, t, ws.slots, ws.tc,
                            ws.meta, ws.seg_count, ws.seg_idx, ws.seg_act, ws.zf, y, ws.xs, token_tiles(ws), form,
                            (const float*)ws.gx, LOPA ? sh.sc.b : sh.sc.gate, sh.sc.up, sh.sc.down, alive_masks(ws), seg_quads(sh.d_ff, ws.nseg));
  };
  if constexpr (NT == 1)
    if (two) return launch(k_gate_up_mfma2<W, LOPA, DENSE, FORM>);
  if constexpr (NT > 1 || !is_f32<W>()) return launch(k_gate_up_mfma<W, LOPA, DENSE, NT, FORM>);
  return hipErrorInvalidValue;  // one tile of fp32 rows: `two` holds
}

template <class W, bool LOPA, bool DENSE, int FORM>
hipError_t gate_nt(const Shape& sh, const Form& f, const float* x, const void* gate_w, const void* w_up, float t,
                   Workspace& ws, float* y, hipStream_t s) {
  if (sh.T <= 16) return gate_mfma<W, LOPA, DENSE, 1, FORM>(sh, f, x, gate_w, w_up, t, ws, y, s);
  if (sh.T <= 32) return gate_mfma<W, LOPA, DENSE, 2, FORM>(sh, f, x, gate_w, w_up, t, ws, y, s);
  return gate_mfma<W, LOPA, DENSE, 4, FORM>(sh, f, x, gate_w, w_up, t, ws, y, s);
}

template <class W, bool LOPA, bool DENSE>
hipError_t gate_form(const Shape& sh, const Form& f, const float* x, const void* gate_w, const void* w_up, float t,
                     Workspace& ws, float* y, hipStream_t s) {
  if constexpr (LOPA)
    if (f.kind() == kFormLoPA) return gate_nt<W, LOPA, DENSE, kFormLoPA>(sh, f, x, gate_w, w_up, t, ws, y, s);
  return f.full() ? gate_nt<W, LOPA, DENSE, kFormAct>(sh, f, x, gate_w, w_up, t, ws, y, s)
                  : gate_nt<W, LOPA, DENSE, kFormDefault>(sh, f, x, gate_w, w_up, t, ws, y, s);
}

// Down grid: S column groups x R row chunks, about kDnWgTarget workgroups, at most
// kDnAtomicsMax fp32 atomics into y (fewer, longer row chunks measured faster than more
// parallel short ones), every chunk within the LDS slot and segment limits.
constexpr int kDnWgTarget = 512;
constexpr int64_t kDnAtomicsMax = 1 << 20;

template <class W, int NT>
hipError_t down_mfma(const Shape& sh, const void* w_down_t, const Workspace& ws, float* y, hipStream_t s) {
  const int C = sh.d / W::EPC;
  const int64_t wcols = DnCfg<NT, W>::WCOLS;
  const int64_t S = ((int64_t)sh.d + wcols - 1) / wcols;
  int64_t R = (kDnWgTarget + S - 1) / S;
  const int64_t amax = kDnAtomicsMax / ((int64_t)sh.T * sh.d);
  if (R > amax) R = amax;
  const int64_t rmin = (ws.nseg + kBlock - 1) / kBlock;
  if (R < rmin) R = rmin;
  // Chunks of at least 64 rows, about: with one 32-row segment a chunk the small layers' chunks doubled
  // in number and a workgroup had two groups of entries between its list and its atomics (int4 d 1024,
  // d_ff 2000, 16 tokens: down kernel 6.3 us at 64 rows, 8.6 at 32; calls 22.8 -> 20.3 us; int8 d 512,
  // d_ff 1500, 32 tokens 22.8 -> 21.5).
  const int64_t most = (sh.d_ff + kSegRowsB - 1) / kSegRowsB;
  if (R > most) R = most;
  if (R < 1) R = 1;
  const int64_t rows_per_seg = (sh.d_ff + ws.nseg - 1) / ws.nseg;
  while (R < ws.nseg && ((ws.nseg + R - 1) / R) * rows_per_seg > kDnSlots) ++R;
  if (((ws.nseg + R - 1) / R) * rows_per_seg > kDnSlots || S * R > INT32_MAX) return hipErrorInvalidValue;
  k_down_mfma<NT, W><<<(int)(S * R), kBlock, 0, s>>>(ws.seg_count, ws.seg_idx, ws.zf, ws.nseg,
                                                     seg_quads(sh.d_ff, ws.nseg), sh.d_ff, (int)R,
                                                     ws.tc, static_cast<const uint4*>(w_down_t), C, sh.d, sh.T, y,
                                                     reinterpret_cast<const uint2*>(alive_masks(ws)));
  return hipGetLastError();
}

// One call of the path for weights of format W (after the tokens are split, if they are).
template <class W>
hipError_t batched_format(const Shape& sh, Gate g, bool dense, const Form& form, const float* x, const void* lopa_a,
                          const void* gate_w, const void* w_up, const void* w_down_t, float t, Workspace& ws,
                          float* y, hipStream_t s) {
  const bool lopa = g == Gate::LoPA;
  hipError_t e = hipSuccess;
  if (lopa) {
    // pre-split tokens (more than 16): one token tile a workgroup
    e = sh.T <= 16 ? z_mfma<W, 1, false>(sh, form, x, lopa_a, ws, s) : z_mfma<W, 1, true>(sh, form, x, lopa_a, ws, s);
    if (e != hipSuccess) return e;
  }
  if (lopa)
    e = dense ? gate_form<W, true, true>(sh, form, x, gate_w, w_up, t, ws, y, s)
              : gate_form<W, true, false>(sh, form, x, gate_w, w_up, t, ws, y, s);
  else
    e = dense ? gate_form<W, false, true>(sh, form, x, gate_w, w_up, t, ws, y, s)
              : gate_form<W, false, false>(sh, form, x, gate_w, w_up, t, ws, y, s);
  if (e != hipSuccess) return e;
  if (sh.T <= 16) return down_mfma<W, 1>(sh, w_down_t, ws, y, s);
  if (sh.T <= 32) return down_mfma<W, 2>(sh, w_down_t, ws, y, s);
  return down_mfma<W, 4>(sh, w_down_t, ws, y, s);
}

}  // namespace

// The matrix-core path addresses every operand with 32-bit byte offsets below 2^31.
// bf16 weights, and int8 / int4 codes (converted to bf16 on their way into the operand
// tiles): rows of whole 16-byte chunks, so d (and LoPA's r) a multiple of 16 / 32.  fp32 weights
// likewise, d and r multiples of 4, at every batch size: against the vector-ALU kernels (which keep
// the other widths) at d 3840, d_ff 14231, r 480, 90%: 2 tokens 57.1 -> 44.5 us a call, 4 109.7 ->
// 55.4, 16 508 -> 90.5, 64 2024 -> 205; d 512, d_ff 2000, standard gating, 3 tokens 21.2 -> 17.6.
bool batched_ok(const Shape& sh, Gate g) {
  if (sh.wdt < 0 || sh.wdt > 3 || sh.T < 2 || sh.T > kTokChunk) return false;
  const int q = sh.wdt == 0 ? 4 : sh.wdt == 1 ? 8 : sh.wdt == 2 ? 16 : 32;  // elements a 16-byte chunk
  const int eb = sh.wdt == 0 ? 4 : 2;                                       // bytes an element, at most
  if (sh.d % q != 0) return false;
  const int64_t lim = int64_t(1) << 31;
  if (eb * (int64_t)sh.d_ff * sh.d >= lim || 4 * (int64_t)kTokChunk * sh.d >= lim) return false;
  if ((int64_t)segments_for(sh.d_ff, kSegGrid2) * 256 * kTokChunk >= lim) return false;
  if (g == Gate::LoPA && (sh.r % q != 0 || eb * (int64_t)sh.d_ff * sh.r >= lim || eb * (int64_t)sh.r * sh.d >= lim ||
                          4 * (int64_t)kTokChunk * sh.d_ff >= lim))  // G x, read through a buffer
    return false;
  return true;
}

// the most segments any gate kernel of this path uses (workspace sizing)
int batched_segments(int d_ff) {
  return d_ff > kSmallDff ? segments_for(d_ff, kSegGrid2) : (d_ff + kSegRowsB - 1) / kSegRowsB;
}

hipError_t launch_split_tokens(const Shape& sh, const float* x, const Workspace& ws, hipStream_t s) {
  return split_tokens<false>(sh, x, ws, s);
}
hipError_t launch_batched(const Shape& sh, Gate g, bool dense, const Form& form, const float* x,
                          const void* lopa_a, const void* gate_w, const void* w_up, const void* w_down_t, float t,
                          Workspace& ws, float* y, hipStream_t s) {
  if (wide64_ok(sh, g, ws))
    return launch_wide64(sh, g, dense, form, x, lopa_a, gate_w, w_up, w_down_t, t, ws, y, s);
  hipError_t e = hipSuccess;
  // more than one token tile: the kernels read the tokens pre-split
  if (sh.T > 16 &&
      (e = sh.wdt == 0 ? split_tokens<true>(sh, x, ws, s) : split_tokens<false>(sh, x, ws, s)) != hipSuccess)
    return e;
  if (sh.wdt == 0) return batched_format<WF32>(sh, g, dense, form, x, lopa_a, gate_w, w_up, w_down_t, t, ws, y, s);
  if (sh.wdt == 2) return batched_format<WI8>(sh, g, dense, form, x, lopa_a, gate_w, w_up, w_down_t, t, ws, y, s);
  if (sh.wdt == 3) return batched_format<WI4>(sh, g, dense, form, x, lopa_a, gate_w, w_up, w_down_t, t, ws, y, s);
  return batched_format<WBf16>(sh, g, dense, form, x, lopa_a, gate_w, w_up, w_down_t, t, ws, y, s);
}


}  // namespace ffn
