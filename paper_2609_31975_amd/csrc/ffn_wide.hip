// gfx950 kernels for calls of more than 64 tokens with bf16 or int8 / int4 weights, and of 33..64
// where d_ff suits them (wide64_ok).
//
// A pass of the 2..64-token kernels re-reads every token for each 64 weight rows and every
// weight row for each 64 tokens: at 200 tokens (8B shape, LoPA r = 512) four passes took 345 us,
// each reading the weights again and 2.3 times their bytes of token fragments.  Here all tokens
// that fit the workspace go in one pass, and every product is tiled on both sides:
//   k_wide_gate_up  a workgroup takes up to 128 rows of the gate and a block of up to 128 tokens:
//                   gate product, thresholds, the block's union of active rows, then the W_up
//                   product of the union rows against the same tokens; zval by quads of entries
//   k_wide_down     a workgroup takes 128 columns of W_down, a chunk of the segments and a block
//                   of tokens: Y[tokens][cols] += Z[tokens][entries] D[entries][cols]
// with k_split_tokens (the tokens as bf16 hi / lo fragment planes) and, for LoPA, k_wide_z (z = A x as
// partial copies) and k_split_z (the same planes for z) before them.
//
// Both products stage both operands in LDS: eight waves, two over the rows (columns), two over the
// tokens and two over the k steps of an iteration, a wave's tile being 64 x 64.  One iteration
// (64 k, 48 KB) is 256 products a wave pair against 96 KB of LDS reads; a wave of 64 x 64 needs
// three 16-byte LDS reads for eight products, which keeps the LDS (128 bytes a clock) near the
// matrix cores' time.  Loads run through registers into two LDS buffers, with one barrier an
// iteration; operands are read from LDS an iteration ahead of their products and between them (see
// wide_product).  At 200 tokens (8B shape) k_wide_gate_up takes 82 us: 49 us with the products alone,
// 65 with their LDS work and no loads, 91 with the weights requested four iterations ahead of their
// products instead of six, 88 with the LDS reads of an iteration in front of its products;
// k_wide_down 68, 75 and 81 us.
// The workgroups of the token blocks of one segment (or chunk) run on one XCD, so that its L2 serves
// the weights to all but the first.
#include "ffn_device.h"
#include "ffn_internal.h"
#include "ffn_mfma.h"

namespace ffn {
namespace {

constexpr int kWThreads = 512;
constexpr int kWTiles = 8;                  // token tiles (of 16) of a block
constexpr int kWRows = 128;                 // most rows of a segment
constexpr int kZRows = 64;                  // rows of A of a workgroup
constexpr int kWCols = 128;                 // columns of a down workgroup
constexpr int kWDnPad = 10;  // iterations past the last one that the down loop looks at
constexpr int kWDnList = kWDnRows + 3 * kWDnSegs + 64 * (kWDnPad + 1);  // packed entries, see k_wide_down
constexpr int kXcds = 8;
constexpr int kWCus = 256;

// Workgroup b of a grid of units x blocks: the blocks of a unit are kXcds apart, on one XCD.
__device__ __forceinline__ void unit_of(int b, int nb, int* unit, int* blk) {
  const int grp = b / (kXcds * nb), in = b - grp * kXcds * nb;
  *blk = in / kXcds;
  *unit = grp * kXcds + in % kXcds;
}

// The two k groups' sums of a wave pair (waves w and w ^ 4) meet: wave w ends with the sums of
// f[i][j] = acc[kg N / 2 + i][j], kg = w >> 2.  buf: 8 N / 2 M 64 f32x4.
template <int N, int M>
__device__ __forceinline__ void join_k(const f32x4_t (&acc)[N][M], f32x4_t* buf, f32x4_t (&f)[N / 2][M]) {
  const int lane = lane_id(), wave = uniform(threadIdx.x / kWave);
  const bool hi = wave >= 4;
#pragma unroll
  for (int i = 0; i < N / 2; ++i)
#pragma unroll
    for (int j = 0; j < M; ++j) buf[((wave * (N / 2) + i) * M + j) * kWave + lane] = hi ? acc[i][j] : acc[N / 2 + i][j];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N / 2; ++i)
#pragma unroll
    for (int j = 0; j < M; ++j)
      f[i][j] = (hi ? acc[N / 2 + i][j] : acc[i][j]) + buf[(((wave ^ 4) * (N / 2) + i) * M + j) * kWave + lane];
}

// Waits for the wave's loads and stores (vmcnt 0, the other counters as they are).
__device__ __forceinline__ void wait_vmem() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// ------------------------------------------------------------------ rows x tokens
// LDS of one product: the rows' chunks in operand order ([k step][row tile][lane group g][row],
// the row index xor-ed with the chunk's place in the iteration so that a row's eight chunks, which
// neighbouring lanes write, fall on distinct banks), and the tokens' hi and lo planes as they are
// in memory.
template <int NT>
struct WideStage {
  uint4 w[2][2][NT][4][16];
  uint4 x[2][2][2][NT][kWave];  // [buffer][plane][k step][token tile][lane]
};

// acc[i][j] += rows (row tile wr + 2 i) . tokens (token tile wt + 2 j) for a wave (kg, wr, wt) over
// its half of the k steps.  roff[i]: the loaded chunk at which row (threadIdx.x / LPR + RPP i)
// starts, or -1.  C: tile chunks (8 elements) a row; the tokens' planes start at xb, part_bytes
// apart, tile nt0 the block's first of ntb, ntt a k step.  Iterations it0 .. it1 - 1 (two k steps
// each) are summed.
template <class W, int RT>
struct WideRows {
  static constexpr int R8 = W::EPC / 8;            // tile chunks per loaded chunk
  static constexpr int LPR = 8 / R8;               // loaded chunks of a row an iteration
  static constexpr int RPP = kWThreads / LPR;      // rows a load of all threads covers
  static constexpr int NL = (32 * RT + RPP - 1) / RPP;
};

template <class W, int RT, int NT>
__device__ __forceinline__ void wide_product(WideStage<NT>& st, const Buf& wb, int C, const int* roff, const Buf& xb,
                                             uint32_t part_bytes, int ntt, int nt0, int ntb, int it0, int it1,
                                             f32x4_t (&acc)[RT][NT / 2]) {
  constexpr int NJ = NT / 2;  // token tiles of a wave
  static_assert(2 * RT <= NT, "the row tiles' space");
  using S = WideRows<W, RT>;
  const int tid = threadIdx.x, lane = lane_id(), wave = uniform(tid / kWave);
  const int nks = (C + 3) / 4, nit = it1 - it0;
  const int kg = wave >> 2, wr = (wave >> 1) & 1, wt = wave & 1, m = lane & 15, g = lane >> 4;
  struct RegsW {
    uint4 w[S::NL];
  };
  // a wave loads token tile wave % NT: with eight tiles both k steps of an iteration, with four
  // k step wave / 4
  constexpr int NK = NT / 4;
  struct RegsX {
    uint4 x[2][NK];  // [plane][k step]
  };
  const int lt = wave % NT, lk = wave / NT;
  const bool tile_ok = lt < ntb;
  auto load_w = [&](RegsW& r, int t) {
    const int it = it0 + t, lc = tid % S::LPR, ch = it * S::LPR + lc;  // the lane's loaded chunk of the row
    const bool cv = it < it1 && ch < C / S::R8;
#pragma unroll
    for (int i = 0; i < S::NL; ++i) r.w[i] = ldb(wb, cv && roff[i] >= 0 ? 16u * (uint32_t)(roff[i] + ch) : kOOB);
  };
  auto load_x = [&](RegsX& r, int t) {
    const int it = it0 + t;
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      const int ks = 2 * it + lk + k;
      const uint32_t off = tile_ok && it < it1 && ks < nks
                               ? 16u * ((uint32_t)(ks * ntt + nt0 + lt) * kWave + (uint32_t)lane)
                               : kOOB;
      r.x[0][k] = ldb(xb, off);
      r.x[1][k] = ldb(xb, off + part_bytes);
    }
  };
  auto put_w = [&](const RegsW& r, int b) {
    const int lc = tid % S::LPR;
#pragma unroll
    for (int i = 0; i < S::NL; ++i) {
      const int row = tid / S::LPR + S::RPP * i;
      if (row < 32 * RT) {
        uint4 t[S::R8];
        put_bf16_chunks<W>(t, r.w[i]);
#pragma unroll
        for (int c = 0; c < S::R8; ++c) {
          const int at = lc * S::R8 + c;  // tile chunk of the iteration
          st.w[b][at >> 2][row >> 4][at & 3][(row & 15) ^ (2 * (at & 3) + 8 * (at >> 2))] = t[c];
        }
      }
    }
  };
  auto put_x = [&](const RegsX& r, int b, int p) {
#pragma unroll
    for (int k = 0; k < NK; ++k) st.x[b][p][lk + k][lt][lane] = r.x[p][k];
  };
  // operands of the wave's k step of the tile in buffer b
  auto read_a = [&](int b, int i) { return bf8(st.w[b][kg][wr + 2 * i][g][m ^ (2 * g + 8 * kg)]); };
  auto read_x = [&](int b, int p, int j) { return bf8(st.x[b][p][kg][wt + 2 * j][lane]); };
  // Iteration it multiplies tile it, whose operands are in registers already, while it reads those
  // of tile it + 1 from the other buffer, writes tile it + 2 over tile it's and requests the tokens
  // of tile it + 4 (from L2) and the weights of tile it + 6 (from HBM).  The barrier that ends an
  // iteration also ends its LDS reads, so two buffers do.  The LDS work is spread between the
  // products of the four token tiles, and a token tile's operands are read into the registers that
  // its products have just released.  Four iterations always run (those past the end load nothing
  // and add zeros), so that no load sits on a conditional path.
  RegsW w0, w1, w2, w3;
  RegsX x0, x1;
  bf16x8_t a0[RT], a1[RT], xh[NJ], xl[NJ];
  load_w(w0, 0), load_x(x0, 0);
  load_w(w1, 1), load_x(x1, 1);
  load_w(w2, 2), load_w(w3, 3);
  put_w(w0, 0), put_x(x0, 0, 0), put_x(x0, 0, 1);
  load_w(w0, 4), load_x(x0, 2);
  put_w(w1, 1), put_x(x1, 1, 0), put_x(x1, 1, 1);
  load_w(w1, 5), load_x(x1, 3);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < RT; ++i) a0[i] = read_a(0, i);
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    xh[j] = read_x(0, 0, j);
    xl[j] = read_x(0, 1, j);
  }
  __syncthreads();
  auto step = [&](const bf16x8_t (&a)[RT], bf16x8_t (&an)[RT], RegsW& w, RegsX& x, int b, int t) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
#pragma unroll
      for (int i = j; i < RT; i += NJ) an[i] = read_a(b ^ 1, i);
#pragma unroll
      for (int i = 0; i < RT; ++i) acc[i][j] = mfma16(a[i], xh[j], acc[i][j]);
#pragma unroll
      for (int i = 0; i < RT; ++i) acc[i][j] = mfma16(a[i], xl[j], acc[i][j]);
      xh[j] = read_x(b ^ 1, 0, j);
      xl[j] = read_x(b ^ 1, 1, j);
      if (j == 0) {
        put_w(w, b);
        load_w(w, t + 6);
      }
      if (j == 1) put_x(x, b, 0);
      if (j == NJ / 2) {
        put_x(x, b, 1);
        load_x(x, t + 4);
      }
      issue_barrier();
    }
    __syncthreads();
  };
  for (int t = 0;; t += 4) {
    step(a0, a1, w2, x0, 0, t);
    step(a1, a0, w3, x1, 1, t + 1);
    step(a0, a1, w0, x0, 0, t + 2);
    step(a1, a0, w1, x1, 1, t + 3);
    if (t + 4 >= nit) break;
  }
}

struct WideArgs {
  const uint4 *gate_w, *w_up;
  const uint4 *xs, *zs;  // token planes of x and (LoPA) z
  int Cg, Cu;            // tile chunks of a gate row, of a W_up row
  int T, d, d_ff, nseg, qps, ntt, nb;  // qps: quads a segment has room for
  int lopa, dense;
  float t;
  Form form;
  const float* gx;                    // G x [T][d_ff] (LoPA with G)
  const float *s_g, *s_up, *s_down;   // row scales (int8 / int4)
  int32_t* seg_count;                 // [nb][nseg]
  int32_t* seg_idx;                   // [nb][d_ff]
  uint4* zf;   // zval by quads: block b's quads at uint4 16 nt0(b) nseg qps, of segment seg from quad
               // seg qps, [quad][token tile of the block][16]
  float* seg_act;  // calls of at most kTokChunk tokens: [T][d_ff], act of entry e of segment w at slot
                   // start(w) + e (the inspection hooks' layout), else null
  int32_t* meta;   // likewise: meta[0] = nseg
  float* y;
};
__host__ __device__ __forceinline__ int wide_iterations(int C) { return (C + 7) / 8; }
__device__ __forceinline__ uint32_t plane_bytes(int C, int ntt) {
  return 16u * (uint32_t)((C + 3) / 4) * (uint32_t)ntt * (uint32_t)kWave;
}

// Gate, union and W_up of one segment (up to 32 RT rows) for one block of tokens.  The activation
// values wait in the segment's own part of the zval buffer ([row][token of the block], the same
// size) for the W_up sums: they are read back before the first zval is written there.
// NT: token tiles of a block, at most (and row tiles of a segment).
template <class W, int NT>
__global__ __launch_bounds__(kWThreads) void k_wide_gate_up(WideArgs a) {
  constexpr bool Q = is_quant<W>();
  constexpr int NJ = NT / 2;
  __shared__ union {
    WideStage<NT> st;
    f32x4_t join[8 * (NT / 4) * NJ * kWave];
  } s;
  __shared__ uint32_t s_mask[kWTiles];
  __shared__ int s_list[kWRows];

  const int tid = threadIdx.x, lane = lane_id(), wave = uniform(tid / kWave);
  const int kg = wave >> 2, wr = (wave >> 1) & 1, wt = wave & 1, m = lane & 15, g = lane >> 4;
  for (int j = blockIdx.x * kWThreads + tid; j < a.T * a.d; j += gridDim.x * kWThreads) a.y[j] = 0.f;
  int seg, blk;
  unit_of(blockIdx.x, a.nb, &seg, &blk);
  if (seg >= a.nseg) return;  // workgroup-uniform
  const Split tiles(a.ntt, a.nb), segs(a.d_ff, a.nseg);
  const int nt0 = tiles.start(blk), ntb = tiles.start(blk + 1) - nt0;  // <= kWTiles
  const int row0 = segs.start(seg), nrows = segs.start(seg + 1) - row0;  // <= kWRows
  uint4* const zq = a.zf + ((size_t)nt0 * a.nseg + (size_t)seg * ntb) * a.qps * 16;
  float* const act = reinterpret_cast<float*>(zq);  // [nrows][16 ntb]
  if (a.meta && blockIdx.x == 0 && tid == 0) a.meta[0] = a.nseg;
  if (tid < kWTiles) s_mask[tid] = 0u;

  // the rows of a product: rows list[k], k < n, of a matrix of C chunks a row
  auto product = [&](const uint4* mat, int C, const uint4* planes, int n, auto row_of, auto& acc) {
    constexpr int RT = sizeof(acc) / sizeof(acc[0]);
    using S = WideRows<W, RT>;
    const uint32_t part = plane_bytes(C, a.ntt);
    const int Cl = C / S::R8;
    int roff[S::NL];
#pragma unroll
    for (int i = 0; i < S::NL; ++i) {
      const int k = tid / S::LPR + S::RPP * i;
      roff[i] = k < n ? row_of(k) * Cl : -1;
    }
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    wide_product<W, RT, NT>(s.st, make_buf(mat, 16u * (uint32_t)a.d_ff * (uint32_t)Cl), C, roff, make_buf(planes, 2 * part),
                        part, a.ntt, nt0, ntb, 0, wide_iterations(C), acc);
  };

  // thresholds of the wave's half of the row tiles: activation values out, the rows that any
  // token of the block activates into s_mask
  auto gate = [&](auto& acc) {
    constexpr int RT = sizeof(acc) / sizeof(acc[0]);
    product(a.gate_w, a.Cg, a.lopa ? a.zs : a.xs, nrows, [&](int k) { return row0 + k; }, acc);
    f32x4_t h[RT / 2][NJ];
    join_k(acc, s.join, h);
    const Buf qb = make_buf(a.s_g, 4u * (uint32_t)a.d_ff);
    const bool has_g = a.lopa && a.form.g_idx;
#pragma unroll
    for (int i = 0; i < RT / 2; ++i) {
      const int rt = wr + 2 * (kg * (RT / 2) + i);
      uint32_t mask = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int rl = 16 * rt + 4 * g + e;
        const bool rv = rl < nrows;
        const float sc = Q ? __int_as_float(ldb32(qb, rv ? 4u * (uint32_t)(row0 + rl) : kOOB)) : 1.f;
        bool any = false;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int nt = wt + 2 * j, tok = 16 * (nt0 + nt) + m;
          const bool tv = nt < ntb && tok < a.T;
          float hv = h[i][j][e];
          if constexpr (Q) hv *= sc;
          if (has_g && rv && tv) hv += a.gx[(size_t)tok * a.d_ff + row0 + rl];
          const bool on = tv && hv > a.t;  // NaN compares false: inactive
          any |= on;
          if (rv && nt < ntb) act[(size_t)rl * 16 * ntb + 16 * nt + m] = on ? gate_value(a.form.act, hv - a.t) : 0.f;
        }
        const uint64_t b = __ballot(any && rv);
#pragma unroll
        for (int gg = 0; gg < 4; ++gg)
          if ((b >> (16 * gg)) & 0xffffull) mask |= 1u << (4 * gg + e);
      }
      if (lane == 0 && mask) atomicOr(&s_mask[rt], mask);
    }
  };
  __syncthreads();
  if constexpr (NT == kWTiles) {
    if (nrows > kWRows / 2) {
      f32x4_t acc[4][NJ];
      gate(acc);
    } else {
      f32x4_t acc[2][NJ];
      gate(acc);
    }
  } else {
    f32x4_t acc[2][NJ];
    gate(acc);
  }
  wait_vmem();  // the activation values are out
  __syncthreads();

  // the union, ascending
  int cnt;
  {
    uint64_t mk[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int n = min(max(nrows - 64 * h, 0), 64);
      const uint64_t valid = n == 64 ? ~0ull : (1ull << n) - 1;
      const uint64_t v = (uint64_t)s_mask[4 * h] | ((uint64_t)s_mask[4 * h + 1] << 16) |
                         ((uint64_t)s_mask[4 * h + 2] << 32) | ((uint64_t)s_mask[4 * h + 3] << 48);
      mk[h] = (a.dense ? ~0ull : v) & valid;
    }
    const int c0 = __popcll(mk[0]);
    cnt = uniform(c0 + __popcll(mk[1]));
    if (tid < kWRows && ((tid < 64 ? mk[0] >> tid : mk[1] >> (tid - 64)) & 1ull)) {
      const int rank = tid < 64 ? __popcll(mk[0] & ((1ull << tid) - 1))
                                : c0 + __popcll(mk[1] & ((1ull << (tid - 64)) - 1));
      s_list[rank] = tid;
      a.seg_idx[(size_t)blk * a.d_ff + row0 + rank] = row0 + tid;
    }
    if (tid == 0) a.seg_count[blk * a.nseg + seg] = cnt;
  }
  __syncthreads();
  if (a.seg_act)
    for (int o = tid; o < cnt * 16 * ntb; o += kWThreads) {  // lanes along the entries
      const int tok = o / cnt, e = o - tok * cnt;
      if (tok < a.T) a.seg_act[(size_t)tok * a.d_ff + row0 + e] = act[(size_t)s_list[e] * 16 * ntb + tok];
    }
  if (cnt == 0) return;  // workgroup-uniform

  // W_up dots of the union rows, then zval = activation value times the dot
  auto up = [&](auto& acc) {
    constexpr int RT = sizeof(acc) / sizeof(acc[0]);
    product(a.w_up, a.Cu, a.xs, cnt, [&](int k) { return row0 + s_list[k]; }, acc);
    float av[RT / 2][NJ][4], su[RT / 2][4], sd[RT / 2][4];
    const Buf ubs = make_buf(a.s_up, 4u * (uint32_t)a.d_ff), dbs = make_buf(a.s_down, 4u * (uint32_t)a.d_ff);
#pragma unroll
    for (int i = 0; i < RT / 2; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int en = 16 * (wr + 2 * (kg * (RT / 2) + i)) + 4 * g + e;
        const int rl = en < cnt ? s_list[en] : 0;
        if constexpr (Q) {
          const uint32_t off = en < cnt ? 4u * (uint32_t)(row0 + rl) : kOOB;
          su[i][e] = __int_as_float(ldb32(ubs, off));
          sd[i][e] = __int_as_float(ldb32(dbs, off));
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int nt = wt + 2 * j;
          av[i][j][e] = en < cnt && nt < ntb ? act[(size_t)rl * 16 * ntb + 16 * nt + m] : 0.f;
        }
      }
    f32x4_t v[RT / 2][NJ];
    join_k(acc, s.join, v);
    wait_vmem();
    __syncthreads();  // every activation value has been read
#pragma unroll
    for (int i = 0; i < RT / 2; ++i) {
      const int q = 4 * (wr + 2 * (kg * (RT / 2) + i)) + g;
      if (4 * q >= cnt) continue;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int nt = wt + 2 * j;
        if (nt >= ntb) continue;
        uint32_t hw[2] = {0u, 0u}, lw[2] = {0u, 0u};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float vu = Q ? v[i][j][e] * su[i][e] : v[i][j][e];
          float zz = 4 * q + e < cnt ? av[i][j][e] * up_value(a.form.silu_up, vu) : 0.f;
          if constexpr (Q) zz *= sd[i][e];
          const __bf16 hb = (__bf16)zz;
          const __bf16 lb = (__bf16)(zz - (float)hb);
          hw[e >> 1] |= (uint32_t)__builtin_bit_cast(uint16_t, hb) << (16 * (e & 1));
          lw[e >> 1] |= (uint32_t)__builtin_bit_cast(uint16_t, lb) << (16 * (e & 1));
        }
        zq[((size_t)q * ntb + nt) * 16 + m] = make_uint4(hw[0], hw[1], lw[0], lw[1]);
      }
    }
  };
  if constexpr (NT == kWTiles) {
    if (cnt > kWRows / 2) {
      f32x4_t acc[4][NJ];
      up(acc);
    } else {
      f32x4_t acc[2][NJ];
      up(acc);
    }
  } else {
    f32x4_t acc[2][NJ];
    up(acc);
  }
}

// ------------------------------------------------------------------ down projection
// The chunk's union entries are packed by quads as in k_down_mfma, 64 entries an iteration: half of
// them for each k group.  The rows go to LDS as they are (two pad chunks a row: the transposing
// reads' eight rows on distinct banks), the zval quads beside them.  The k groups' sums meet in LDS,
// then go to y with one fp32 atomic per token and column.
template <class W, int NT>
__global__ __launch_bounds__(kWThreads) void k_wide_down(const int32_t* __restrict__ seg_count,
                                                         const int32_t* __restrict__ seg_idx,
                                                         const uint4* __restrict__ zf, int nseg, int qps, int d_ff,
                                                         int R, int ntt, int nb, const uint4* __restrict__ w_down_t,
                                                         int C, int d, int T, float* __restrict__ y) {
  constexpr int R8 = W::EPC / 8, LPR = kWCols / W::EPC, RPP = kWThreads / LPR, NL = (64 + RPP - 1) / RPP;
  constexpr int PITCH = kWCols / 8 + 2, NJ = NT / 2;
  __shared__ union {
    struct {
      uint4 w[2][64 * PITCH];
      uint4 z[2][2][2][NT][kWave];  // [buffer][k group][hi, lo][token tile][lane]
    } st;
    f32x4_t join[8 * (NJ / 2) * 4 * kWave];
  } s;
  __shared__ int s_row[kWDnList], s_zq[kWDnList / 4];
  __shared__ int s_wquads[kWThreads / kWave], s_cnt[kWDnSegs], s_quad[kWDnSegs];

  const int S = (d + kWCols - 1) / kWCols;
  int unit, blk;
  unit_of(blockIdx.x, nb, &unit, &blk);
  if (unit >= S * R) return;  // workgroup-uniform
  const int chunk = unit / S, cgrp = unit % S;
  const Split chunks(nseg, R), segs(d_ff, nseg), tiles(ntt, nb);
  const int nt0 = tiles.start(blk), ntb = tiles.start(blk + 1) - nt0;
  const int seg_lo = chunks.start(chunk), seg_hi = chunks.start(chunk + 1);
  const int nsc = seg_hi - seg_lo;  // <= kWDnSegs, guaranteed by the host
  const int tid = threadIdx.x, lane = lane_id(), wave = uniform(tid / kWave);
  const int kg = wave >> 2, wc = (wave >> 1) & 1, wt = wave & 1, m = lane & 15, g = lane >> 4;
  const Buf db = make_buf(w_down_t, 16u * (uint32_t)d_ff * (uint32_t)C);
  const Buf zb = make_buf(zf + (size_t)nt0 * nseg * qps * 16, 256u * (uint32_t)nseg * (uint32_t)qps * (uint32_t)ntb);

  // the packed list (rows at most kWDnRows, guaranteed by the host)
  const int c = tid < nsc ? seg_count[blk * nseg + seg_lo + tid] : 0;
  const int quads = wave_inclusive_scan((c + 3) >> 2);
  if (lane == kWave - 1) s_wquads[wave] = quads;
  __syncthreads();
  int qbase = 0, nquad = 0;
#pragma unroll
  for (int w = 0; w < kWThreads / kWave; ++w) {
    const int v = s_wquads[w];
    qbase += w < wave ? v : 0;
    nquad += v;
  }
  nquad = uniform(nquad);
  const int nit = (nquad + 15) / 16;
  if (tid < nsc) {
    s_cnt[tid] = c;
    s_quad[tid] = qbase + quads - ((c + 3) >> 2);
  }
  for (int o = 4 * nquad + tid; o < 64 * (nit + kWDnPad); o += kWThreads) {
    s_row[o] = -1;
    if ((o & 3) == 0) s_zq[o >> 2] = -1;
  }
  __syncthreads();
  {
    // half-segments of 64 rows, a wave each, SU in flight
    constexpr int SU = 8, WV = kWThreads / kWave;
    const Buf ib = make_buf(seg_idx + (size_t)blk * d_ff, 4u * (uint32_t)d_ff);
    for (int u0 = wave; u0 < 2 * nsc; u0 += WV * SU) {
      int v[SU];
#pragma unroll
      for (int u = 0; u < SU; ++u) {
        const int hs = u0 + u * WV, sg = hs >> 1, e = 64 * (hs & 1) + lane;
        const bool ok = hs < 2 * nsc && e < s_cnt[hs < 2 * nsc ? sg : 0];
        v[u] = ldb32(ib, ok ? 4u * (uint32_t)(segs.start(seg_lo + sg) + e) : kOOB);
      }
#pragma unroll
      for (int u = 0; u < SU; ++u) {
        const int hs = u0 + u * WV, sg = hs >> 1, e = 64 * (hs & 1) + lane;
        if (hs < 2 * nsc && e < ((s_cnt[sg] + 3) & ~3)) {
          const int o = 4 * s_quad[sg] + e;
          s_row[o] = e < s_cnt[sg] ? v[u] : -1;
          if ((e & 3) == 0) s_zq[o >> 2] = (seg_lo + sg) * qps + (e >> 2);
        }
      }
    }
  }
  __syncthreads();

  f32x4_t acc[NJ][4];  // [token tile wt + 2 j][16 columns 64 wc + 16 c]
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) acc[j][cc] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  struct RegsW {
    uint4 w[NL];
  };
  // a wave loads the zval of token tile wave % NT: with eight tiles both k groups of an iteration,
  // with four k group wave / 4
  constexpr int NK = NT / 4;
  const int lt = wave % NT, lk = wave / NT;
  struct RegsZ {
    u32x4_t z[2 * NK];
  };
  struct Place {  // list entries of a load
    int row[NL], zq[2 * NK];
  };
  const int lc = tid % LPR, ch = cgrp * LPR + lc;
  const bool tile_ok = lt < ntb;
  auto rows = [&](Place& a, int it) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int e = tid / LPR + RPP * i;
      a.row[i] = s_row[64 * it + (e < 64 ? e : 0)];
    }
  };
  auto zqs = [&](Place& a, int it) {
#pragma unroll
    for (int j = 0; j < 2 * NK; ++j) a.zq[j] = s_zq[16 * it + 8 * lk + 4 * j + g];
  };
  auto load_w = [&](RegsW& r, const Place& a) {
#pragma unroll
    for (int i = 0; i < NL; ++i)
      r.w[i] = ldb(db, tid / LPR + RPP * i < 64 && a.row[i] >= 0 && ch < C ? 16u * (uint32_t)(a.row[i] * C + ch) : kOOB);
  };
  auto load_z = [&](RegsZ& r, const Place& a) {
#pragma unroll
    for (int j = 0; j < 2 * NK; ++j)
      r.z[j] = __builtin_bit_cast(
          u32x4_t, ldb(zb, tile_ok && a.zq[j] >= 0
                               ? 16u * (((uint32_t)a.zq[j] * (uint32_t)ntb + (uint32_t)lt) * 16u + (uint32_t)m)
                               : kOOB));
  };
  auto put_w = [&](const RegsW& r, int b) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int e = tid / LPR + RPP * i;
      if (e < 64) put_bf16_chunks<W>(&s.st.w[b][e * PITCH + lc * R8], r.w[i]);
    }
  };
  // the quads 4 g and 16 + 4 g of the 32 entries of k group lk + k as one hi and one lo operand
  auto put_z = [&](const RegsZ& r, int b, auto kc) {
    constexpr int k = decltype(kc)::value;
    if constexpr (k < NK) {
      s.st.z[b][lk + k][0][lt][lane] =
          __builtin_bit_cast(uint4, __builtin_shufflevector(r.z[2 * k], r.z[2 * k + 1], 0, 1, 4, 5));
      s.st.z[b][lk + k][1][lt][lane] =
          __builtin_bit_cast(uint4, __builtin_shufflevector(r.z[2 * k], r.z[2 * k + 1], 2, 3, 6, 7));
    }
  };
  // The transposing reads as in k_down_mfma: 32 entries of the k group, 16 of the wave's 64 columns.
  auto read_d = [&](int b, int cc) {
    constexpr int ROWB = 16 * PITCH;
    const char* src = reinterpret_cast<const char*>(&s.st.w[b][32 * kg * PITCH]) +
                      (4 * (lane >> 4) + ((lane >> 2) & 3)) * ROWB + 8 * (lane & 3) + 128 * wc + 32 * cc;
    const uint2 lo = lds_read_tr16(src), hi = lds_read_tr16(src + 16 * ROWB);
    return bf8(make_uint4(lo.x, lo.y, hi.x, hi.y));
  };
  auto read_z = [&](int b, int p, int j) { return bf8(s.st.z[b][kg][p][wt + 2 * j][lane]); };
  if (nit > 0) {  // the loop of wide_product, the list entries read one iteration ahead of their loads
    RegsW w0, w1, w2, w3;
    RegsZ z0, z1;
    bf16x8_t d0[4], d1[4], zh[NJ], zl[NJ];
    Place a;
    rows(a, 0), zqs(a, 0);
    load_w(w0, a), load_z(z0, a);
    rows(a, 1), zqs(a, 1);
    load_w(w1, a), load_z(z1, a);
    rows(a, 2);
    load_w(w2, a);
    rows(a, 3);
    load_w(w3, a);
    rows(a, 4), zqs(a, 2);
    put_w(w0, 0), put_z(z0, 0, Int<0>{}), put_z(z0, 0, Int<1>{});
    load_w(w0, a), load_z(z0, a);
    rows(a, 5), zqs(a, 3);
    put_w(w1, 1), put_z(z1, 1, Int<0>{}), put_z(z1, 1, Int<1>{});
    load_w(w1, a), load_z(z1, a);
    rows(a, 6), zqs(a, 4);
    __syncthreads();
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) d0[cc] = read_d(0, cc);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      zh[j] = read_z(0, 0, j);
      zl[j] = read_z(0, 1, j);
    }
    __syncthreads();
    auto step = [&](const bf16x8_t (&dc)[4], bf16x8_t (&dn)[4], RegsW& w, RegsZ& z, int b, int t) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
#pragma unroll
        for (int cc = j; cc < 4; cc += NJ) dn[cc] = read_d(b ^ 1, cc);
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) acc[j][cc] = mfma16(zh[j], dc[cc], acc[j][cc]);
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) acc[j][cc] = mfma16(zl[j], dc[cc], acc[j][cc]);
        zh[j] = read_z(b ^ 1, 0, j);
        zl[j] = read_z(b ^ 1, 1, j);
        if (j == 0) {
          put_w(w, b);
          load_w(w, a);
        }
        if (j == 1) put_z(z, b, Int<0>{});
        if (j == NJ / 2) {
          put_z(z, b, Int<1>{});
          load_z(z, a);
        }
        if (j == NJ - 1) {
          rows(a, t + 7);
          zqs(a, t + 5);
        }
        issue_barrier();
      }
      __syncthreads();
    };
    for (int t = 0;; t += 4) {
      step(d0, d1, w2, z0, 0, t);
      step(d1, d0, w3, z1, 1, t + 1);
      step(d0, d1, w0, z0, 0, t + 2);
      step(d1, d0, w1, z1, 1, t + 3);
      if (t + 4 >= nit) break;
    }
  }
  f32x4_t f[NJ / 2][4];
  join_k(acc, s.join, f);
#pragma unroll
  for (int j = 0; j < NJ / 2; ++j) {
    const int nt = wt + 2 * (NJ / 2 * kg + j);
    if (nt >= ntb) continue;
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) {
      const int col = cgrp * kWCols + 64 * wc + 16 * cc + m;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int tok = 16 * (nt0 + nt) + 4 * g + e;
        if (tok < T && col < d) unsafeAtomicAdd(y + (size_t)tok * d + col, f[j][cc][e]);
      }
    }
  }
}

// ------------------------------------------------------------------ LoPA z = A x
// Workgroup (rows 64 u .. of A, block of tokens, part p of the iterations): partial copy p of z,
// zp[p][T][r].  The parts spread the few rows of A over the chip (r = 512, 200 tokens: 16 units, 16
// parts of four iterations each: 9.4 us; 19.6 on the batch kernels' grid of 16-row
// tiles, each with workgroups for every token tile); k_split_z adds them.
template <class W, int NT>
__global__ __launch_bounds__(kWThreads) void k_wide_z(const uint4* __restrict__ A, const uint4* __restrict__ xs, int C,
                                                      int T, int r, int ntt, int nb, int P, float* __restrict__ zp,
                                                      const float* __restrict__ s_a, GWork gw) {
  if (g_precompute(gw)) return;
  constexpr int NJ = NT / 2;
  __shared__ union {
    WideStage<NT> st;
    f32x4_t join[8 * NJ * kWave];
  } s;
  const int tid = threadIdx.x, lane = lane_id(), wave = uniform(tid / kWave);
  const int kg = wave >> 2, wr = (wave >> 1) & 1, wt = wave & 1, m = lane & 15, g = lane >> 4;
  const int p = blockIdx.x % P, ub = blockIdx.x / P, blk = ub % nb, row0 = ub / nb * kZRows;
  const Split tiles(ntt, nb), its(wide_iterations(C), P);
  const int nt0 = tiles.start(blk), ntb = tiles.start(blk + 1) - nt0;
  const int n = min(kZRows, r - row0);
  const uint32_t part = plane_bytes(C, ntt);
  constexpr int RT = kZRows / 32;
  using S = WideRows<W, RT>;
  const int Cl = C / S::R8;
  int roff[S::NL];
#pragma unroll
  for (int i = 0; i < S::NL; ++i) {
    const int k = tid / S::LPR + S::RPP * i;
    roff[i] = k < n ? (row0 + k) * Cl : -1;
  }
  f32x4_t acc[RT][NJ];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  wide_product<W, RT, NT>(s.st, make_buf(A, 16u * (uint32_t)r * (uint32_t)Cl), C, roff, make_buf(xs, 2 * part), part, ntt,
                      nt0, ntb, its.start(p), its.start(p + 1), acc);
  f32x4_t f[RT / 2][NJ];
  join_k(acc, s.join, f);
#pragma unroll
  for (int i = 0; i < RT / 2; ++i) {
    const int kl = 16 * (wr + 2 * (kg * (RT / 2) + i)) + 4 * g, k = row0 + kl;
    if (kl >= n) continue;  // r is a multiple of 8: four rows or none
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int tok = 16 * (nt0 + wt + 2 * j) + m;
      f32x4_t v = f[i][j];
      if constexpr (is_quant<W>()) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] *= s_a[k + e];
      }
      if (wt + 2 * j < ntb && tok < T) *reinterpret_cast<f32x4_t*>(zp + ((size_t)p * T + tok) * r + k) = v;
    }
  }
}

// z as fragment planes like the tokens' (k_split_tokens), from its `copies` partial copies
// [copies][T][r], added in order.
__global__ __launch_bounds__(kBlock) void k_split_z(const float* __restrict__ zp, int copies, int r, int T, int nks,
                                                    int ntt, uint4* __restrict__ zs) {
  const int n = nks * ntt * kWave, i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const int lane = i % kWave, fr = i / kWave, nt = fr % ntt, ks = fr / ntt;
  const int tok = 16 * nt + (lane & 15), k = 32 * ks + 8 * (lane >> 4);
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (tok < T && k < r) {  // r is a multiple of 8
    const float* p = zp + (size_t)tok * r + k;
#pragma unroll 4
    for (int c = 0; c < copies; ++c, p += (size_t)T * r) {
      const float4 a = reinterpret_cast<const float4*>(p)[0], b = reinterpret_cast<const float4*>(p)[1];
      v[0] += a.x, v[1] += a.y, v[2] += a.z, v[3] += a.w, v[4] += b.x, v[5] += b.y, v[6] += b.z, v[7] += b.w;
    }
  }
  bf16x8_t hi, lo;
  split8(v, hi, lo);
  zs[i] = __builtin_bit_cast(uint4, hi);
  zs[n + i] = __builtin_bit_cast(uint4, lo);
}

// ------------------------------------------------------------------ host side
struct WideLayout {
  int nseg, qps, ntt, nb;
  int zparts;    // partial copies of z there is room for
  Workspace ws;  // tc, z, gx, xs of the shared kernels
  int32_t *seg_count, *seg_idx, *meta;
  uint4 *zs, *zf;
  float* seg_act;
};

// The pass's regions in the workspace, behind the z slots (which stay as they are); returns the bytes.
size_t wide_layout(int T, int d, int d_ff, int r, bool has_g, void* base, size_t head, WideLayout* out) {
  WideLayout w{};
  w.ntt = (T + 15) / 16;
  w.nb = (w.ntt + kWTiles - 1) / kWTiles;
  // Rows a segment: 64 where the workgroups of those (one a CU) take one round, else 128, whose product
  // reads the tokens half as often.  bf16, standard gating, 128 -> 64 rows: d 4096, d_ff 11000, 100 tokens
  // (172 workgroups of 64) 156 -> 135 us.  64 -> 128: 200 tokens (344) 225 -> 170, d 8192, d_ff 21000, 65
  // tokens (329) 414 -> 345.
  const int big = (d_ff + kWRows - 1) / kWRows;
  const int rows = 2 * (int64_t)big * w.nb <= kWCus ? kWRows / 2 : kWRows;
  w.nseg = (d_ff + rows - 1) / rows;
  w.qps = ((d_ff + w.nseg - 1) / w.nseg + 3) / 4;
  size_t off = head;
  char* b = static_cast<char*>(base);
  auto take = [&](size_t bytes) {
    char* p = b ? b + off : nullptr;
    off += (bytes + 255) / 256 * 256;
    return p;
  };
  w.ws.tc = T;
  w.ws.r = r;
  w.seg_count = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)w.nb * w.nseg));
  w.seg_idx = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)w.nb * d_ff));
  w.ws.xs = reinterpret_cast<uint4*>(take(sizeof(uint4) * 2 * (size_t)((d + 31) / 32) * w.ntt * kWave));
  w.zf = reinterpret_cast<uint4*>(take(sizeof(uint4) * 16 * (size_t)w.ntt * w.nseg * w.qps));
  if (r > 0) {
    // the partial copies of z lie where zval goes later; a copy of its own where not even two fit there
    w.zparts = (int)(16 * (size_t)w.ntt * w.nseg * w.qps * sizeof(uint4) / (sizeof(float) * (size_t)T * r));
    w.ws.z = reinterpret_cast<float*>(w.zf);
    if (w.zparts < 2) {
      w.zparts = 1;
      w.ws.z = reinterpret_cast<float*>(take(sizeof(float) * (size_t)T * r));
    }
    w.zs = reinterpret_cast<uint4*>(take(sizeof(uint4) * 2 * (size_t)((r + 31) / 32) * w.ntt * kWave));
    if (has_g) w.ws.gx = reinterpret_cast<float*>(take(sizeof(float) * (size_t)T * d_ff));
  }
  if (out) *out = w;
  return off;
}

// z's partial copies, `*parts` of them: about one workgroup a CU, at least four iterations each.
template <class W, int NT>
hipError_t wide_z(const Shape& sh, const Form& form, const float* x, const void* lopa_a, const WideLayout& w, int* parts,
                  hipStream_t s) {
  const int C = sh.d / 8, units = (sh.r + kZRows - 1) / kZRows * w.nb;
  int P = (kWCus + units - 1) / units;
  const int most = wide_iterations(C) / 4;
  if (P > most) P = most;
  if (P > w.zparts) P = w.zparts;
  if (P < 1) P = 1;
  *parts = P;
  const int grid = units * P;
  const GWork gw{form, x, w.ws.gx, sh.T, sh.d, sh.d_ff, grid};
  const int extra = form.g_idx ? (g_items(sh.d_ff, sh.T) + kWThreads - 1) / kWThreads : 0;
  k_wide_z<W, NT><<<grid + extra, kWThreads, 0, s>>>(static_cast<const uint4*>(lopa_a), w.ws.xs, C, sh.T, sh.r, w.ntt, w.nb, P,
                                                 w.ws.z, sh.sc.a, gw);
  return hipGetLastError();
}

}  // namespace

// Row chunks of the down grid (units of S column groups x token blocks, one workgroup a CU): chunks of
// at least 512 rows (each adds T d fp32 atomics) and at most kWDnRows, kWDnSegs; of these counts the one
// with the least rounds over the CUs times a workgroup's iterations and kWDnFixed more (its list, first
// loads, sums and atomics).  A chunk too many costs a round: d 5120 (40 column groups), d_ff 15000, 33
// tokens, 7 chunks 59.4 us, 6 40.7; d 3072, d_ff 15000, 64 tokens, 11 chunks 51.1, 10 31.7.
constexpr int kWDnFixed = 8;
int wide_down_chunks(int units, int d_ff, int nseg) {
  const int rows = (d_ff + nseg - 1) / nseg;
  int per = kWDnRows / rows;
  if (per > kWDnSegs) per = kWDnSegs;
  const int least = (nseg + per - 1) / per, most = (d_ff + 511) / 512;
  int best = least;
  int64_t cost = INT64_MAX;
  for (int c = least; c == least || (c <= most && (int64_t)units * (c - 1) < 4 * kWCus); ++c) {
    const int64_t rounds = ((int64_t)units * c + kWCus - 1) / kWCus, t = rounds * (64 * kWDnFixed + d_ff / c);
    if (t < cost) cost = t, best = c;  // in rows, 64 an iteration
  }
  return best < nseg ? best : nseg;
}

namespace {

template <class W, int NT>
hipError_t wide_kernels(const Shape& sh, const WideArgs& a, const WideLayout& w, const void* w_down_t, hipStream_t s) {
  const int units = (w.nseg + kXcds - 1) / kXcds * kXcds;
  const hipError_t e = launch_gate_kernel_n(k_wide_gate_up<W, NT>, units * w.nb, kWThreads, s, a);
  if (e != hipSuccess) return e;
  const int S = (sh.d + kWCols - 1) / kWCols, R = wide_down_chunks(S * w.nb, sh.d_ff, w.nseg);
  const int du = (S * R + kXcds - 1) / kXcds * kXcds;
  k_wide_down<W, NT><<<du * w.nb, kWThreads, 0, s>>>(w.seg_count, w.seg_idx, w.zf, w.nseg, w.qps, sh.d_ff, R, w.ntt, w.nb,
                                                 static_cast<const uint4*>(w_down_t), sh.d / W::EPC, sh.d, sh.T, a.y);
  return hipGetLastError();
}

template <int NT>
hipError_t wide_format(const Shape& sh, Gate g, bool dense, const Form& form, const float* x, const void* lopa_a,
                       const void* gate_w, const void* w_up, const void* w_down_t, float t, const WideLayout& w, float* y,
                       hipStream_t s) {
  const bool lopa = g == Gate::LoPA;
  hipError_t e = launch_split_tokens(sh, x, w.ws, s);
  if (e != hipSuccess) return e;
  if (lopa) {
    int copies = 1;
    if (sh.wdt == 2) e = wide_z<WI8, NT>(sh, form, x, lopa_a, w, &copies, s);
    else if (sh.wdt == 3) e = wide_z<WI4, NT>(sh, form, x, lopa_a, w, &copies, s);
    else e = wide_z<WBf16, NT>(sh, form, x, lopa_a, w, &copies, s);
    if (e != hipSuccess) return e;
    if (form.rms_eps > 0.f) {
      e = launch_rms_norm(w.ws.z, copies, sh.T, sh.T, sh.r, form.rms_gain, form.rms_eps, s);
      if (e != hipSuccess) return e;
      copies = 1;  // the normalised z; the others are zeros now
    }
    const int nks = (sh.r + 31) / 32, n = nks * w.ntt * kWave;
    k_split_z<<<(n + kBlock - 1) / kBlock, kBlock, 0, s>>>(w.ws.z, copies, sh.r, sh.T, nks, w.ntt, w.zs);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  WideArgs a{};
  a.gate_w = static_cast<const uint4*>(gate_w);
  a.w_up = static_cast<const uint4*>(w_up);
  a.xs = w.ws.xs;
  a.zs = w.zs;
  a.Cu = sh.d / 8;
  a.Cg = lopa ? sh.r / 8 : a.Cu;
  a.T = sh.T;
  a.d = sh.d;
  a.d_ff = sh.d_ff;
  a.nseg = w.nseg;
  a.qps = w.qps;
  a.ntt = w.ntt;
  a.nb = w.nb;
  a.lopa = lopa;
  a.dense = dense;
  a.t = t;
  a.form = form;
  a.gx = w.ws.gx;
  a.s_g = lopa ? sh.sc.b : sh.sc.gate;
  a.s_up = sh.sc.up;
  a.s_down = sh.sc.down;
  a.seg_count = w.seg_count;
  a.seg_idx = w.seg_idx;
  a.zf = w.zf;
  a.seg_act = w.seg_act;
  a.meta = w.meta;
  a.y = y;
  if (sh.wdt == 2) return wide_kernels<WI8, NT>(sh, a, w, w_down_t, s);
  if (sh.wdt == 3) return wide_kernels<WI4, NT>(sh, a, w, w_down_t, s);
  return wide_kernels<WBf16, NT>(sh, a, w, w_down_t, s);
}

}  // namespace

// Bytes of workspace that a pass of sh.T tokens uses, `head` included.
size_t wide_pass_bytes(const Shape& sh, Gate g, const Form& form, size_t head) {
  return wide_layout(sh.T, sh.d, sh.d_ff, g == Gate::LoPA ? sh.r : 0, form.g_idx != nullptr, nullptr, head, nullptr);
}

namespace {
// A pass's regions fit `bytes` of workspace and every byte offset is below 2^31.
bool wide_pass_fits(const Shape& sh, Gate g, const Form& form, size_t head, size_t bytes) {
  const int64_t lim = int64_t(1) << 31;
  const int r = g == Gate::LoPA ? sh.r : 0;
  WideLayout w;
  return wide_layout(sh.T, sh.d, sh.d_ff, r, form.g_idx != nullptr, nullptr, head, &w) <= bytes &&
         256 * (int64_t)w.nseg * w.qps * kWTiles < lim && 4 * (int64_t)sh.T * sh.d < lim / 4 &&
         4 * (int64_t)sh.T * (r > 0 ? r : 1) < lim / 4;
}

// Passes of 64 against one pass here, 90%: 8B shape LoPA r = 512, 65 / 96 / 128 / 200 / 256 tokens
// 119.2 / 174.2 / 203.2 / 351.9 / 405.8 -> 108.1 / 116.8 / 126.7 / 162.7 / 170.6 us; d 512, d_ff 2000, 100
// tokens 55.9 -> 36.5; 70B shape LoPA r = 1024, 100 tokens 640.8 -> 319.9.
// A few tokens past 64 leave a second pass little to do, and 64 and the rest is then the cheaper way where
// this path's latency counts.  One pass / 64 and the rest, us a call:
//   one token over (the single-token kernels take it), bf16 LoPA d 128, d_ff 400 37.3 / 30.7, d 512,
//   d_ff 1500 41.6 / 42.4; standard gating d 256, d_ff 700 30.3 / 28.5, d 384, d_ff 1200 34.8 / 35.6;
//   one over long rows of few neurons, standard gating, d 4096: int4 d_ff 9000 115.0 / 105.7, 13000
//   122.3 / 120.9; int8 9000 111.1 / 106.9, 11000 115.1 / 115.9; bf16 5000 103.0 / 99.3, 7000 107.3 / 106.6;
//   LoPA, 72 tokens: int4 d 128, d_ff 400 39.4 / 36.1, d 384, d_ff 1152 45.1 / 43.5; int8 39.0 / 36.7, 44.3 /
//   44.7; bf16 d 32, d_ff 1000 6 % slower in one pass, d 256, d_ff 700 38.0 / 39.6.
bool rest_is_cheap(const Shape& sh, Gate g) {
  const int64_t n = (int64_t)sh.d * sh.d_ff;
  const bool lopa = g == Gate::LoPA, codes = sh.wdt != 1;
  if (sh.T == kTokChunk + 1 && n <= (lopa ? 1500000 : 640000)) return true;
  if (sh.T == kTokChunk + 1 && !lopa && sh.d >= 2048 && sh.d_ff <= (sh.wdt == 3 ? 12288 : sh.wdt == 2 ? 9216 : 6144))
    return true;
  if (!lopa) return false;
  return sh.T <= (codes && n <= 130000 ? 96 : 80) && n <= (codes ? 475000 : 130000);
}
}  // namespace

// Tokens of the passes of a call of sh.T: as few equal passes (in whole token tiles, of at most
// kWidePass) as have room for their regions in `bytes` of workspace, or 0 if the path does not take
// the call: 65 tokens or more a pass, bf16 or quantized rows that the 2..64-token kernels take.  A
// last pass of fewer tokens than the others is checked by itself: a layout need not shrink with its
// tokens (fewer blocks can mean smaller segments and so fewer zval quads, and z's copies then a
// region of their own).
int wide_pass_tokens(const Shape& sh, Gate g, const Form& form, size_t head, size_t bytes) {
  if (sh.wdt < 1 || sh.wdt > 3 || sh.T <= kTokChunk || rest_is_cheap(sh, g)) return 0;
  Shape one = sh;
  one.T = kTokChunk;
  if (!batched_ok(one, g)) return 0;
  for (int n = (sh.T + kWidePass - 1) / kWidePass;; ++n) {
    const int per = ((sh.T + n - 1) / n + 15) / 16 * 16;
    if (per <= kTokChunk) return 0;
    Shape pass = sh, last = sh;
    pass.T = sh.T < per ? sh.T : per;
    last.T = sh.T - (sh.T - 1) / per * per;
    if (wide_pass_fits(pass, g, form, head, bytes) &&
        (last.T <= kTokChunk || wide_pass_fits(last, g, form, head, bytes)))
      return per;
  }
}

hipError_t launch_wide(const Shape& sh, Gate g, bool dense, const Form& form, const float* x, const void* lopa_a,
                       const void* gate_w, const void* w_up, const void* w_down_t, float t, void* base, size_t head,
                       size_t bytes, float* y, hipStream_t s) {
  WideLayout w;
  if (wide_layout(sh.T, sh.d, sh.d_ff, g == Gate::LoPA ? sh.r : 0, form.g_idx != nullptr, base, head, &w) > bytes)
    return hipErrorInvalidValue;  // not a pass of wide_pass_tokens
  return wide_format<kWTiles>(sh, g, dense, form, x, lopa_a, gate_w, w_up, w_down_t, t, w, y, s);
}

// The regions of a pass of at most kTokChunk tokens, all in the workspace's own: zval and z's partial
// copies in zf (16 quads a segment of 64 rows, as there), z's planes in seg_zval.
void wide64_layout(const Shape& sh, Gate g, const Workspace& ws, WideLayout* out) {
  WideLayout w{};
  w.ntt = (ws.tc + 15) / 16;
  w.nb = 1;
  w.nseg = (sh.d_ff + kWRows / 2 - 1) / (kWRows / 2);
  w.qps = kWRows / 8;
  w.ws = ws;
  w.seg_count = ws.seg_count;
  w.seg_idx = ws.seg_idx;
  w.zf = ws.zf;
  if (g == Gate::LoPA) {
    w.zs = reinterpret_cast<uint4*>(ws.seg_zval);
    w.ws.z = reinterpret_cast<float*>(ws.zf);
    w.zparts = (int)(256 * (size_t)w.ntt * w.nseg * w.qps / (sizeof(float) * (size_t)sh.T * sh.r));
  }
  w.seg_act = ws.seg_act;
  w.meta = ws.meta;
  *out = w;
}

// Where 33..64 tokens take these kernels instead of the register-tiled ones: where segments of 64
// rows leave at most an eighth of the compute units idle in their last round (k_gate_up_mfma balances
// its segments over them whatever d_ff is), and the rows are long enough to carry the passes over z and
// the wider down workgroups.  Register-tiled -> these, 90%, us a call at 33 / 48 / 64 tokens:
//   bf16 d 1024, d_ff 16000, r 128   42.6 -> 47.9 / 47.2 -> 49.6 / 46.5 -> 53.2
//   int8                             41.5 -> 45.8 / 46.1 -> 46.8 / 45.4 -> 51.0
//   bf16 d 2048, d_ff 14336, r 256   58.8 -> 60.4 / 68.0 -> 62.7 / 64.4 -> 66.9
//   bf16 standard gating             63.8 -> 65.5 / 72.3 -> 66.7 / 68.4 -> 72.1
//   int8 / int4 64 tokens, r 256     62.7 -> 62.4 / 62.4 -> 62.7
//   bf16 d 2304, d_ff 14336, r 288   63.8 -> 63.8 / 72.1 -> 66.4 / 70.4 -> 71.3
//   bf16 d 4096, d_ff 14336, r 512   93.3 -> 87.4 / 108.9 -> 89.7 / 102.0 -> 95.9
//   bf16 standard gating             106.3 -> 101.0 / 121.6 -> 102.8 / 114.3 -> 112.4
//   int8 r 512                       90.2 -> 76.5 / 105.2 -> 79.0 / 98.3 -> 83.6
//   int4 r 512                       88.9 -> 81.5 / 104.1 -> 83.8 / 97.0 -> 86.8
//   bf16 r 512, the full form        100.8 -> 97.2 / - / 113.2 -> 108.2
// Fewer segments in the last round, bf16 standard gating at 64 tokens: d 4096 5 % slower here at 165 of
// them (d_ff 10500), even at 216 (13824); d 2304 6 % and 1 % slower.  LoPA, fewer tokens and codes gain
// from 188 on at d 4096; the line at 224 gives those up.  17 tokens, 8B shape: 63.4 -> 77.0.
// LoPA's z has to fit the regions above (ranks larger than d_ff do not).
constexpr int kWide64MinD = 2304, kWide64MinDQuant = 2048;
bool wide64_ok(const Shape& sh, Gate g, const Workspace& ws) {
  if (sh.wdt < 1 || sh.wdt > 3 || sh.T < kWide64Min || ws.tc > kTokChunk || !batched_ok(sh, g)) return false;
  if (sh.d < (sh.wdt == 1 ? kWide64MinD : kWide64MinDQuant)) return false;
  const int nseg = (sh.d_ff + kWRows / 2 - 1) / (kWRows / 2), rounds = (nseg + kWCus - 1) / kWCus;
  if (8 * nseg < 7 * kWCus * rounds) return false;
  if (g != Gate::LoPA) return true;
  WideLayout w;
  wide64_layout(sh, g, ws, &w);
  return w.zparts >= 1 &&
         sizeof(uint4) * 2 * (size_t)((sh.r + 31) / 32) * w.ntt * kWave <= sizeof(float) * (size_t)ws.tc * ws.slots;
}

hipError_t launch_wide64(const Shape& sh, Gate g, bool dense, const Form& form, const float* x, const void* lopa_a,
                         const void* gate_w, const void* w_up, const void* w_down_t, float t, Workspace& ws, float* y,
                         hipStream_t s) {
  WideLayout w;
  wide64_layout(sh, g, ws, &w);
  ws.nseg = w.nseg;
  return wide_format<4>(sh, g, dense, form, x, lopa_a, gate_w, w_up, w_down_t, t, w, y, s);
}

}  // namespace ffn
