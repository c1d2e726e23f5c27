// fp32 attention along one sequence dimension and its gradients (Eq. 3 per
// head; grouped key/value heads and a key length of its own for
// cross-attention): fp32 storage, fp32 products and accumulation, no operand
// rounded anywhere.
//
// Head widths up to 128 run on the fp32 matrix instruction
// (v_mfma_f32_32x32x2_f32).  Bound: the matrix cores, so the layout spends no
// instruction on moving operands between products.
//  * A wave owns 32 rows (queries in the forward and dQ kernels, keys in the
//    dK/dV kernel) as MFMA columns and keeps them in registers; the other side's
//    rows pass through LDS in tiles of 32, fetched one tile ahead into registers,
//    shared by the work-group's waves.
//  * Scores are computed as (tile rows) x (own rows): lane l32 + 32 g holds, for
//    its own row l32, tile rows 8 r4 + 4 g + i in register 4 r4 + i.  That is the
//    B operand of the d-row products (O^T = V^T P^T, dQ^T = K^T dZ^T, dV^T = dO^T P,
//    dK^T = Q^T dZ) as it stands, two tile rows (one per lane half) per MFMA, and
//    the A operand is read from the same LDS rows, 32 consecutive floats a half.
//  * Softmax statistics are per lane (one swap across the halves); the running
//    maximum is exact and a move rescales the accumulators.
//  * 4 waves (128 rows) share a work-group's tiles, in the forward 2 where 64 rows do;
//    1 wave when there are at most 32 rows, with one LDS buffer instead of two so that
//    more groups fit a CU.
// Registers, not LDS, set the occupancy (one or two waves per SIMD from D = 64 on), and
// the one-wave kernels, whose wave fetches whole tiles alone, run out of them in dK/dV:
// 10 spilled at D = 72 (44 bytes a lane), 134 at 96, 627 at 128 (four waves: 140).
// Measured (16 heads of 72): 8 frames of L = 256 forward 47 us (51 TFLOP/s), dQ 55
// and dK/dV 68 us; before, one wave walking a unit's keys with plain FMAs took
// 1095 us and the gradients, one thread per row and 32 columns, 9.7 + 10.7 ms.
// 256 units of L = 8: 31 (34) us forward, 90 (625) us backward.
//
// A few keys (wave_per_unit, thread_per_row below) are a fraction of a 32-row tile: the
// forward then runs plain FMAs, a wave per unit or a thread per row.
// Wider heads run the general kernels at the end: one thread per (unit, row,
// 32-column slice of the output), plain FMAs.
#include <math.h>

#include <algorithm>

#include "dsp_internal.h"

namespace dsp {
namespace {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

// Where a running maximum starts: finite, so that scores of -inf have probability 0
// (not NaN) before a row's first finite one.
constexpr float kLowest = -3.402823466e38f;

constexpr int DC = 32;  // output columns per thread of the general kernels

// Both directions' arguments; forward: o, lse are outputs and in = q's layout.
struct ParamsF {
  const float* q;
  const float* k;
  const float* v;
  const float* o;
  const float* dout;
  const float* lse;
  float* out_o;    // forward
  float* out_lse;  // forward, may be null
  float* dq;
  float* dk;
  float* dv;
  float* delta;
  int64_t b_q, x_q, r_q, b_kv, x_kv, r_kv, b_o, x_o, r_o;
  int64_t X, H, L, Lk, grp, D, n_dc;
  uint32_t n_blk;  // row blocks per unit
  int64_t first;   // this launch's first unit
  float scale;
  bool vec;       // every row starts on 16 bytes and D is a multiple of 4
};

__device__ __forceinline__ float other_half(float v) { return __shfl_xor(v, 32, 64); }

__device__ __forceinline__ float4 load4(const float* p, int64_t left, bool vec) {
  float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  if (left <= 0) return v;
  if (vec) return *reinterpret_cast<const float4*>(p);
  v.x = p[0];
  if (left > 1) v.y = p[1];
  if (left > 2) v.z = p[2];
  if (left > 3) v.w = p[3];
  return v;
}

// Own rows: lane (l32, g) holds columns 8 c + 4 g + {0..3} of its row.
template <int DP>
__device__ __forceinline__ void own_row(const float* row, bool valid, int64_t D, bool vec, int g,
                                        float4 (&r)[DP / 8]) {
#pragma unroll
  for (int c = 0; c < DP / 8; ++c) r[c] = load4(row + 8 * c + 4 * g, valid ? D - (8 * c + 4 * g) : 0, vec);
}

// 32 rows of a tensor: global -> registers -> LDS (pitch DP + 4 floats, an odd
// number of 16-byte chunks); rows past `rows` and columns past D are zero.
template <int DP, int NTHR>
struct RowTile {
  static constexpr int P = DP + 4, CPR = DP / 4;
  static constexpr int LOADS = (32 * CPR + NTHR - 1) / NTHR;
  static constexpr int ELEMS = 32 * P + 32;  // d-row reads of the last row run up to 32 floats on (results dropped)
  float4 pre[LOADS];
  // REPEAT: the last row fills up the group of 8 that d-row products read with it
  template <bool REPEAT = false>
  __device__ __forceinline__ void load(const float* base, int64_t stride, int64_t rows, int64_t D, bool vec) {
    const int last = (int)min(rows, (int64_t)32) - 1, end = REPEAT ? last | 7 : last;
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int e = (int)threadIdx.x + NTHR * i, r = e / CPR, c = (e % CPR) * 4;
      pre[i] = load4(base + (REPEAT ? min(r, last) : r) * stride + c, r <= end ? D - c : 0, vec);
    }
  }
  __device__ __forceinline__ void store(float* lds) const {
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int e = (int)threadIdx.x + NTHR * i, r = e / CPR, c = (e % CPR) * 4;
      if (32 * CPR % NTHR == 0 || r < 32) *reinterpret_cast<float4*>(lds + r * P + c) = pre[i];
    }
  }
};

// acc[tile row][own row] += tile . own^T
template <int DP>
__device__ __forceinline__ void score_step(const float* tile, const float4& own, int c, int l32, int g, floatx16& acc) {
  const float4 a = *reinterpret_cast<const float4*>(tile + l32 * (DP + 4) + 8 * c + 4 * g);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, own.x, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, own.y, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, own.z, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, own.w, acc, 0, 0, 0);
}

// acc_t[d][own row] += tile^T[d][tile row] w[tile row][own row], d = 32 t + l32.
// Groups of 8 tile rows past `rows` (weights 0) are left out.
template <int DP, int NT>
__device__ __forceinline__ void drow_product(const float* tile, const floatx16& w, int64_t rows, int l32, int g,
                                             floatx16 (&acc)[NT]) {
#pragma unroll
  for (int r4 = 0; r4 < 4; ++r4) {
    if (8 * r4 >= rows) break;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float* row = tile + (8 * r4 + 4 * g + e) * (DP + 4) + l32;
#pragma unroll
      for (int t = 0; t < NT; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(row[32 * t], w[4 * r4 + e], acc[t], 0, 0, 0);
    }
  }
}

template <int NT>
__device__ __forceinline__ void zero(floatx16 (&a)[NT]) {
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) a[t][r] = 0.0f;
}

// row[d] = acc[d] * f for the lane's own row
template <int NT>
__device__ __forceinline__ void store_own(float* row, const floatx16 (&acc)[NT], int64_t D, bool vec, int g, float f) {
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const int64_t d = 32 * t + 8 * r4 + 4 * g;
      if (d >= D) continue;
      const float v[4] = {acc[t][4 * r4] * f, acc[t][4 * r4 + 1] * f, acc[t][4 * r4 + 2] * f, acc[t][4 * r4 + 3] * f};
      if (vec) {
        *reinterpret_cast<float4*>(row + d) = make_float4(v[0], v[1], v[2], v[3]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (d + e < D) row[d + e] = v[e];
      }
    }
}

// The work-group's block of a unit's rows: units in contiguous ranges per XCD
// (their tiles are then shared through one L2).
__device__ __forceinline__ uint32_t xcd_block() {
  const uint32_t n = gridDim.x, per = n >> 3, extra = n & 7u, xcd = blockIdx.x & 7u;
  return xcd * per + (xcd < extra ? xcd : extra) + (blockIdx.x >> 3);
}

template <int DP, int NW>
struct Geo {
  static constexpr int NTHR = 64 * NW, NB = NW == 1 ? 1 : 2, NT = (DP + 31) / 32;
  using Tile = RowTile<DP, NTHR>;
};

template <int DP, int NW>
__global__ __launch_bounds__(64 * NW) void attn_f32_mfma_kernel(ParamsF p) {
  using G = Geo<DP, NW>;
  constexpr int NB = G::NB, NT = G::NT, TE = G::Tile::ELEMS;
  __shared__ __attribute__((aligned(16))) float lds[NB * 2 * TE];
  const int lane = threadIdx.x & 63, l32 = lane & 31, g = lane >> 5;
  const uint32_t blk = xcd_block();
  const int64_t unit = p.first + blk / p.n_blk, qi = (int64_t)(blk % p.n_blk) * (32 * NW) + 32 * (threadIdx.x >> 6) + l32;
  const int64_t h = unit % p.H, bx = unit / p.H, xx = bx % p.X, bb = bx / p.X;
  const bool valid = qi < p.L;
  float4 q[DP / 8];
  own_row<DP>(p.q + bb * p.b_q + xx * p.x_q + h * p.D + qi * p.r_q, valid, p.D, p.vec, g, q);
  const int64_t kvb = bb * p.b_kv + xx * p.x_kv + (h / p.grp) * p.D;
  const float *kg = p.k + kvb, *vg = p.v + kvb;

  typename G::Tile kt, vt;
  kt.load(kg, p.r_kv, p.Lk, p.D, p.vec);
  vt.load(vg, p.r_kv, p.Lk, p.D, p.vec);
  floatx16 o[NT];
  zero(o);
  float m = kLowest, l = 0.0f;
  int buf = 0;
  for (int64_t k0 = 0; k0 < p.Lk; k0 += 32) {
    float* ks = lds + buf * 2 * TE;
    float* vs = ks + TE;
    if (NB == 1) __syncthreads();  // the previous tile is consumed
    kt.store(ks);
    vt.store(vs);
    __syncthreads();  // (two buffers: every wave is past the tile before the previous)
    if (k0 + 32 < p.Lk) {
      kt.load(kg + (k0 + 32) * p.r_kv, p.r_kv, p.Lk - k0 - 32, p.D, p.vec);
      vt.load(vg + (k0 + 32) * p.r_kv, p.r_kv, p.Lk - k0 - 32, p.D, p.vec);
    }
    if (NB == 2) buf ^= 1;
    floatx16 s[1];
    zero(s);
#pragma unroll
    for (int c = 0; c < DP / 8; ++c) score_step<DP>(ks, q[c], c, l32, g, s[0]);
    float mt = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[0][r] *= p.scale;
      if (k0 + 32 > p.Lk && k0 + 8 * (r / 4) + 4 * g + r % 4 >= p.Lk) s[0][r] = -INFINITY;
      mt = fmaxf(mt, s[0][r]);
    }
    mt = fmaxf(mt, other_half(mt));
    if (__any(mt > m)) {
      const float mn = fmaxf(m, mt), corr = expf(m - mn);  // 0 for the first tile
      l *= corr;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] *= corr;
      m = mn;
    }
    float sum = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[0][r] = expf(s[0][r] - m);
      sum += s[0][r];
    }
    l += sum;
    drow_product<DP, NT>(vs, s[0], p.Lk - k0, l32, g, o);
  }
  l += other_half(l);
  if (l == 0.0f) l = NAN;  // a softmax over scores that are all -inf
  if (!valid) return;
  store_own<NT>(p.out_o + bb * p.b_o + xx * p.x_o + h * p.D + qi * p.r_o, o, p.D, p.vec, g, 1.0f / l);
  if (p.out_lse && g == 0) p.out_lse[unit * p.L + qi] = m + logf(l);
}

// dQ (and Delta = rowsum(dO * O)) for 32 NW queries of a query head
template <int DP, int NW>
__global__ __launch_bounds__(64 * NW) void attn_bwd_f32_dq_mfma_kernel(ParamsF p) {
  using G = Geo<DP, NW>;
  constexpr int NB = G::NB, NT = G::NT, TE = G::Tile::ELEMS;
  __shared__ __attribute__((aligned(16))) float lds[NB * 2 * TE];
  const int lane = threadIdx.x & 63, l32 = lane & 31, g = lane >> 5;
  const uint32_t blk = xcd_block();
  const int64_t unit = p.first + blk / p.n_blk, qi = (int64_t)(blk % p.n_blk) * (32 * NW) + 32 * (threadIdx.x >> 6) + l32;
  const int64_t h = unit % p.H, bx = unit / p.H, xx = bx % p.X, bb = bx / p.X;
  const bool valid = qi < p.L;
  const int64_t qb = bb * p.b_q + xx * p.x_q + h * p.D + qi * p.r_q;
  const int64_t ob = bb * p.b_o + xx * p.x_o + h * p.D + qi * p.r_o;
  float4 q[DP / 8], d[DP / 8];
  own_row<DP>(p.q + qb, valid, p.D, p.vec, g, q);
  own_row<DP>(p.dout + ob, valid, p.D, p.vec, g, d);
  float delta = 0.0f;
  {
    float4 o[DP / 8];
    own_row<DP>(p.o + ob, valid, p.D, p.vec, g, o);
#pragma unroll
    for (int c = 0; c < DP / 8; ++c)
      delta = fmaf(d[c].x, o[c].x, fmaf(d[c].y, o[c].y, fmaf(d[c].z, o[c].z, fmaf(d[c].w, o[c].w, delta))));
    delta += other_half(delta);
  }
  const float lse = valid ? p.lse[unit * p.L + qi] : INFINITY;  // rows past L: probabilities 0
  if (valid && g == 0) p.delta[unit * p.L + qi] = delta;
  const int64_t kvb = bb * p.b_kv + xx * p.x_kv + (h / p.grp) * p.D;
  const float *kg = p.k + kvb, *vg = p.v + kvb;

  typename G::Tile kt, vt;
  kt.load(kg, p.r_kv, p.Lk, p.D, p.vec);
  vt.load(vg, p.r_kv, p.Lk, p.D, p.vec);
  floatx16 dq[NT];
  zero(dq);
  int buf = 0;
  for (int64_t k0 = 0; k0 < p.Lk; k0 += 32) {
    float* ks = lds + buf * 2 * TE;
    float* vs = ks + TE;
    if (NB == 1) __syncthreads();
    kt.store(ks);
    vt.store(vs);
    __syncthreads();
    if (k0 + 32 < p.Lk) {
      kt.load(kg + (k0 + 32) * p.r_kv, p.r_kv, p.Lk - k0 - 32, p.D, p.vec);
      vt.load(vg + (k0 + 32) * p.r_kv, p.r_kv, p.Lk - k0 - 32, p.D, p.vec);
    }
    if (NB == 2) buf ^= 1;
    floatx16 s[2];
    zero(s);
#pragma unroll
    for (int c = 0; c < DP / 8; ++c) {
      score_step<DP>(ks, q[c], c, l32, g, s[0]);
      score_step<DP>(vs, d[c], c, l32, g, s[1]);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[0][r] = expf(s[0][r] * p.scale - lse) * (s[1][r] - delta);
      // (the whole product: an infinite Delta or dO row times 0 is not 0)
      if (k0 + 32 > p.Lk && k0 + 8 * (r / 4) + 4 * g + r % 4 >= p.Lk) s[0][r] = 0.0f;
    }
    drow_product<DP, NT>(ks, s[0], p.Lk - k0, l32, g, dq);
  }
  if (valid) store_own<NT>(p.dq + qb, dq, p.D, p.vec, g, p.scale);
}

// dK and dV for 32 NW keys of a key/value head: the query tiles of every query
// head of its group in turn (a fixed order)
template <int DP, int NW>
__global__ __launch_bounds__(64 * NW) void attn_bwd_f32_dkv_mfma_kernel(ParamsF p) {
  using G = Geo<DP, NW>;
  constexpr int NB = G::NB, NT = G::NT, TE = G::Tile::ELEMS;
  __shared__ __attribute__((aligned(16))) float lds[NB * (2 * TE + 64)];
  const int lane = threadIdx.x & 63, l32 = lane & 31, g = lane >> 5;
  const uint32_t blk = xcd_block();
  const int64_t Hkv = p.H / p.grp;
  const int64_t unit = p.first + blk / p.n_blk, key = (int64_t)(blk % p.n_blk) * (32 * NW) + 32 * (threadIdx.x >> 6) + l32;
  const int64_t hk = unit % Hkv, bx = unit / Hkv, xx = bx % p.X, bb = bx / p.X;
  const bool valid = key < p.Lk;
  const int64_t kvb = bb * p.b_kv + xx * p.x_kv + hk * p.D + key * p.r_kv;
  float4 k[DP / 8], v[DP / 8];
  own_row<DP>(p.k + kvb, valid, p.D, p.vec, g, k);
  own_row<DP>(p.v + kvb, valid, p.D, p.vec, g, v);
  floatx16 dk[NT], dv[NT];
  zero(dk);
  zero(dv);
  typename G::Tile qt, dt;
  float stat = 0.0f;  // thread t < 32: lse of tile row t, t in [32, 64): Delta of row t - 32
  // tile i: query head hk grp + i / n_q, rows 32 (i % n_q) ..
  const int64_t n_q = (p.L + 31) / 32, n = p.grp * n_q;
  auto fetch = [&](int64_t i) {
    const int64_t hq = hk * p.grp + i / n_q, r0 = (i % n_q) * 32;
    // (Q rows past L repeat a real row: against zeros the score of an infinite key, and with it
    // the probability, would be NaN)
    qt.template load<true>(p.q + bb * p.b_q + xx * p.x_q + hq * p.D + r0 * p.r_q, p.r_q, p.L - r0, p.D, p.vec);
    dt.load(p.dout + bb * p.b_o + xx * p.x_o + hq * p.D + r0 * p.r_o, p.r_o, p.L - r0, p.D, p.vec);
    if (threadIdx.x < 64) {
      const int64_t r = r0 + l32, at = (bx * p.H + hq) * p.L + r;
      // rows past L: lse +inf, so their probabilities are 0
      stat = threadIdx.x < 32 ? (r < p.L ? p.lse[at] : INFINITY) : (r < p.L ? p.delta[at] : 0.0f);
    }
  };
  fetch(0);
  int buf = 0;
  for (int64_t i = 0; i < n; ++i) {
    float* qs = lds + buf * (2 * TE + 64);
    float* ds = qs + TE;
    float* st = ds + TE;
    if (NB == 1) __syncthreads();
    qt.store(qs);
    dt.store(ds);
    if (threadIdx.x < 64) st[threadIdx.x] = stat;
    __syncthreads();
    if (i + 1 < n) fetch(i + 1);
    if (NB == 2) buf ^= 1;
    floatx16 s[2];
    zero(s);
#pragma unroll
    for (int c = 0; c < DP / 8; ++c) {
      score_step<DP>(qs, k[c], c, l32, g, s[0]);
      score_step<DP>(ds, v[c], c, l32, g, s[1]);
    }
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const float4 ls = *reinterpret_cast<const float4*>(st + 8 * r4 + 4 * g);
      const float4 de = *reinterpret_cast<const float4*>(st + 32 + 8 * r4 + 4 * g);
      const float lv[4] = {ls.x, ls.y, ls.z, ls.w}, dl[4] = {de.x, de.y, de.z, de.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 4 * r4 + e;
        s[0][r] = expf(s[0][r] * p.scale - lv[e]);
        s[1][r] = s[0][r] * (s[1][r] - dl[e]);
      }
    }
    const int64_t left = p.L - (i % n_q) * 32;
    drow_product<DP, NT>(ds, s[0], left, l32, g, dv);
    drow_product<DP, NT>(qs, s[1], left, l32, g, dk);
  }
  if (!valid) return;
  store_own<NT>(p.dk + kvb, dk, p.D, p.vec, g, p.scale);
  store_own<NT>(p.dv + kvb, dv, p.D, p.vec, g, 1.0f);
}

// ---------------------------------------------------------------- few keys
// Forward, one wave per unit, plain FMAs: lanes own queries lane, lane + 64, .. with the
// query row and the D output columns in registers, the keys and values pass through
// LDS in chunks of 32 rows (every lane reads the same row: a broadcast), and the softmax
// runs online.  A few keys are a fraction of the 32-row tile the matrix instructions
// work through, and this kernel moves only the rows there are.
template <int D>
__global__ __launch_bounds__(64) void attn_f32_unit_kernel(ParamsF p) {
  constexpr int KC = 32;
  __shared__ __attribute__((aligned(16))) float ks[KC * D];
  __shared__ __attribute__((aligned(16))) float vs[KC * D];
  const int lane = threadIdx.x;
  const int64_t unit = p.first + blockIdx.x;
  const int64_t h = unit % p.H, bx = unit / p.H, xx = bx % p.X, bb = bx / p.X;
  const float* qg = p.q + bb * p.b_q + xx * p.x_q + h * D;
  const int64_t kvb = bb * p.b_kv + xx * p.x_kv + (h / p.grp) * D;
  const float *kg = p.k + kvb, *vg = p.v + kvb;
  float* og = p.out_o + bb * p.b_o + xx * p.x_o + h * D;
  for (int64_t q0 = 0; q0 < p.L; q0 += 64) {
    const int64_t qi = q0 + lane;
    const bool valid = qi < p.L;
    float qr[D], acc[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
      qr[d] = valid ? qg[qi * p.r_q + d] : 0.0f;
      acc[d] = 0.0f;
    }
    float m = kLowest, l = 0.0f;
    for (int64_t k0 = 0; k0 < p.Lk; k0 += KC) {
      const int nk = (int)min((int64_t)KC, p.Lk - k0);
      __syncthreads();  // the previous chunk is consumed
      for (int e = lane; e < nk * D; e += 64) {
        const int r = e / D, c = e - r * D;
        ks[e] = kg[(k0 + r) * p.r_kv + c];
        vs[e] = vg[(k0 + r) * p.r_kv + c];
      }
      __syncthreads();
      for (int j = 0; j < nk; ++j) {
        float sc = 0.0f;
#pragma unroll
        for (int d = 0; d < D; ++d) sc = fmaf(qr[d], ks[j * D + d], sc);
        sc *= p.scale;
        if (sc > m) {
          const float corr = expf(m - sc);  // 0 for the first key
          l *= corr;
#pragma unroll
          for (int d = 0; d < D; ++d) acc[d] *= corr;
          m = sc;
        }
        const float e = expf(sc - m);
        l += e;
#pragma unroll
        for (int d = 0; d < D; ++d) acc[d] = fmaf(e, vs[j * D + d], acc[d]);
      }
    }
    if (l == 0.0f) l = NAN;  // a softmax over scores that are all -inf
    if (valid) {
      const float inv = 1.0f / l;
      float* orow = og + qi * p.r_o;
#pragma unroll
      for (int d = 0; d < D; ++d) orow[d] = acc[d] * inv;
      if (p.out_lse) p.out_lse[unit * p.L + qi] = m + logf(l);
    }
  }
}

// ---------------------------------------------------------------- general kernels (any head width)

__device__ __forceinline__ float dotf(const float* a, const float* b, int64_t n) {
  float s = 0.0f;
  for (int64_t d = 0; d < n; ++d) s = fmaf(a[d], b[d], s);
  return s;
}

// A first pass over the keys finds the row maximum of the scaled scores, a second
// accumulates exp(score - max) and the weighted values of the thread's columns.
__global__ __launch_bounds__(256) void attn_f32_kernel(ParamsF p, int64_t total) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (tid >= total) return;
  // tid -> (unit, query, column slice), slice fastest
  const int64_t dc = tid % p.n_dc, uq = tid / p.n_dc;
  const int64_t qi = uq % p.L, unit = uq / p.L;
  const int64_t h = unit % p.H, bx = unit / p.H, xx = bx % p.X, bb = bx / p.X;
  const float* qrow = p.q + bb * p.b_q + xx * p.x_q + h * p.D + qi * p.r_q;
  const int64_t kv_base = bb * p.b_kv + xx * p.x_kv + (h / p.grp) * p.D;
  const float* kb = p.k + kv_base;
  const float* vb = p.v + kv_base;
  float m = -INFINITY;
  for (int64_t j = 0; j < p.Lk; ++j) m = fmaxf(m, dotf(qrow, kb + j * p.r_kv, p.D) * p.scale);
  const int64_t c0 = dc * DC;
  const int64_t nc = min((int64_t)DC, p.D - c0);
  float acc[DC];
#pragma unroll
  for (int c = 0; c < DC; ++c) acc[c] = 0.0f;
  float l = 0.0f;
  for (int64_t j = 0; j < p.Lk; ++j) {
    const float e = expf(dotf(qrow, kb + j * p.r_kv, p.D) * p.scale - m);
    l += e;
    const float* vrow = vb + j * p.r_kv + c0;
#pragma unroll
    for (int c = 0; c < DC; ++c)
      if (c < nc) acc[c] = fmaf(e, vrow[c], acc[c]);
  }
  float* orow = p.out_o + bb * p.b_o + xx * p.x_o + h * p.D + qi * p.r_o + c0;
  const float inv = 1.0f / l;
  if (p.out_lse && dc == 0) p.out_lse[unit * p.L + qi] = m + logf(l);
#pragma unroll
  for (int c = 0; c < DC; ++c)
    if (c < nc) orow[c] = acc[c] * inv;
}

__global__ __launch_bounds__(256) void attn_bwd_f32_dq_kernel(ParamsF p, int64_t total) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (tid >= total) return;
  const int64_t c0 = (tid % p.n_dc) * DC, ur = tid / p.n_dc;
  const int64_t nc = min((int64_t)DC, p.D - c0);
  const int64_t row = ur % p.L, unit = ur / p.L;
  const int64_t h = unit % p.H, bx = unit / p.H, xx = bx % p.X, bb = bx / p.X;
  const float* qrow = p.q + bb * p.b_q + xx * p.x_q + h * p.D + row * p.r_q;
  const int64_t ob = bb * p.b_o + xx * p.x_o + h * p.D + row * p.r_o;
  const int64_t kvb = bb * p.b_kv + xx * p.x_kv + (h / p.grp) * p.D;
  const float* drow = p.dout + ob;
  const float delta = dotf(drow, p.o + ob, p.D);
  const float lse = p.lse[unit * p.L + row];
  if (c0 == 0) p.delta[unit * p.L + row] = delta;
  float acc[DC];
#pragma unroll
  for (int c = 0; c < DC; ++c) acc[c] = 0.0f;
  for (int64_t j = 0; j < p.Lk; ++j) {
    const float* krow = p.k + kvb + j * p.r_kv;
    const float pr = expf(dotf(qrow, krow, p.D) * p.scale - lse);
    const float dz = pr * (dotf(drow, p.v + kvb + j * p.r_kv, p.D) - delta);
#pragma unroll
    for (int c = 0; c < DC; ++c)
      if (c < nc) acc[c] = fmaf(dz, krow[c0 + c], acc[c]);
  }
  float* out = p.dq + bb * p.b_q + xx * p.x_q + h * p.D + row * p.r_q + c0;
#pragma unroll
  for (int c = 0; c < DC; ++c)
    if (c < nc) out[c] = acc[c] * p.scale;
}

__global__ __launch_bounds__(256) void attn_bwd_f32_dkv_kernel(ParamsF p, int64_t total) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (tid >= total) return;
  const int64_t Hkv = p.H / p.grp;
  const int64_t c0 = (tid % p.n_dc) * DC, ur = tid / p.n_dc;
  const int64_t nc = min((int64_t)DC, p.D - c0);
  const int64_t key = ur % p.Lk, unit = ur / p.Lk;
  const int64_t hk = unit % Hkv, bx = unit / Hkv, xx = bx % p.X, bb = bx / p.X;
  const int64_t kvb = bb * p.b_kv + xx * p.x_kv + hk * p.D + key * p.r_kv;
  const float* krow = p.k + kvb;
  const float* vrow = p.v + kvb;
  float ak[DC], av[DC];
#pragma unroll
  for (int c = 0; c < DC; ++c) ak[c] = av[c] = 0.0f;
  for (int64_t hq = hk * p.grp; hq < (hk + 1) * p.grp; ++hq) {
    const int64_t uq = bx * p.H + hq;
    for (int64_t i = 0; i < p.L; ++i) {
      const float* qrow = p.q + bb * p.b_q + xx * p.x_q + hq * p.D + i * p.r_q;
      const float* drow = p.dout + bb * p.b_o + xx * p.x_o + hq * p.D + i * p.r_o;
      const float pr = expf(dotf(qrow, krow, p.D) * p.scale - p.lse[uq * p.L + i]);
      const float dz = pr * (dotf(drow, vrow, p.D) - p.delta[uq * p.L + i]);
#pragma unroll
      for (int c = 0; c < DC; ++c)
        if (c < nc) {
          ak[c] = fmaf(dz, qrow[c0 + c], ak[c]);
          av[c] = fmaf(pr, drow[c0 + c], av[c]);
        }
    }
  }
  float* ok = p.dk + kvb + c0;
  float* ov = p.dv + kvb + c0;
#pragma unroll
  for (int c = 0; c < DC; ++c)
    if (c < nc) {
      ok[c] = ak[c] * p.scale;
      ov[c] = av[c];
    }
}

bool rows_al16(const void* p, const int64_t st[3]) {
  return reinterpret_cast<uintptr_t>(p) % 16 == 0 && st[0] % 4 == 0 && st[1] % 4 == 0 && st[2] % 4 == 0;
}

// The padded head width whose instance takes width D (0: none).
int padded_width(int64_t D) { return D <= 16 ? 16 : D <= 32 ? 32 : D <= 64 ? 64 : D <= 72 ? 72 : D <= 96 ? 96 : D <= 128 ? 128 : 0; }

// Whether the forward runs a wave per unit.  Times (wave per unit / matrix kernel, us),
// units of L = Lk rows:
//   D = 72: 1024 units of 3 rows 8 / 9, of 4 9 / 9; 8192 of 4 36 / 54, of 6 47 / 54, of 8 60 / 56;
//   D = 96: 8192 of 4 59 / 62; D = 32: 1024 of 4 6 / 6, 8192 of 6 17 / 22, of 8 21 / 22, of 10 26 / 24;
//   D = 16: 8192 of 8 14 / 14, of 33 42 / 46; 32768 of 8 34 / 44, of 33 120 / 165, of 64 on 300 keys 888 / 956,
//   of 65 413 / 517.
// At D = 16 the matrix tiles' padding also decides for many longer units: 32-row waves
// and 32-key tiles against 64-row waves and single keys.
bool wave_per_unit(int64_t D, int64_t units, int64_t L, int64_t Lk) {
  if (D != 16 && D != 32 && D != 64 && D != 72 && D != 80 && D != 96) return false;
  if (L <= 64 && Lk <= (D <= 32 ? 4 : 3)) return true;
  if (L <= 64 && units >= 2048 && Lk <= (D <= 32 ? 8 : D <= 80 ? 6 : 4)) return true;
  if (L <= 64 && units >= 16384 && D <= 32 && Lk <= 10) return true;
  if (D > 16 || units < 8192 || L <= 32 || L > 256) return false;
  const int64_t waves = L <= 64 ? 2 : (L + 127) / 128 * 4;  // of the matrix kernel
  return 2 * ((L + 63) / 64) * Lk * 100 <= 95 * waves * ((Lk + 31) / 32) * 32;
}

// Whether the forward's general kernel (a thread per row and 32 columns) is the faster
// one at the other widths: a few keys of very many short units.  (general / matrix, us)
// D = 40: 4096 units of one row 18 / 24, 8192 of 3 37 / 45, 32768 of 4 240 / 167; D = 24: 8192 of
// one 20 / 22, 32768 of 2 34 / 72; D = 8: 8192 of 4 11 / 14, of 5 15 / 14, 32768 of 6 36 / 44.
bool thread_per_row(int64_t D, int64_t units, int64_t L, int64_t Lk) {
  if (L > 64 || D >= 96) return false;
  if (D < 16) return Lk <= (units >= 16384 ? 6 : units >= 8192 ? 4 : 0);
  if (D < 32) return units >= 16384 && Lk <= 2;
  return Lk <= (units >= 8192 ? 3 : units >= 4096 ? 2 : 0);
}

enum Which { FWD, DQ, DKV };

template <int DP, int NW>
void launch_mfma_fwd(const ParamsF& p, uint32_t blocks, hipStream_t s) {
  hipLaunchKernelGGL((attn_f32_mfma_kernel<DP, NW>), dim3(blocks), dim3(64 * NW), 0, s, p);
}

template <int DP, int NW>
void launch_mfma(Which which, const ParamsF& p, uint32_t blocks, hipStream_t s) {
  const dim3 g(blocks), b(64 * NW);
  if (which == FWD)
    launch_mfma_fwd<DP, NW>(p, blocks, s);
  else if (which == DQ)
    hipLaunchKernelGGL((attn_bwd_f32_dq_mfma_kernel<DP, NW>), g, b, 0, s, p);
  else
    hipLaunchKernelGGL((attn_bwd_f32_dkv_mfma_kernel<DP, NW>), g, b, 0, s, p);
}

// One kernel over `units` units of `rows` owned rows each.
int launch_units(Which which, ParamsF p, int64_t units, int64_t rows, hipStream_t s) {
  if (which == FWD && wave_per_unit(p.D, units, p.L, p.Lk)) {
    const int64_t most = grid_blocks(64);
    for (p.first = 0; p.first < units; p.first += most) {
      const dim3 g((uint32_t)std::min(most, units - p.first)), b(64);
      switch (p.D) {
        case 16: hipLaunchKernelGGL(attn_f32_unit_kernel<16>, g, b, 0, s, p); break;
        case 32: hipLaunchKernelGGL(attn_f32_unit_kernel<32>, g, b, 0, s, p); break;
        case 64: hipLaunchKernelGGL(attn_f32_unit_kernel<64>, g, b, 0, s, p); break;
        case 72: hipLaunchKernelGGL(attn_f32_unit_kernel<72>, g, b, 0, s, p); break;
        case 80: hipLaunchKernelGGL(attn_f32_unit_kernel<80>, g, b, 0, s, p); break;
        default: hipLaunchKernelGGL(attn_f32_unit_kernel<96>, g, b, 0, s, p); break;
      }
      const int st = last_launch_status();
      if (st != DSP_OK) return st;
    }
    return DSP_OK;
  }
  // 33 to 64 rows: two waves where there are enough units (D = 72, us with four / two waves:
  // 8192 units of 33 rows 319 / 165, 1024 43 / 27, 64 12.3 / 12.9: few units gain from four
  // waves fetching a tile).  In the gradients four hold fewer registers.
  const int nw = rows <= 32 ? 1 : rows <= 64 && which == FWD && units >= 512 ? 2 : 4;
  const int64_t n_blk = (rows + 32 * nw - 1) / (32 * nw), most = grid_blocks(64 * nw) / n_blk;  // units of one grid
  const int dp = padded_width(p.D);
  if (dp && most > 0 && !(which == FWD && thread_per_row(p.D, units, p.L, p.Lk))) {
    // one launch, or several where the threads are too many for a grid
    p.n_blk = (uint32_t)n_blk;
    for (p.first = 0; p.first < units; p.first += most) {
      const uint32_t n = (uint32_t)(std::min(most, units - p.first) * n_blk);
#define DSP_F32_CASE(DP_)                                 \
  case DP_:                                               \
    nw == 1   ? launch_mfma<DP_, 1>(which, p, n, s)       \
    : nw == 2 ? launch_mfma_fwd<DP_, 2>(p, n, s)          \
              : launch_mfma<DP_, 4>(which, p, n, s);      \
    break
      switch (dp) {
        DSP_F32_CASE(16);
        DSP_F32_CASE(32);
        DSP_F32_CASE(64);
        DSP_F32_CASE(72);
        DSP_F32_CASE(96);
        DSP_F32_CASE(128);
      }
#undef DSP_F32_CASE
      const int st = last_launch_status();
      if (st != DSP_OK) return st;
    }
    return DSP_OK;
  }
  const int64_t total = units * rows * p.n_dc, gen = (total + 255) / 256;
  if (gen >= (int64_t(1) << 31)) return DSP_ERR_SHAPE;
  const dim3 g((uint32_t)gen), b(256);
  if (which == FWD)
    hipLaunchKernelGGL(attn_f32_kernel, g, b, 0, s, p, total);
  else if (which == DQ)
    hipLaunchKernelGGL(attn_bwd_f32_dq_kernel, g, b, 0, s, p, total);
  else
    hipLaunchKernelGGL(attn_bwd_f32_dkv_kernel, g, b, 0, s, p, total);
  return last_launch_status();
}

}  // namespace

int launch_attn_f32(const AttnArgs& a, hipStream_t s) {
  ParamsF p = {};
  p.q = static_cast<const float*>(a.q);
  p.k = static_cast<const float*>(a.k);
  p.v = static_cast<const float*>(a.v);
  p.out_o = static_cast<float*>(a.o);
  p.out_lse = a.lse;
  const int64_t in[3] = {a.b_stride_in, a.x_stride_in, a.r_stride_in};
  const int64_t kv[3] = {a.b_stride_kv, a.x_stride_kv, a.r_stride_kv};
  const int64_t out[3] = {a.b_stride_out, a.x_stride_out, a.r_stride_out};
  p.b_q = in[0];
  p.x_q = in[1];
  p.r_q = in[2];
  p.b_kv = kv[0];
  p.x_kv = kv[1];
  p.r_kv = kv[2];
  p.b_o = out[0];
  p.x_o = out[1];
  p.r_o = out[2];
  p.X = a.X;
  p.H = a.H;
  p.L = a.L;
  p.Lk = a.Lk;
  p.grp = a.H / a.Hkv;
  p.D = a.D;
  p.n_dc = (a.D + DC - 1) / DC;
  p.scale = a.scale;
  p.vec = a.D % 4 == 0 && rows_al16(a.q, in) && rows_al16(a.k, kv) && rows_al16(a.v, kv) && rows_al16(a.o, out);
  if (a.B * a.X * a.L == 0) return DSP_OK;
  return launch_units(FWD, p, a.B * a.X * a.H, a.L, s);
}

int launch_attn_bwd_f32(const AttnBwdArgs& a, hipStream_t s) {
  ParamsF p = {};
  p.q = static_cast<const float*>(a.q);
  p.k = static_cast<const float*>(a.k);
  p.v = static_cast<const float*>(a.v);
  p.o = static_cast<const float*>(a.o);
  p.dout = static_cast<const float*>(a.dout);
  p.dq = static_cast<float*>(a.dq);
  p.dk = static_cast<float*>(a.dk);
  p.dv = static_cast<float*>(a.dv);
  p.lse = a.lse;
  p.delta = a.delta;
  p.b_q = a.q_strides[0];
  p.x_q = a.q_strides[1];
  p.r_q = a.q_strides[2];
  p.b_kv = a.kv_strides[0];
  p.x_kv = a.kv_strides[1];
  p.r_kv = a.kv_strides[2];
  p.b_o = a.o_strides[0];
  p.x_o = a.o_strides[1];
  p.r_o = a.o_strides[2];
  p.X = a.X;
  p.H = a.H;
  p.L = a.L;
  p.Lk = a.Lk;
  p.grp = a.H / a.Hkv;
  p.D = a.D;
  p.n_dc = (a.D + DC - 1) / DC;
  p.scale = a.scale;
  p.vec = a.D % 4 == 0 && rows_al16(a.q, a.q_strides) && rows_al16(a.k, a.kv_strides) &&
          rows_al16(a.v, a.kv_strides) && rows_al16(a.o, a.o_strides) && rows_al16(a.dout, a.o_strides) &&
          rows_al16(a.dq, a.q_strides) && rows_al16(a.dk, a.kv_strides) && rows_al16(a.dv, a.kv_strides);
  if (a.B * a.X * a.L == 0) return DSP_OK;
  const int st = launch_units(DQ, p, a.B * a.X * a.H, a.L, s);
  if (st != DSP_OK || a.Lk == 0) return st;
  return launch_units(DKV, p, a.B * a.X * a.Hkv, a.Lk, s);
}

}  // namespace dsp
