// One attention sublayer of the projection-only fp32 chain in one kernel, for
// small shapes: for a group of L consecutive token rows (a frame for the
// spatial half, a spatial location for the temporal half -- the reshape of
// Eq. 7-8),
//     out_rows = Attn(x_rows W_qkv + b_qkv) W_o + b_o
// with Attn the per-head softmax attention of Eq. 3 (heads as in Eq. 1-2).
// At these sizes the separate GEMM and attention launches are bound by their
// fixed costs (dispatch and one global round trip each), not by work; here one
// work-group loads its rows and the weights in one round trip, keeps every
// intermediate in LDS, and writes the sublayer's output rows -- in (B, S, T)
// order for the spatial half, which performs the Switch on the way out.
// Arithmetic is fp32 (products on v_mfma_f32_16x16x4_f32 or FMAs, expf), the softmax
// two-pass with the exact row maximum.
//   Bound by latency: one group is a few microseconds on one CU.  The two
// projections run on the matrix instruction, a 16 x 16 tile per wave, because with one
// thread per output column their LDS reads (five 16-byte reads per 16 FMAs) took
// half the kernel's time; a (head, query) task of the attention is shared by 4
// lanes, each with every fourth key, because at these sizes there are fewer tasks than
// threads.  Tiny chain (4 groups of 16, then 16 of 4, C = 64): 12.0 + 7.9 -> 9.2 + 7.3 us
// in a kernel trace; 16 groups of 64, then 64 of 16: 70 -> 39 us a call, 14 of 40 and 80 of
// 7: 30.5 -> 23.7.
#include <math.h>

#include "dsp_internal.h"

namespace dsp {
namespace {

constexpr int CH_CMAX = 64, CH_LMAX = 64;
constexpr int CH_SPLIT = 4;  // lanes per (head, query) task
// LDS floats for the largest shape: rows (pitch C + 4), W_qkv (pitch C + 4), qkv (pitch 3C + 4)
constexpr int CH_LDS = CH_LMAX * (CH_CMAX + 4) + 3 * CH_CMAX * (CH_CMAX + 4) + CH_LMAX * (3 * CH_CMAX + 4);

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;

struct ChainParams {
  const float* x;  // group g's row r at x + (g * L + r) * C
  const float* wqkv;  // [3C][C], stored [out][in]
  const float* bqkv;  // [3C] or null
  const float* wo;    // [C][C]
  const float* bo;    // [C] or null
  float* y;           // row rs.map(g * L + r); may alias x (each group reads its rows before writing them)
                      // x, y and the weights 16-byte aligned
  int L, C, H, D;
  float scale;
  RowSwap rs;
};

// out[m][n] = b[n] + sum_k a[m][k] w[n][k] for all m < M, n < N, in 16 x 16 tiles, one
// wave each: lane (i, c) = (lane % 16, lane / 16) reads 4 reduction indices 16 j + 4 c
// of row i of both operands at a time, which feed 4 MFMAs.  k16: the reduction in
// steps of 16, zero-padded in both operands.  Tiles past M or N read LDS that holds
// something else, into outputs that are not stored.
template <typename Store>
__device__ __forceinline__ void chain_gemm(const float* a, const float* w, int pitch, int k16, const float* bias, int M,
                                           int N, int n_waves, Store store) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = lane & 15, c = lane >> 4;
  const int nt = (N + 15) / 16, tiles = ((M + 15) / 16) * nt;
  for (int tile = wave; tile < tiles; tile += n_waves) {
    const int m0 = tile / nt * 16, n0 = tile % nt * 16;
    const int n = n0 + i;
    const float b = bias && n < N ? bias[n] : 0.0f;
    const float* ar = a + (m0 + i) * pitch + 4 * c;
    const float* wr = w + (n0 + i) * pitch + 4 * c;
    floatx4 acc = {b, b, b, b};
    for (int j = 0; j < k16; ++j) {
      const float4 x = *reinterpret_cast<const float4*>(ar + 16 * j), y = *reinterpret_cast<const float4*>(wr + 16 * j);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x, y.x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x.y, y.y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x.z, y.z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x.w, y.w, acc, 0, 0, 0);
    }
    // the lane holds rows m0 + 4 c + {0..3} of column n
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (m0 + 4 * c + r < M && n < N) store(m0 + 4 * c + r, n, acc[r]);
  }
}

// NTH threads: 1024 for head widths up to 32 (more waves for the two GEMMs' tiles
// and more tasks at once; the attention's per-thread registers still fit), 256 for 64
template <int DT, int NTH>
__global__ __launch_bounds__(NTH) void chain_sublayer_f32_kernel(ChainParams p) {
  const int L = p.L, C = p.C, H = p.H;
  constexpr int D = DT;
  constexpr int CH_NT = NTH;
  const int C3 = 3 * C;
  const int k16 = (C + 15) / 16;
  const int WP = 16 * k16 + 4;  // pitch of the rows and the weights (floats): float4 rows
  const int QP = C3 + 4;        // qkv row pitch: float4 rows
  __shared__ __attribute__((aligned(16))) float smem[CH_LDS];
  float* xs = smem;                 // [L][WP]: the input rows, later the attention output
  float* ws = xs + L * WP;          // [3C][WP]: W_qkv, later W_o
  float* qs = ws + C3 * WP;         // [L][QP]: q | k | v
  const int t = threadIdx.x;
  const int64_t row0 = (int64_t)blockIdx.x * L;

  // ---- one round trip: every load of the group's rows, W_qkv and W_o is
  // issued before any is used (float4 chunks; rows are multiples of 4 floats)
  constexpr int X4 = CH_LMAX * CH_CMAX / 4 / CH_NT, WQ4 = 3 * CH_CMAX * CH_CMAX / 4 / CH_NT,
                WO4 = CH_CMAX * CH_CMAX / 4 / CH_NT;
  // chunks past the end re-read the last one (always in bounds, so every
  // load is one unconditional 16-byte load); the stores below skip them
  const int nx = L * C, nq = C3 * C, no = C * C;
  float4 xr[X4], wq[WQ4], wo4[WO4];
#pragma unroll
  for (int i = 0; i < X4; ++i)
    xr[i] = *reinterpret_cast<const float4*>(p.x + row0 * C + min(4 * (t + i * CH_NT), nx - 4));
#pragma unroll
  for (int i = 0; i < WQ4; ++i)
    wq[i] = *reinterpret_cast<const float4*>(p.wqkv + min(4 * (t + i * CH_NT), nq - 4));
#pragma unroll
  for (int i = 0; i < WO4; ++i)
    wo4[i] = *reinterpret_cast<const float4*>(p.wo + min(4 * (t + i * CH_NT), no - 4));
  // chunk at element e (4 floats of one row) of a matrix into its LDS row e / C
  auto put = [&](float* base, int e, float4 v) { *reinterpret_cast<float4*>(base + (e / C) * WP + e % C) = v; };
  // the reduction's padding, C % 16 columns of zeros in the rows and the weights
  // (W_o takes rows of W_qkv, whose padding it keeps)
  if (C % 16)
    for (int r = t; r < L + C3; r += CH_NT)
      for (int c = C; c < 16 * k16; ++c) xs[r * WP + c] = 0.0f;
#pragma unroll
  for (int i = 0; i < X4; ++i) {
    const int e = 4 * (t + i * CH_NT);
    if (e < nx) put(xs, e, xr[i]);
  }
#pragma unroll
  for (int i = 0; i < WQ4; ++i) {
    const int e = 4 * (t + i * CH_NT);
    if (e < nq) put(ws, e, wq[i]);
  }
  __syncthreads();

  // ---- qkv = x W_qkv + b_qkv
  chain_gemm(xs, ws, WP, k16, p.bqkv, L, C3, CH_NT / 64, [&](int m, int n, float v) { qs[m * QP + n] = v; });
  __syncthreads();

  // ---- W_o into LDS (the W_qkv rows are no longer read)
#pragma unroll
  for (int i = 0; i < WO4; ++i) {
    const int e = 4 * (t + i * CH_NT);
    if (e < no) put(ws, e, wo4[i]);
  }
  // ---- attention per (head, query) task: scores against the L keys, exact row
  // maximum, exp, row sum, probability-weighted values; output into xs.  CH_SPLIT
  // neighbouring lanes share a task, lane `part` with keys part, part + CH_SPLIT, ..
  // (every lane of a wave runs the same number of rounds, so the exchanges see
  // all of a task's lanes)
  const int part = t % CH_SPLIT;
  for (int t0 = 0; t0 < H * L * CH_SPLIT; t0 += CH_NT) {
    const bool live = t0 + t < H * L * CH_SPLIT;
    const int task = live ? (t0 + t) / CH_SPLIT : 0;
    const int h = task / L, i = task - h * L;
    float qr[D];
#pragma unroll
    for (int d = 0; d < D; d += 4) {
      const float4 v = *reinterpret_cast<const float4*>(qs + i * QP + h * D + d);
      qr[d] = v.x; qr[d + 1] = v.y; qr[d + 2] = v.z; qr[d + 3] = v.w;
    }
    // the scores are recomputed in the second pass rather than kept: a loop
    // over the keys instead of a register array unrolled to the largest L
    // keeps the code small (a short kernel run once pays for every
    // instruction-cache line it touches)
    auto score = [&](int j) {
      const float* kr = qs + j * QP + C + h * D;
      float acc = 0.0f;
#pragma unroll
      for (int d = 0; d < D; d += 4) {
        const float4 v = *reinterpret_cast<const float4*>(kr + d);
        acc = fmaf(qr[d], v.x, acc);
        acc = fmaf(qr[d + 1], v.y, acc);
        acc = fmaf(qr[d + 2], v.z, acc);
        acc = fmaf(qr[d + 3], v.w, acc);
      }
      return acc * p.scale;
    };
    float mx = -INFINITY;
#pragma unroll 2
    for (int j = part; j < L; j += CH_SPLIT) mx = fmaxf(mx, score(j));
#pragma unroll
    for (int o = 1; o < CH_SPLIT; o *= 2) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    float l = 0.0f;
    float o[D];
#pragma unroll
    for (int d = 0; d < D; ++d) o[d] = 0.0f;
#pragma unroll 2
    for (int j = part; j < L; j += CH_SPLIT) {
      const float e = expf(score(j) - mx);
      l += e;
      const float* vr = qs + j * QP + 2 * C + h * D;
#pragma unroll
      for (int d = 0; d < D; d += 4) {
        const float4 v = *reinterpret_cast<const float4*>(vr + d);
        o[d] = fmaf(e, v.x, o[d]);
        o[d + 1] = fmaf(e, v.y, o[d + 1]);
        o[d + 2] = fmaf(e, v.z, o[d + 2]);
        o[d + 3] = fmaf(e, v.w, o[d + 3]);
      }
    }
#pragma unroll
    for (int x = 1; x < CH_SPLIT; x *= 2) {
      l += __shfl_xor(l, x, 64);
#pragma unroll
      for (int d = 0; d < D; ++d) o[d] += __shfl_xor(o[d], x, 64);
    }
    const float inv = 1.0f / l;
    if (live) {
#pragma unroll
      for (int d = 0; d < D; d += 4)
        if ((d / 4) % CH_SPLIT == part)
          *reinterpret_cast<float4*>(xs + i * WP + h * D + d) =
              make_float4(o[d] * inv, o[d + 1] * inv, o[d + 2] * inv, o[d + 3] * inv);
    }
  }
  __syncthreads();

  // ---- out = o W_o + b_o, rows written at rs.map(global row)
  {
    const RowSwap rs = p.rs;
    float* const y = p.y;
    chain_gemm(xs, ws, WP, k16, p.bo, L, C, CH_NT / 64,
               [=](int m, int n, float v) { y[rs.map((int)(row0 + m)) * C + n] = v; });
  }
}

}  // namespace

bool chain_sublayer_f32_fits(int64_t L, int C, int H) {
  // float4 rows of x, q, k, v; head widths with an instance of the kernel
  if (L < 1 || L > CH_LMAX || C < 4 || C > CH_CMAX || H < 1 || C % H) return false;
  const int D = C / H;
  return D == 8 || D == 16 || D == 32 || D == 64;
}

int launch_chain_sublayer_f32(const float* x, const float* wqkv, const float* bqkv, const float* wo, const float* bo,
                              float* y, int64_t groups, int L, int C, int H, float scale, RowSwap rs, hipStream_t s) {
  if (groups == 0) return DSP_OK;
  if (!chain_sublayer_f32_fits(L, C, H) || groups >= (int64_t(1) << 31) || groups * L >= (int64_t(1) << 31))
    return DSP_ERR_SHAPE;
  ChainParams p;
  p.x = x;
  p.wqkv = wqkv;
  p.bqkv = bqkv;
  p.wo = wo;
  p.bo = bo;
  p.y = y;
  p.L = L;
  p.C = C;
  p.H = H;
  p.D = C / H;
  p.scale = scale;
  p.rs = rs;
  switch (p.D) {
    case 8: hipLaunchKernelGGL((chain_sublayer_f32_kernel<8, 1024>), dim3((uint32_t)groups), dim3(1024), 0, s, p); break;
    case 16: hipLaunchKernelGGL((chain_sublayer_f32_kernel<16, 1024>), dim3((uint32_t)groups), dim3(1024), 0, s, p); break;
    case 32: hipLaunchKernelGGL((chain_sublayer_f32_kernel<32, 1024>), dim3((uint32_t)groups), dim3(1024), 0, s, p); break;
    case 64: hipLaunchKernelGGL((chain_sublayer_f32_kernel<64, 256>), dim3((uint32_t)groups), dim3(256), 0, s, p); break;
    default: return DSP_ERR_SHAPE;
  }
  return last_launch_status();
}

}  // namespace dsp
