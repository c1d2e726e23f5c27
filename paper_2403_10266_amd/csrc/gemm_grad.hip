// Gradient GEMMs of the block's linear maps (the backward of Eq. 1's W^O, the
// Q/K/V projections and Eq. 5's W_1, W_2).  With y = x W^T (W stored [out][in],
// as in the forward), the gradients are
//   dx = dy W          -- [tokens, in]  = [tokens, out] x [out, in]
//   dW = dy^T x        -- [out, in]     = [out, tokens] x [tokens, in]
// so one operand, or both, has its reduction index strided in memory.  (The block's
// bf16 backward transposes its weights once and takes dx through the forward's
// tiles where it can; the dx kernel here serves dsp_linear_bwd_data and widths that
// are not multiples of 64.)
//
// Design for gfx950, on v_mfma_f32_32x32x16_bf16 like the forward GEMM, B rows on the
// MFMA M side so a lane owns one output row:
//  * dx: 256 x 128 tiles, 4 waves of 128 x 64, 64-wide k slices through LDS, the next
//    slice prefetched into registers.  dy keeps the forward's LDS layout [rows][k]
//    (144-byte rows); W is copied as it lies, [k][rows], and its fragments are
//    read with ds_read_b64_tr_b16, which gives each lane 8 k values of one row in
//    the order {4g..4g+3, 8+4g..8+4g+3} of a 16-k step.  dy is then read in the same
//    k order (two 8-byte reads), so the two sides of every MFMA agree.
//    Epilogues: fp32 output; bf16 output; the GELU / ReLU backward, out =
//    acc * act'(u) with u the saved pre-activation (bf16), rounded to bf16.
//  * dW: gemm_grad_tt_dma_kernel below.  The reduction over all tokens is cut into
//    splits, one per grid z; each writes fp32 partial sums to its own slab of a
//    workspace and a second kernel adds the slabs in a fixed order (no atomics:
//    deterministic).
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "attn_bf16_common.h"
#include "direct_lds.h"
#include "dsp_internal.h"

namespace dsp {
namespace {

constexpr int GBM = 256, GBN = 128, GBK = 64;
constexpr int GNTHR = 256;
constexpr int NPITCH = GBK + 8;   // natural tiles: 144-byte rows

template <int ROWS>
struct TPitch {
  static constexpr int P = ROWS + 8;  // transposed tiles: an odd multiple of 16 bytes
};

// d/du (u Phi(u)) = Phi(u) + u phi(u), with erf by Abramowitz and Stegun
// 7.1.26 (|error| <= 1.5e-7).  The exp(-z^2) of erf's tail at z = u / sqrt(2)
// is exp(-u^2 / 2) = sqrt(2 pi) phi(u): one exponential serves both terms.
__device__ __forceinline__ float gelu_grad(float u) {
  const float z = u * 0.70710678118654752f;
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, fabsf(z), 1.0f));
  float poly = fmaf(1.061405429f, t, -1.453152027f);
  poly = fmaf(poly, t, 1.421413741f);
  poly = fmaf(poly, t, -0.284496736f);
  poly = fmaf(poly, t, 0.254829592f);
  poly *= t;
  const float e = __builtin_amdgcn_exp2f(-z * z * 1.4426950408889634f);
  const float erf = copysignf(1.0f - poly * e, z);
  return fmaf(0.5f, erf, 0.5f) + u * (0.3989422804014327f * e);
}

struct GradArgs {
  const bf16* a;
  const bf16* b;
  const bf16* aux;  // saved pre-activation for the activation backward epilogues
  void* out;        // [M][N] (or, with splits > 1, the fp32 workspace [splits][M][N])
  int64_t lda, ldb;
  int M, N, K, n_ntiles, n_tiles, k_per_split;
};

// One operand's tile of one k slice: global -> registers -> LDS, and its MFMA
// fragments.  ROWS = tile rows on the M or N side (256 or 128).
template <int ROWS, bool TRANS>
struct Operand {
  static constexpr int CHUNKS = ROWS * GBK / 8;    // 16-byte chunks per slice
  static constexpr int LOADS = CHUNKS / GNTHR;
  static constexpr int ELEMS = TRANS ? GBK * TPitch<ROWS>::P : ROWS * NPITCH;
  static_assert(CHUNKS % GNTHR == 0, "loader shape");

  const bf16* base;
  int64_t ld;
  int r0, rows_valid, k_total;
  u32x4 pre[LOADS];
  uint32_t off[LOADS];
  int lds_off[LOADS];
  bool col_ok[LOADS];

  __device__ void init(const bf16* p, int64_t ld_, int r0_, int rows_total, int k_total_) {
    base = p;
    ld = ld_;
    r0 = r0_;
    rows_valid = min(ROWS, rows_total - r0_);
    k_total = k_total_;
    const int t = threadIdx.x;
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      if (!TRANS) {
        // chunk (row t/8 + 32 i, k columns 8 (t % 8) .. + 7)
        const int row = (t >> 3) + 32 * i, kc = t & 7;
        off[i] = (uint32_t)row * (uint32_t)(ld * 2) + (uint32_t)kc * 16u;
        lds_off[i] = row * NPITCH + kc * 8;
        col_ok[i] = true;
      } else {
        // chunk (k row r, columns 8 c .. + 7), ROWS / 8 chunks per k row
        constexpr int CPR = ROWS / 8;
        const int c = t % CPR, r = t / CPR + (GNTHR / CPR) * i;
        off[i] = (uint32_t)r * (uint32_t)(ld * 2) + (uint32_t)c * 16u;
        lds_off[i] = r * TPitch<ROWS>::P + c * 8;
        col_ok[i] = 8 * c < rows_valid;
      }
    }
  }

  // loads the slice starting at reduction index k0 (rows / k past the end read zero)
  __device__ void load(int k0) {
    if (!TRANS) {
      const __amdgpu_buffer_rsrc_t rs =
          make_rsrc(base + (int64_t)r0 * ld, (uint32_t)max(rows_valid, 0) * (uint32_t)(ld * 2));
      const bool kin = k0 + 8 * (int)(threadIdx.x & 7) < k_total;
#pragma unroll
      for (int i = 0; i < LOADS; ++i)
        pre[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, kin ? off[i] + (uint32_t)k0 * 2u : 0xFFFFFFF0u, 0, 0);
    } else {
      const int krows = max(0, min(GBK, k_total - k0));
      const __amdgpu_buffer_rsrc_t rs =
          make_rsrc(base + (int64_t)k0 * ld + r0, (uint32_t)krows * (uint32_t)(ld * 2));
#pragma unroll
      for (int i = 0; i < LOADS; ++i)
        pre[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, col_ok[i] ? off[i] : 0xFFFFFFF0u, 0, 0);
    }
  }

  __device__ void store(bf16* lds) const {
#pragma unroll
    for (int i = 0; i < LOADS; ++i) *reinterpret_cast<u32x4*>(lds + lds_off[i]) = pre[i];
  }

  // fragment of tile rows rbase .. rbase + 31 for 16-k step ks: lane
  // (l32 + 32g) gets row rbase + l32 at k = 16 ks + {4g..4g+3, 8+4g..8+4g+3}
  __device__ static bf16x8 frag(const bf16* lds, int rbase, int ks, int lane) {
    const int l32 = lane & 31, g = lane >> 5;
    if (!TRANS) {
      const bf16* row = lds + (rbase + l32) * NPITCH + 16 * ks + 4 * g;
      const shortx4 lo = *reinterpret_cast<const shortx4*>(row);
      const shortx4 hi = *reinterpret_cast<const shortx4*>(row + 8);
      return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    } else {
      constexpr int P = TPitch<ROWS>::P;
      const int j16 = lane & 15, mbase = 16 * ((lane >> 4) & 1);
      const int row = 16 * ks + 4 * g + (j16 >> 2);
      const int col = rbase + mbase + 4 * (j16 & 3);
      const shortx4 lo = lds_read_tr(lds + row * P + col);
      const shortx4 hi = lds_read_tr(lds + (row + 8) * P + col);
      return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  }
};

template <int EPI>
__global__ __launch_bounds__(GNTHR, 2) void gemm_grad_kernel(GradArgs p) {
  using OA = Operand<GBM, false>;
  using OB = Operand<GBN, true>;
  __shared__ __attribute__((aligned(16))) bf16 As[OA::ELEMS];
  __shared__ __attribute__((aligned(16))) bf16 Bs[OB::ELEMS];

  // XCD-aware order (tiles m-major, n fastest; each XCD a contiguous range)
  uint32_t bid = blockIdx.x;
  if ((p.n_tiles & 7) == 0) bid = (bid & 7u) * ((uint32_t)p.n_tiles >> 3) + (bid >> 3);
  const int mt = bid / p.n_ntiles;
  const int nt = bid - mt * p.n_ntiles;
  const int m0 = mt * GBM, n0 = nt * GBN;

  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wm = wave & 1, wn = wave >> 1;
  const int l32 = lane & 31, g = lane >> 5;

  OA a;
  OB b;
  a.init(p.a, p.lda, m0, p.M, p.K);
  b.init(p.b, p.ldb, n0, p.N, p.K);

  floatx16 acc[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  const int nk = (p.K + GBK - 1) / GBK;
  if (nk > 0) {
    a.load(0);
    b.load(0);
    a.store(As);
    b.store(Bs);
  }
  __syncthreads();
  for (int it = 0; it < nk; ++it) {
    const bool more = it + 1 < nk;
    if (more) {
      a.load((it + 1) * GBK);
      b.load((it + 1) * GBK);
    }
#pragma unroll
    for (int ks = 0; ks < GBK / 16; ++ks) {
      bf16x8 af[4], bfr[2];
#pragma unroll
      for (int j = 0; j < 4; ++j) af[j] = OA::frag(As, wm * 128 + 32 * j, ks, lane);
#pragma unroll
      for (int i = 0; i < 2; ++i) bfr[i] = OB::frag(Bs, wn * 64 + 32 * i, ks, lane);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[i], af[j], acc[i][j], 0, 0, 0);
    }
    if (more) {
      __syncthreads();
      a.store(As);
      b.store(Bs);
      __syncthreads();
    }
  }

  // epilogue: lane owns row m = .. + l32 and columns n = .. + 8 r4 + 4g + {0..3}
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int m = m0 + wm * 128 + 32 * j + l32;
    if (m >= p.M) continue;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const int n = n0 + wn * 64 + 32 * i + 8 * r4 + 4 * g;
        if (n >= p.N) continue;   // N % 4 == 0: the group of 4 is whole
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[i][j][4 * r4 + e];
        const int64_t off = (int64_t)m * p.N + n;
        if (EPI == DSP_GRAD_EPI_F32) {
          *reinterpret_cast<float4*>(static_cast<float*>(p.out) + off) = make_float4(v[0], v[1], v[2], v[3]);
        } else {
          if (EPI == DSP_GRAD_EPI_GELU_BWD || EPI == DSP_GRAD_EPI_RELU_BWD) {
            const uint2 uw = *reinterpret_cast<const uint2*>(p.aux + off);
            const bf16x2 u01 = __builtin_bit_cast(bf16x2, uw.x), u23 = __builtin_bit_cast(bf16x2, uw.y);
            const float u[4] = {(float)u01[0], (float)u01[1], (float)u23[0], (float)u23[1]};
#pragma unroll
            for (int e = 0; e < 4; ++e)
              v[e] *= EPI == DSP_GRAD_EPI_GELU_BWD ? gelu_grad(u[e]) : (u[e] > 0.0f ? 1.0f : 0.0f);
          }
          bf16x2 lo = {(bf16)v[0], (bf16)v[1]};
          bf16x2 hi = {(bf16)v[2], (bf16)v[3]};
          uint2 w;
          w.x = __builtin_bit_cast(uint32_t, lo);
          w.y = __builtin_bit_cast(uint32_t, hi);
          *reinterpret_cast<uint2*>(static_cast<bf16*>(p.out) + off) = w;
        }
      }
  }
}

// out[i] = sum over z of ws[z][i], z in order (deterministic)
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float4* __restrict__ ws, float4* out,
                                                            int64_t n4, int splits) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n4) return;
  float4 s = ws[i];
  for (int z = 1; z < splits; ++z) {
    const float4 v = ws[(int64_t)z * n4 + i];
    s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
  }
  out[i] = s;
}

// db[n] = sum over rows m of dy[m][n] (fp32), the bias gradient.  A pass over dy,
// bound by memory; its problem is parallelism, since few columns meet many rows
// and the caller lends no scratch for partial sums.  So one work-group of 1024
// threads takes G 16-byte chunks (bf16: 8 columns each; fp32: one column per
// thread, as rows need no alignment there) of every row: G threads on a row,
// 1024 / G rows at a time, eight loads of each thread in flight.  The rows' sums
// then meet in a fixed tree (lanes, then waves in order): deterministic, and a
// shorter chain of fp32 adds than a walk down the column.
//   13600 bf16 rows of 1152 / 3456 / 4608 columns: 22 / 24 / 31 us (1.4 / 3.9 / 4.0 TB/s),
// where one thread walking down 4 columns (two to five work-groups on the chip, one
// load in flight each) took 3750 / 3720 / 3570 us; 2048 fp32 rows 470 -> 5-11 us.
constexpr int CS_THREADS = 1024, CS_UNROLL = 8;

template <bool BF, int G>
__global__ __launch_bounds__(CS_THREADS) void colsum_kernel(const void* __restrict__ dyp, float* db, int64_t M, int N,
                                                            int first) {  // this launch's first work-group
  constexpr int V = BF ? 8 : 1;              // columns per thread
  constexpr int R = CS_THREADS / G;          // rows per step
  constexpr int W = CS_THREADS / 64;
  __shared__ float part[W][G * V];
  // neighbouring column groups share cache lines: give each XCD a contiguous range
  const uint32_t nb = gridDim.x;
  uint32_t bid = blockIdx.x;
  if ((nb & 7u) == 0) bid = (bid & 7u) * (nb >> 3) + (bid >> 3);
  bid += (uint32_t)first;
  const int c = threadIdx.x % G, r = threadIdx.x / G;
  const int n = ((int)bid * G + c) * V;
  float s[V];
#pragma unroll
  for (int i = 0; i < V; ++i) s[i] = 0.0f;
  if (n < N) {  // bf16: N is a multiple of 8, a chunk is whole
    const auto add = [&](int64_t m) {
      if constexpr (BF) {
        const u32x4 w = *reinterpret_cast<const u32x4*>(static_cast<const bf16*>(dyp) + m * N + n);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          s[2 * i] += __uint_as_float(w[i] << 16);
          s[2 * i + 1] += __uint_as_float(w[i] & 0xFFFF0000u);
        }
      } else {
        s[0] += static_cast<const float*>(dyp)[m * N + n];
      }
    };
    int64_t m = r;
    for (; m + (CS_UNROLL - 1) * R < M; m += CS_UNROLL * R) {
#pragma unroll
      for (int u = 0; u < CS_UNROLL; ++u) add(m + u * R);
    }
    for (; m < M; m += R) add(m);
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < V; ++i) {
#pragma unroll
    for (int o = 32; o >= G; o >>= 1) s[i] += __shfl_xor(s[i], o, 64);
    if (lane < G) part[wave][lane * V + i] = s[i];
  }
  __syncthreads();
  if (threadIdx.x < G * V) {
    float t = 0.0f;
#pragma unroll
    for (int w = 0; w < W; ++w) t += part[w][threadIdx.x];
    const int col = (int)bid * G * V + (int)threadIdx.x;
    if (col < N) db[col] = t;
  }
}

// A few rows: one thread per 16-byte chunk (bf16) or column (fp32).  The tree of a
// 1024-thread work-group takes longer than the rows do (8 fp32 rows of 64 columns with
// their weight gradient 6.6 against 7.8 us; 16 bf16 rows of 8192 24.2 against 21.0).
constexpr int kFewRows = 8;
template <bool BF>
__global__ __launch_bounds__(256) void colsum_few_kernel(const void* __restrict__ dyp, float* db, int M, int N) {
  constexpr int V = BF ? 8 : 1;
  const int64_t n = ((int64_t)blockIdx.x * 256 + threadIdx.x) * V;
  if (n >= N) return;
  float s[V] = {};
  for (int m = 0; m < M; ++m) {
    if constexpr (BF) {  // N is a multiple of 8
      const u32x4 w = *reinterpret_cast<const u32x4*>(static_cast<const bf16*>(dyp) + (int64_t)m * N + n);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s[2 * i] += __uint_as_float(w[i] << 16);
        s[2 * i + 1] += __uint_as_float(w[i] & 0xFFFF0000u);
      }
    } else {
      s[0] += static_cast<const float*>(dyp)[(int64_t)m * N + n];
    }
  }
#pragma unroll
  for (int i = 0; i < V; ++i) db[n + i] = s[i];
}

// ---------------------------------------------------------------------------
// Weight gradient: out[M][N] = sum over k of a[k][m] b[k][n] (both operands stored
// with the reduction index as rows: dW = dy^T x), fp32, the reduction split over
// blockIdx.z into fp32 partials.  Tiles of 64 TM x 64 TN (4 waves of 32 TM x 32 TN): the
// k rows of both operands go from memory straight into a ring of NS LDS buffers of 64
// rows, and OCC work-groups share a CU (see gemm_bf16_dma_kernel in gemm.hip, whose
// schedule this is).  Fragments are read with ds_read_b64_tr_b16 (k order
// {4g..4g+3, 8+4g..8+4g+3} on both sides).  Rows lie unpadded; the 16-byte chunk p of
// row r holds columns of logical chunk p ^ f(r), where f spreads the four consecutive
// rows of a transposed read over the banks: 64-byte groups are exchanged by the row's
// two low bits where a row is a multiple of 256 bytes, by its second bit where it is
// 128 off one.  Columns past the end re-read the last whole chunk (they only enter
// outputs that are not stored); a slice that ends before 64 rows is loaded through
// registers, zero-filled, after the whole ones.
//   At 13600 tokens the matrix cores are busy 46-50% of the time (3456 and 4608 x 1152, waves
// wait 16%, LDS serves fragment reads 20%): no one unit is full.  us: 3456 x 1152
// 135 -> 114, 4608 x 1152 181 -> 151, 1152 x 4608 204 -> 152, 1152 x 1152 70 -> 53 (with the
// partials' reduction; before: register-staged 256-wide tiles, one work-group per CU);
// 2000 tokens, 1152 x 1152: 50 -> 17 (256 x 128 tiles before).
template <int TM, int TN, int NS, int OCC>
__global__ __launch_bounds__(GNTHR, OCC) void gemm_grad_tt_dma_kernel(GradArgs p) {
  constexpr int BMT = 64 * TM, BNT = 64 * TN;
  constexpr int CA = BMT / 8, CB = BNT / 8;   // 16-byte chunks per k row
  constexpr int STAGE = GBK * (BMT + BNT);    // elements of one slice of both operands
  constexpr int NP = TM >= 2 ? 2 : 1, RPP = BMT / NP, HR = RPP / 2, BPP = TM / NP;
  constexpr int SPF = BNT + 4;                // staged output row pitch (fp32)
  constexpr int LDS_ELEMS = NS * STAGE > RPP * SPF * 2 ? NS * STAGE : RPP * SPF * 2;
  __shared__ __attribute__((aligned(1024))) bf16 lds[LDS_ELEMS];

  // tile order: contiguous ranges per XCD, m fastest within groups of 1024 rows
  uint32_t bid = blockIdx.x;
  {
    const uint32_t per = (uint32_t)p.n_tiles >> 3, extra = (uint32_t)p.n_tiles & 7u, xcd = bid & 7u;
    bid = xcd * per + min(xcd, extra) + (bid >> 3);
  }
  constexpr int GROUP = 1024 / BMT;
  const int n_mt = p.n_tiles / p.n_ntiles;
  const int per_group = GROUP * p.n_ntiles;
  const int grp = (int)bid / per_group;
  const int first_m = grp * GROUP;
  const int gm = min(GROUP, n_mt - first_m);
  const int rem = (int)bid - grp * per_group;
  const int m0 = (first_m + rem % gm) * BMT, n0 = (rem / gm) * BNT;
  const int kb = blockIdx.z * p.k_per_split;
  const int ke = min(p.K, kb + p.k_per_split);

  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wm = wave & 1, wn = wave >> 1;
  const int l32 = lane & 31, g = lane >> 5;
  const int j16 = lane & 15, mbase = 16 * ((lane >> 4) & 1);

  constexpr int A_LOADS = GBK * CA / GNTHR, B_LOADS = GBK * CB / GNTHR, NL = A_LOADS + B_LOADS;
  auto swz = [](int chunks, int row) { return chunks % 16 == 0 ? (row & 3) * 4 : ((row >> 1) & 1) * 4; };
  // chunk e of an operand's slice: k row e / C, logical chunk (e % C) ^ f(row)
  auto row_of = [&](int i) { return ((int)threadIdx.x + GNTHR * (i < A_LOADS ? i : i - A_LOADS)) / (i < A_LOADS ? CA : CB); };
  auto col_of = [&](int i) {  // its logical chunk, clamped to the operand's columns
    const int C = i < A_LOADS ? CA : CB, e = (int)threadIdx.x + GNTHR * (i < A_LOADS ? i : i - A_LOADS);
    const int last = (i < A_LOADS ? p.M - m0 : p.N - n0) / 8 - 1;
    return min((e % C) ^ swz(C, e / C), last);
  };
  const uint32_t a_row = (uint32_t)(p.lda * 2), b_row = (uint32_t)(p.ldb * 2);
  uint32_t goff[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i)
    goff[i] = (uint32_t)row_of(i) * (i < A_LOADS ? a_row : b_row) + (uint32_t)col_of(i) * 16u;
  // resources over 64 k rows from the range's first (the last row ends with its columns)
  const u32x4 ra0 = dma_rsrc(p.a + (int64_t)kb * p.lda + m0, GBK * a_row - (uint32_t)m0 * 2u);
  const u32x4 rb0 = dma_rsrc(p.b + (int64_t)kb * p.ldb + n0, GBK * b_row - (uint32_t)n0 * 2u);
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) bf16*)lds + (uint32_t)wave * 1024u);
  auto dma = [&](int i, int kt, int buf) {
    const uint32_t at = lds0 + (uint32_t)buf * (STAGE * 2) +
                        (i < A_LOADS ? i * (GNTHR * 16) : GBK * BMT * 2 + (i - A_LOADS) * (GNTHR * 16));
    const uint64_t add = (uint64_t)kt * GBK * (i < A_LOADS ? a_row : b_row);
    dma_b128(dma_advance(i < A_LOADS ? ra0 : rb0, add), goff[i], 0u, at);
  };

  floatx16 acc[TN][TM];
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.0f;
  // fragment of the 32 columns of block `blk`: k rows 16 ks + 4 g + (j16 >> 2) and 8 on
  auto frag = [&](const bf16* t, int C, int blk, int ks) {
    const int q = j16 >> 2, x = C % 16 == 0 ? q : (q >> 1);
    const bf16* at = t + (16 * ks + 4 * g + q) * (8 * C) + ((blk ^ x) * 32 + mbase + 4 * (j16 & 3));
    const shortx4 lo = lds_read_tr(at), hi = lds_read_tr(at + 64 * C);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  bf16x8 af[2][TM], wf[2][TN];
  auto fread = [&](int slot, int buf, int ks) {
    const bf16* As = lds + buf * STAGE;
    const bf16* Bs = As + GBK * BMT;
#pragma unroll
    for (int b = 0; b < TM; ++b) af[slot][b] = frag(As, CA, wm * TM + b, ks);
#pragma unroll
    for (int a = 0; a < TN; ++a) wf[slot][a] = frag(Bs, CB, wn * TN + a, ks);
  };
  // one slice, as in gemm_bf16_dma_kernel
  auto slice = [&](int kt, int buf, auto more_c, auto left_c, auto ld_c) {
    constexpr bool MORE = decltype(more_c)::value, LD = decltype(ld_c)::value;
    constexpr int LEFT = decltype(left_c)::value, NMF = TM * TN;
    const int nbuf = buf + 1 == NS ? 0 : buf + 1;
#pragma unroll
    for (int ks = 0; ks < GBK / 16; ++ks) {
      const int cur = ks & 1;
      if (ks + 1 < GBK / 16) {
        fread(cur ^ 1, buf, ks + 1);
      } else if (MORE) {
        wait_barrier<LEFT * NL>();
        fread(cur ^ 1, nbuf, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < NMF; ++j) {
        const int a = j / TM, bb = j % TM;
        acc[a][bb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[cur][a], af[cur][bb], acc[a][bb], 0, 0, 0);
        if (LD && ks + 1 == GBK / 16) {
#pragma unroll
          for (int i = j * NL / NMF; i < (j + 1) * NL / NMF; ++i) dma(i, kt + NS, buf);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  using yes = std::true_type;
  using no = std::false_type;
  using zero = std::integral_constant<int, 0>;
  const int nk = max(0, ke - kb) / GBK;  // whole slices
  if (nk > 0) {
    for (int t = 0; t < min(NS, nk); ++t)
#pragma unroll
      for (int i = 0; i < NL; ++i) dma(i, t, t);
    if (nk >= NS)
      wait_barrier<(NS - 1) * NL>();
    else
      wait_barrier<0>();
    fread(0, 0, 0);
    int kt = 0, buf = 0;
    for (; kt + NS < nk; ++kt) {
      slice(kt, buf, yes{}, std::integral_constant<int, NS - 2>{}, yes{});
      buf = buf + 1 == NS ? 0 : buf + 1;
    }
    for (; kt + 1 < nk; ++kt) {
      slice(kt, buf, yes{}, zero{}, no{});
      buf = buf + 1 == NS ? 0 : buf + 1;
    }
    slice(kt, buf, no{}, zero{}, no{});
  }
  const int tail = max(0, ke - kb) - nk * GBK;
  if (tail > 0) {
    const int k0 = kb + nk * GBK;
    const __amdgpu_buffer_rsrc_t ta = make_rsrc(p.a + (int64_t)k0 * p.lda + m0, (uint32_t)tail * a_row - (uint32_t)m0 * 2u);
    const __amdgpu_buffer_rsrc_t tb = make_rsrc(p.b + (int64_t)k0 * p.ldb + n0, (uint32_t)tail * b_row - (uint32_t)n0 * 2u);
    u32x4 v[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i)
      v[i] = __builtin_amdgcn_raw_buffer_load_b128(i < A_LOADS ? ta : tb, row_of(i) < tail ? goff[i] : 0xFFFFFFF0u, 0, 0);
    __syncthreads();  // every wave has read its last fragments
#pragma unroll
    for (int i = 0; i < NL; ++i)
      *reinterpret_cast<u32x4*>(lds + (i < A_LOADS ? i * GNTHR * 8 : GBK * BMT + (i - A_LOADS) * GNTHR * 8) +
                                threadIdx.x * 8) = v[i];
    __syncthreads();
    fread(0, 0, 0);
    slice(0, 0, no{}, zero{}, no{});
  }

  // fp32 partial (or the result, unsplit), staged through LDS in NP passes (rows
  // HR pass + [0, HR) of each wave row half) and stored as whole 16-byte row chunks
  float* out = static_cast<float*>(p.out) + (int64_t)blockIdx.z * p.M * p.N;
  constexpr int CPR = BNT / 4, PER = RPP * CPR / GNTHR;
  float* sf = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int pass = 0; pass < NP; ++pass) {
    __syncthreads();  // pass 0: the last fragments are read; pass 1: pass 0's rows are read
#pragma unroll
    for (int h = 0; h < BPP; ++h)
#pragma unroll
      for (int a = 0; a < TN; ++a)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          const floatx16& t = acc[a][BPP * pass + h];
          *reinterpret_cast<float4*>(sf + (wm * HR + 32 * h + l32) * SPF + wn * TN * 32 + 32 * a + 8 * r4 + 4 * g) =
              make_float4(t[4 * r4], t[4 * r4 + 1], t[4 * r4 + 2], t[4 * r4 + 3]);
        }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int c = (int)threadIdx.x + GNTHR * q;
      const int sr = c / CPR, cc = c % CPR;
      const int m = m0 + (sr / HR) * (BMT / 2) + HR * pass + sr % HR, n = n0 + 4 * cc;
      if (m < p.M && n < p.N)
        *reinterpret_cast<float4*>(out + (int64_t)m * p.N + n) =
            *reinterpret_cast<const float4*>(sf + sr * SPF + 4 * cc);
    }
  }
}

// Tile shapes of the weight gradient and their times: a launch of `tiles` *
// splits work-groups takes full rounds of 256 * levels and one of the rest, with
// 1 .. levels of them per CU; a round with j per CU takes a[j - 1] + b[j - 1] * (64-row
// slices) microseconds, and each partial of the reduction a write and a read at
// about 4 TB/s each.  Estimates, not a fit: slopes scaled from the forward tiles (same
// schedule).  Against 61 measured calls of 15 us and more (1 to 32768 tokens, the linear
// maps of widths 1152 and 2048) they are off by 18% on average, 46% at most, always short:
// one round of few slices costs about 7 us more than they say.
struct GradTile {
  int tm, tn, levels;
  double a[3], b[3];
};
constexpr GradTile kGradTiles[5] = {{2, 3, 2, {4.0, 5.0}, {0.76, 1.30}},
                                    {2, 2, 2, {3.0, 4.0}, {0.62, 0.98}},
                                    {2, 2, 1, {4.0}, {0.53}},
                                    {1, 2, 3, {2.0, 2.5, 3.0}, {0.55, 0.62, 0.98}},
                                    {1, 1, 2, {2.0, 2.0}, {0.25, 0.42}}};

struct GradChoice {
  int tile, splits;
};
// the fastest tile shape and split count, of at most max_splits
GradChoice choose_grad(int64_t M, int64_t N, int64_t K, int max_splits) {
  GradChoice best = {-1, 1};
  double best_cost = 0.0;
  const int64_t slices = (K + GBK - 1) / GBK;
  for (int i = 0; i < 5; ++i) {
    const GradTile& t = kGradTiles[i];
    const int64_t tiles = ((M + 64 * t.tm - 1) / (64 * t.tm)) * ((N + 64 * t.tn - 1) / (64 * t.tn));
    for (int s = 1; s <= max_splits; ++s) {
      const int64_t per = (slices + s - 1) / s;
      if (s > 1 && per * (s - 1) >= slices) break;  // the last split would be empty
      const int64_t wgs = tiles * s, round = 256 * t.levels, rest = wgs % round;
      double cost = (double)(wgs / round) * (t.a[t.levels - 1] + t.b[t.levels - 1] * (double)per);
      if (rest) {
        const int j = (int)((rest + 255) / 256) - 1;
        cost += t.a[j] + t.b[j] * (double)per;
      }
      if (s > 1) cost += 3.0 + (double)s * (double)M * (double)N * 1e-6;
      if (best.tile < 0 || cost < best_cost) {
        best = {i, s};
        best_cost = cost;
      }
    }
  }
  return best;
}

int launch_reduce(const float* ws, void* out, int64_t n, int splits, hipStream_t s) {
  const int64_t n4 = n / 4;
  hipLaunchKernelGGL(splitk_reduce_kernel, dim3((uint32_t)((n4 + 255) / 256)), dim3(256), 0, s,
                     reinterpret_cast<const float4*>(ws), static_cast<float4*>(out), n4, splits);
  return last_launch_status();
}

int launch_grad_tt(GradArgs p, int max_splits, float* ws, hipStream_t s) {
  const GradChoice c = choose_grad(p.M, p.N, p.K, ws ? max_splits : 1);
  const GradTile& t = kGradTiles[c.tile];
  const int64_t n_nt = (p.N + 64 * t.tn - 1) / (64 * t.tn), tiles = ((p.M + 64 * t.tm - 1) / (64 * t.tm)) * n_nt;
  if (tiles >= (int64_t(1) << 31)) return DSP_ERR_SHAPE;
  p.n_ntiles = (int)n_nt;
  p.n_tiles = (int)tiles;
  p.k_per_split = ((p.K + GBK - 1) / GBK + c.splits - 1) / c.splits * GBK;
  void* out = p.out;
  if (c.splits > 1) p.out = ws;
  const dim3 grid((uint32_t)tiles, 1, (uint32_t)c.splits), block(GNTHR);
  switch (c.tile) {
    case 0: hipLaunchKernelGGL((gemm_grad_tt_dma_kernel<2, 3, 2, 2>), grid, block, 0, s, p); break;
    case 1: hipLaunchKernelGGL((gemm_grad_tt_dma_kernel<2, 2, 2, 2>), grid, block, 0, s, p); break;
    case 2: hipLaunchKernelGGL((gemm_grad_tt_dma_kernel<2, 2, 4, 1>), grid, block, 0, s, p); break;
    case 3: hipLaunchKernelGGL((gemm_grad_tt_dma_kernel<1, 2, 2, 3>), grid, block, 0, s, p); break;
    default: hipLaunchKernelGGL((gemm_grad_tt_dma_kernel<1, 1, 4, 2>), grid, block, 0, s, p); break;
  }
  const int st = last_launch_status();
  if (st != DSP_OK || c.splits == 1) return st;
  return launch_reduce(ws, out, (int64_t)p.M * p.N, c.splits, s);
}

template <int EPI>
int launch_grad(GradArgs p, hipStream_t s) {
  const int64_t n_mt = (p.M + GBM - 1) / GBM, n_nt = (p.N + GBN - 1) / GBN;
  const int64_t tiles = n_mt * n_nt;
  p.n_ntiles = (int)n_nt;
  p.n_tiles = (int)tiles;
  hipLaunchKernelGGL((gemm_grad_kernel<EPI>), dim3((uint32_t)tiles), dim3(GNTHR), 0, s, p);
  return last_launch_status();
}

// out = a + b (fp32); out may alias a or b
__global__ __launch_bounds__(256) void add_f32_kernel(const float* a, const float* b, float* out, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) out[i] = a[i] + b[i];
}

}  // namespace

int launch_add_f32(const float* a, const float* b, float* out, int64_t n, hipStream_t s) {
  if (n == 0) return DSP_OK;
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, 65536);
  hipLaunchKernelGGL(add_f32_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, a, b, out, n);
  return last_launch_status();
}

// Work-groups of 16 columns (one 64-byte piece of a row): 72 of them at 1152
// columns.
int launch_colsum_f32(const float* dy, float* db, int64_t M, int N, hipStream_t s) {
  if (N == 0) return DSP_OK;
  if (M <= kFewRows) {
    hipLaunchKernelGGL(colsum_few_kernel<false>, dim3((uint32_t)(((int64_t)N + 255) / 256)), dim3(256), 0, s, dy, db,
                       (int)M, N);
    return last_launch_status();
  }
  constexpr int G = 16;
  // one launch, or several where the threads are too many for a grid (2^26 columns)
  const int64_t groups = ((int64_t)N + G - 1) / G, most = grid_blocks(CS_THREADS);
  for (int64_t first = 0; first < groups; first += most) {
    hipLaunchKernelGGL((colsum_kernel<false, G>), dim3((uint32_t)std::min(most, groups - first)), dim3(CS_THREADS), 0,
                       s, dy, db, M, N, (int)first);
    const int st = last_launch_status();
    if (st != DSP_OK) return st;
  }
  return DSP_OK;
}

// The partials a caller's workspace provides for (the launch takes as many as it
// needs of them; choose_grad decides): the split count minimising rounds of work-groups
// of 256-row tiles times slices per split plus the extra partials' write and read,
// with at least 32 slices in each split but the last, so that a reduction of at most 63 x
// 64 - 64 = 3968 runs without a workspace.  The size is part of the interface: callers
// allocate it, and programs that stored it must find it enough.
int grad_splits(int64_t M, int64_t N, int64_t K) {
  const bool big = M >= 512 && N >= 512 && M % 8 == 0 && N % 8 == 0 && K >= 2048 &&
                   (int64_t)GBK * M * 2 < (int64_t(1) << 31) && (int64_t)GBK * N * 2 < (int64_t(1) << 31) &&
                   M * N < (int64_t(1) << 31);
  const int bn = !big ? 128 : N >= 2048 ? 256 : 192;
  const int64_t slots = big ? 256 : 512;
  const int64_t tiles = ((M + 255) / 256) * ((N + bn - 1) / bn);
  const int64_t slices = (K + GBK - 1) / GBK;
  const double per_split = (double)M * (double)N * (big ? 8e-7 : 5.5e-7);
  int best = 1;
  double best_cost = 0.0;
  for (int s = 1; s <= 16; ++s) {
    const int64_t per = (slices + s - 1) / s;
    if (per < 32 || per * (s - 1) >= slices) break;  // too short, or the last split empty
    const int64_t rounds = (tiles * s + slots - 1) / slots;
    const double cost = (double)rounds * (double)(per + 2) + (s > 1 ? s * per_split : 0.0);
    if (s == 1 || cost < best_cost) {
      best = s;
      best_cost = cost;
    }
  }
  return best;
}

extern "C" uint32_t dsp_choice_weight_grad(int64_t M, int64_t N, int64_t K, int* splits) {
  const GradChoice c = choose_grad(N, K, M, grad_splits(N, K, M));
  *splits = c.splits;
  const GradTile& t = kGradTiles[c.tile];
  return (uint32_t)(64 * t.tm << 16 | 64 * t.tn) | (c.tile == 2 ? 1u << 31 : 0u);
}

bool grad_gemm_fits(int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb) {
  // 32-bit tile offsets: GBM (or GBK) rows of a row stride in bytes
  return M < (int64_t(1) << 31) && N < (int64_t(1) << 31) && K < (int64_t(1) << 31) &&
         (int64_t)GBM * lda * 2 < (int64_t(1) << 31) && (int64_t)GBM * ldb * 2 < (int64_t(1) << 31) &&
         ((M + GBM - 1) / GBM) * ((N + GBN - 1) / GBN) < (int64_t(1) << 31);
}

int launch_gemm_grad(const void* a, int ta, int64_t lda, const void* b, int tb, int64_t ldb, const void* aux,
                     void* out, int64_t M, int64_t N, int64_t K, int epi, int splits, float* ws, hipStream_t s) {
  if (M == 0 || N == 0) return DSP_OK;
  GradArgs p;
  p.a = static_cast<const bf16*>(a);
  p.b = static_cast<const bf16*>(b);
  p.aux = static_cast<const bf16*>(aux);
  p.out = out;
  p.lda = lda;
  p.ldb = ldb;
  p.M = (int)M;
  p.N = (int)N;
  p.K = (int)K;
  if (ta == 1 && tb == 1) return epi == DSP_GRAD_EPI_F32 ? launch_grad_tt(p, splits, ws, s) : DSP_ERR_ARG;
  if (ta != 0 || tb != 1 || splits != 1) return DSP_ERR_ARG;  // the gradients' other layout
  switch (epi) {
    case DSP_GRAD_EPI_F32: return launch_grad<DSP_GRAD_EPI_F32>(p, s);
    case DSP_GRAD_EPI_BF16: return launch_grad<DSP_GRAD_EPI_BF16>(p, s);
    case DSP_GRAD_EPI_GELU_BWD: return launch_grad<DSP_GRAD_EPI_GELU_BWD>(p, s);
    case DSP_GRAD_EPI_RELU_BWD: return launch_grad<DSP_GRAD_EPI_RELU_BWD>(p, s);
    default: return DSP_ERR_ARG;
  }
}

// 16 columns per work-group (G = 2), or 32 where that still gives every second
// CU one.
int launch_colsum_bf16(const void* dy, float* db, int64_t M, int N, hipStream_t s) {
  if (N == 0) return DSP_OK;
  if (M <= kFewRows) {
    hipLaunchKernelGGL(colsum_few_kernel<true>, dim3((uint32_t)((N / 8 + 255) / 256)), dim3(256), 0, s, dy, db, (int)M, N);
    return last_launch_status();
  }
  if (N >= 128 * 32)
    hipLaunchKernelGGL((colsum_kernel<true, 4>), dim3((uint32_t)((N + 31) / 32)), dim3(CS_THREADS), 0, s, dy, db, M, N,
                       0);
  else
    hipLaunchKernelGGL((colsum_kernel<true, 2>), dim3((uint32_t)((N + 15) / 16)), dim3(CS_THREADS), 0, s, dy, db, M, N,
                       0);
  return last_launch_status();
}

}  // namespace dsp
