// fp32 GEMMs of the block: the linear maps (Eq. 1, 5) and their gradients, fp32
// operands, fp32 products and fp32 accumulation on the matrix cores
// (v_mfma_f32_32x32x2_f32, 256 flops per clock and CU: twice the rate of plain
// fp32 FMAs, and no operand is rounded).  One kernel,
//   out[m][n] = epilogue(sum_k A(m, k) B(n, k)),
// with A(m, k) = a[m * lda + k] (TA = 0) or a[k * lda + m] (TA = 1) and B
// likewise: the forward is (0, 0), dx = dy W is (0, 1), dW = dy^T x is (1, 1).
//
// Bound: the matrix cores.  A 32x32x2 MFMA occupies its SIMD for 64 cycles and
// needs one float per lane and operand, so neither LDS nor L2 bandwidth decides
// the tile.  What does is having several waves on every SIMD at the few thousand
// rows that fp32 runs have: 4 waves on a 64 x 64 tile (each a quarter), K in slices
// of 32 through two LDS buffers with one barrier per slice, the next slice's
// global loads issued during the current one's MFMAs.  (128 x 128 tiles: 77
// against 92 TFLOP/s at 4096 x 3456 x 1152 and 32 against 64 at 2048 x 1152 x 1152,
// both with masked loads.)
//  * Few tiles: KS groups of 4 waves share a tile, each with 1 / KS of the
//    reduction and buffers of its own, and group 0 adds the partial sums in order
//    (deterministic, no workspace).  Alone on its SIMD a wave waits for every
//    slice's loads and fragments.
//  * An operand with the reduction contiguous lies [row][k] in LDS; a lane reads
//    4 k values at once (16 bytes), lanes 0-31 those of k 0-3 and lanes 32-63
//    those of k 4-7 of a group of 8, which feed 4 MFMAs of the two k halves each.
//  * One stored with the reduction strided lies [k][row] and is read a float at a
//    time in the same k order; 32 consecutive lanes read consecutive floats.
//  * B rows are the MFMA's M side, so a lane owns one output row and four
//    consecutive columns per register group.
// Rates: 114 TFLOP/s at 4096 x 3456 x 1152 (80% of the matrix cores' rate at the
// 2.17 GHz the chip runs at), 80 at 2048 x 1152 x 1152 (576 tiles on 256 CUs).
// Before, the forward ran 64 x 64 tiles of plain FMAs (37 and 25) and the
// gradients one thread per output (0.7-1.1 TFLOP/s).
// Any size, stride and 4-byte alignment is accepted: 16-byte loads and stores
// where the rows allow them, single floats otherwise (a wave-uniform choice).
#include <math.h>

#include <algorithm>

#include "dsp_internal.h"

namespace dsp {
namespace {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

enum { FE_NONE = 0, FE_GELU, FE_RESID, FE_RELU, FE_GELU_BWD, FE_RELU_BWD };

constexpr int FBK = 32, FTHR = 256;  // threads: of one group of 4 waves
constexpr int FT = 64;               // tile

struct F32Gemm {
  const float* a;
  const float* b;
  const float* bias;   // [N] or null
  const float* resid;  // FE_RESID: [M][N], read at the unswapped row
  const float* aux;    // backward epilogues: the saved pre-activation [M][N]
  float* out;
  float* pre;          // FE_GELU / FE_RELU: also receives the pre-activation (may be null)
  int64_t lda, ldb, M, N, K;
  uint32_t n_mt, n_nt;
  uint32_t first, count;  // this launch's tiles
  int epi;
  bool vec_n;  // 16-byte stores allowed
  RowSwap rs;
};

// One operand's 32-wide K slices of a 64-row tile: global -> registers -> LDS.
// VEC: every chunk of 4 floats starts on 16 bytes and lies wholly inside or
// outside the operand.
template <bool TRANS, bool VEC>
struct F32Operand {
  static constexpr int P = TRANS ? FT + 4 : FBK + 4;
  static constexpr int ELEMS = TRANS ? FBK * P : FT * P;
  static constexpr int LOADS = FT * FBK / 4 / FTHR;
  static constexpr int CPL = TRANS ? FT / 4 : FBK / 4;  // chunks per line
  float4 pre[LOADS];
  const float* ptr[LOADS];  // each chunk's address in the next slice
  int rows_in[LOADS];       // rows of the chunk inside the operand (TRANS: 0..4, else 0 or 1)
  int64_t step;

  // t: thread of the group; the range starts at reduction index k0.  Chunks of
  // rows past the end point at the tile's first row: what they load only enters
  // outputs that are not stored.
  __device__ __forceinline__ void init(int t, const float* base, int64_t ld, int64_t r0, int64_t rows, int64_t k0) {
    step = TRANS ? FBK * ld : FBK;
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int line = (t + FTHR * i) / CPL, c = ((t + FTHR * i) % CPL) * 4;
      // element j of the chunk: row r (+ j if TRANS), reduction index k (+ j if not)
      const int64_t r = r0 + (TRANS ? c : line), k = k0 + (TRANS ? line : c);
      rows_in[i] = r < rows ? (TRANS ? (int)min(rows - r, (int64_t)4) : 1) : 0;
      const int64_t rc = r < rows ? r : r0;
      ptr[i] = base + (TRANS ? k * ld + rc : rc * ld + k);
    }
  }
  // a slice wholly inside the range (VEC only)
  __device__ __forceinline__ void load_full() {
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      pre[i] = *reinterpret_cast<const float4*>(ptr[i]);
      ptr[i] += step;
    }
  }
  // any slice: `avail` of its reduction indices are in the range, the rest zero
  __device__ __forceinline__ void load_masked(int t, int64_t avail) {
    const int kl = (int)max((int64_t)0, min(avail, (int64_t)FBK));
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int line = (t + FTHR * i) / CPL, c = ((t + FTHR * i) % CPL) * 4;
      const int n = TRANS ? (line < kl ? rows_in[i] : 0) : (rows_in[i] ? kl - c : 0);
      const float* p = ptr[i];
      pre[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if constexpr (VEC) {
        if (n > 0) pre[i] = *reinterpret_cast<const float4*>(p);
      } else {
        if (n > 0) pre[i].x = p[0];
        if (n > 1) pre[i].y = p[1];
        if (n > 2) pre[i].z = p[2];
        if (n > 3) pre[i].w = p[3];
      }
      ptr[i] += step;
    }
  }
  __device__ __forceinline__ void store(int t, float* lds) const {
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int e = t + FTHR * i;
      *reinterpret_cast<float4*>(lds + (e / CPL) * P + (e % CPL) * 4) = pre[i];
    }
  }
  // 4 reduction indices 8 c8 + 4 g + {0..3} of tile row `row`
  __device__ __forceinline__ static float4 frag(const float* lds, int row, int c8, int g) {
    const int k = 8 * c8 + 4 * g;
    if constexpr (!TRANS) return *reinterpret_cast<const float4*>(lds + row * P + k);
    return make_float4(lds[k * P + row], lds[(k + 1) * P + row], lds[(k + 2) * P + row], lds[(k + 3) * P + row]);
  }
};

// One output with the epilogue applied; off_r and off are its offsets before
// and after the row swap.
__device__ __forceinline__ float f32_epilogue(const F32Gemm& p, float v, int64_t off_r, int64_t off, int64_t n) {
  if (p.bias) v += p.bias[n];
  switch (p.epi) {
    case FE_GELU:
      if (p.pre) p.pre[off] = v;
      return 0.5f * v * (1.0f + erff(v * 0.70710678118654752f));
    case FE_RELU:
      if (p.pre) p.pre[off] = v;
      return fmaxf(v, 0.0f);
    case FE_RESID:
      return v + p.resid[off_r];
    case FE_GELU_BWD: {
      const float u = p.aux[off];
      return v * (0.5f * (1.0f + erff(u * 0.70710678118654752f)) + u * 0.3989422804014327f * expf(-0.5f * u * u));
    }
    case FE_RELU_BWD:
      return p.aux[off] > 0.0f ? v : 0.0f;
    default:
      return v;
  }
}

template <bool TA, bool TB, int KS, bool VEC>
__global__ __launch_bounds__(FTHR* KS) void gemm_f32_mfma_kernel(F32Gemm p) {
  using OA = F32Operand<TA, VEC>;
  using OB = F32Operand<TB, VEC>;
  constexpr int STAGE = OA::ELEMS + OB::ELEMS;
  __shared__ __attribute__((aligned(16))) float lds[KS * 2 * STAGE];

  // Tile order: a contiguous range of tiles per XCD (one L2 each), in groups of
  // 8 m-tiles with m fastest, so the tiles running together share A and B rows.
  const uint32_t per = p.count >> 3, extra = p.count & 7u;
  const uint32_t xcd = blockIdx.x & 7u;
  const uint32_t tile = p.first + xcd * per + (xcd < extra ? xcd : extra) + (blockIdx.x >> 3);
  const uint32_t grp = tile / (8 * p.n_nt), first = grp * 8;
  const uint32_t gm = p.n_mt - first < 8 ? p.n_mt - first : 8, rem = tile - grp * 8 * p.n_nt;
  const int64_t m0 = (int64_t)(first + rem % gm) * FT, n0 = (int64_t)(rem / gm) * FT;

  const int t = threadIdx.x % FTHR, ks = KS > 1 ? (int)threadIdx.x / FTHR : 0;
  const int lane = t & 63, wave = t >> 6;
  const int l32 = lane & 31, g = lane >> 5;
  const int wm = (wave & 1) * 32, wn = (wave >> 1) * 32;

  OA oa;
  OB ob;
  floatx16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;

  // this group's slices: all groups take the same number of steps (past its
  // range, or K, a group loads zeros), so the barriers are uniform
  const int64_t slices = (p.K + FBK - 1) / FBK, steps = (slices + KS - 1) / KS;
  const int64_t kb = ks * steps * FBK, ke = min(p.K, kb + steps * FBK);
  float* stage = lds + ks * 2 * STAGE;
  oa.init(t, p.a, p.lda, m0, p.M, kb);
  ob.init(t, p.b, p.ldb, n0, p.N, kb);
  oa.load_masked(t, ke - kb);
  ob.load_masked(t, ke - kb);
  oa.store(t, stage);
  ob.store(t, stage + OA::ELEMS);
  __syncthreads();
  // one slice; `next` issues the next one's loads behind the first fragment reads
  auto slice = [&](int buf, auto next) {
    const float* As = stage + buf * STAGE;
    const float* Bs = As + OA::ELEMS;
#pragma unroll
    for (int c8 = 0; c8 < FBK / 8; ++c8) {
      const float4 af = OA::frag(As, wm + l32, c8, g), bf = OB::frag(Bs, wn + l32, c8, g);
      if (c8 == 0) next();
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(bf.x, af.x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(bf.y, af.y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(bf.z, af.z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(bf.w, af.w, acc, 0, 0, 0);
    }
  };
  auto put = [&](int buf) {  // this buffer was last read before the previous barrier
    oa.store(t, stage + buf * STAGE);
    ob.store(t, stage + buf * STAGE + OA::ELEMS);
    __syncthreads();
  };
  // Slices that are whole in every group load without a mask or a branch (a
  // branch between two ways to load made every slice wait for its own loads:
  // 352 against 309 us at 4096 x 3456 x 1152); the rest of the range follows.
  const int64_t whole = VEC ? min(steps, max((int64_t)0, (p.K - (KS - 1) * steps * FBK) / FBK)) : 0;
  int64_t st = 0;
  for (; st + 1 < whole; ++st) {
    slice(st & 1, [&] {
      oa.load_full();
      ob.load_full();
    });
    put((st + 1) & 1);
  }
  for (; st + 1 < steps; ++st) {
    slice(st & 1, [&] {
      oa.load_masked(t, ke - kb - (st + 1) * FBK);
      ob.load_masked(t, ke - kb - (st + 1) * FBK);
    });
    put((st + 1) & 1);
  }
  slice(st & 1, [] {});
  if constexpr (KS > 1) {
    // groups 1 .. KS - 1 leave their sums in LDS, group 0 adds them in order
    static_assert((KS - 1) * FTHR * 16 <= KS * 2 * STAGE, "the partial sums fit the buffers");
    __syncthreads();  // every fragment is read
    if (ks > 0) {
#pragma unroll
      for (int r = 0; r < 16; ++r) lds[((ks - 1) * 16 + r) * FTHR + t] = acc[r];
    }
    __syncthreads();
    if (ks > 0) return;
#pragma unroll
    for (int q = 0; q < KS - 1; ++q)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] += lds[(q * 16 + r) * FTHR + t];
  }

  // the lane owns row m = .. + l32 and columns n = .. + 8 r4 + 4 g + {0..3}
  const int64_t m = m0 + wm + l32;
  if (m >= p.M) return;
  const int64_t orow = (p.rs.outer ? p.rs.map((int)m) : m) * p.N, irow = m * p.N;
#pragma unroll
  for (int r4 = 0; r4 < 4; ++r4) {
    const int64_t n = n0 + wn + 8 * r4 + 4 * g;
    if (n >= p.N) continue;
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = acc[4 * r4 + e];
      if (p.vec_n || n + e < p.N) v[e] = f32_epilogue(p, v[e], irow + n + e, orow + n + e, n + e);
    }
    if (p.vec_n) {
      *reinterpret_cast<float4*>(p.out + orow + n) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n + e < p.N) p.out[orow + n + e] = v[e];
    }
  }
}

// A gradient whose reduction is a few terms: one thread per output.  The tiles above work
// through 32 terms whatever there are (dW of one row, 64 x 64: 4.4 against 5.7 us;
// 1152 x 1152: 6.3 against 7.5, of 8 rows 8.9 against 7.5).
template <bool TA>
__global__ __launch_bounds__(256) void gemm_f32_few_terms_kernel(F32Gemm p) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x, N = (uint32_t)p.N;
  if (i >= (uint32_t)(p.M * p.N)) return;
  const uint32_t m = i / N, n = i - m * N;
  float v = 0.0f;
  for (int k = 0; k < (int)p.K; ++k) v = fmaf(p.a[TA ? k * p.lda + m : m * p.lda + k], p.b[k * p.ldb + n], v);
  p.out[i] = f32_epilogue(p, v, i, i, n);
}
bool few_terms(int64_t M, int64_t N, int64_t K) {
  return K <= 2 ? M * N < (int64_t(1) << 31) : K <= 16 && M * N <= 65536;
}

bool al16(const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }

// Groups per tile: as many as keep the whole grid resident at once (256 CUs, at
// most 16 waves on each), while each still has a few slices.  us with 1 / 2 / 4
// groups (masked loads), K = 1152: 72 tiles 42.5 / 34 / 31, 288 tiles 61 / 55 / 62,
// 576 tiles 82 / 106 / 94; K = 4608: 72 tiles 238 / 162 / 121, 288 tiles 238 / 205 /
// 240.  With whole slices loaded unmasked: 26 and 49 us (K = 1152, 72 and 288 tiles).

template <bool TA, bool TB>
int launch_f32(F32Gemm p, hipStream_t s) {
  if (p.M == 0 || p.N == 0) return DSP_OK;
  const bool vec = al16(p.a) && p.lda % 4 == 0 && (TA ? p.M : p.K) % 4 == 0 && al16(p.b) && p.ldb % 4 == 0 &&
                   (TB ? p.N : p.K) % 4 == 0;
  p.vec_n = al16(p.out) && p.N % 4 == 0;
  const int64_t n_mt = (p.M + FT - 1) / FT, n_nt = (p.N + FT - 1) / FT;
  // (tile indices and the 8-tile group size are 32-bit)
  if (n_mt >= (int64_t(1) << 31) || n_nt >= (int64_t(1) << 28) || n_mt * n_nt >= (int64_t(1) << 31))
    return DSP_ERR_SHAPE;
  p.n_mt = (uint32_t)n_mt;
  p.n_nt = (uint32_t)n_nt;
  const int64_t tiles = n_mt * n_nt;
  const int ks = tiles <= 256 && p.K >= 16 * FBK ? 4 : tiles <= 512 && p.K >= 8 * FBK ? 2 : 1;
  const dim3 block((uint32_t)(ks * FTHR));
#define DSP_F32_LAUNCH(KS_)                                                               \
  do {                                                                                    \
    if (vec)                                                                              \
      hipLaunchKernelGGL((gemm_f32_mfma_kernel<TA, TB, KS_, true>), grid, block, 0, s, p);  \
    else                                                                                  \
      hipLaunchKernelGGL((gemm_f32_mfma_kernel<TA, TB, KS_, false>), grid, block, 0, s, p); \
  } while (0)
  // one launch, or several where the threads are too many for a grid (2^30 rows)
  const int64_t most = grid_blocks(ks * FTHR);
  for (int64_t first = 0; first < tiles; first += most) {
    p.first = (uint32_t)first;
    p.count = (uint32_t)std::min(most, tiles - first);
    const dim3 grid(p.count);
    if (ks == 4)
      DSP_F32_LAUNCH(4);
    else if (ks == 2)
      DSP_F32_LAUNCH(2);
    else
      DSP_F32_LAUNCH(1);
    const int st = last_launch_status();
    if (st != DSP_OK) return st;
  }
#undef DSP_F32_LAUNCH
  return DSP_OK;
}

}  // namespace

int launch_linear_f32(const float* a, const float* w, const float* bias, const float* residual, float* out, int64_t M,
                      int N, int K, int epilogue, hipStream_t s, float* pre, RowSwap rs) {
  if (pre && epilogue != DSP_EPI_GELU && epilogue != DSP_EPI_RELU) return DSP_ERR_ARG;
  F32Gemm p = {};
  switch (epilogue) {
    case DSP_EPI_NONE: case DSP_EPI_F32: p.epi = FE_NONE; break;
    case DSP_EPI_GELU: p.epi = FE_GELU; break;
    case DSP_EPI_RESID: p.epi = FE_RESID; break;
    case DSP_EPI_RELU: p.epi = FE_RELU; break;
    default: return DSP_ERR_ARG;
  }
  p.a = a;
  p.b = w;
  p.bias = bias;
  p.resid = residual;
  p.out = out;
  p.pre = pre;
  p.lda = p.ldb = K;
  p.M = M;
  p.N = N;
  p.K = K;
  p.rs = rs;
  return launch_f32<false, false>(p, s);
}

int launch_gemm_grad_f32(const float* a, int ta, int64_t lda, const float* b, int tb, int64_t ldb, const float* aux,
                         float* out, int64_t M, int64_t N, int64_t K, int epi, hipStream_t s) {
  F32Gemm p = {};
  p.epi = epi == DSP_GRAD_EPI_GELU_BWD ? FE_GELU_BWD : epi == DSP_GRAD_EPI_RELU_BWD ? FE_RELU_BWD : FE_NONE;
  p.a = a;
  p.b = b;
  p.aux = aux;
  p.out = out;
  p.lda = lda;
  p.ldb = ldb;
  p.M = M;
  p.N = N;
  p.K = K;
  if (!tb) return DSP_ERR_ARG;  // the gradients' layouts: B always has its reduction index strided
  if (M > 0 && N > 0 && few_terms(M, N, K)) {
    const dim3 grid((uint32_t)((M * N + 255) / 256));
    if (ta)
      hipLaunchKernelGGL(gemm_f32_few_terms_kernel<true>, grid, dim3(256), 0, s, p);
    else
      hipLaunchKernelGGL(gemm_f32_few_terms_kernel<false>, grid, dim3(256), 0, s, p);
    return last_launch_status();
  }
  return ta ? launch_f32<true, true>(p, s) : launch_f32<false, true>(p, s);
}

}  // namespace dsp
