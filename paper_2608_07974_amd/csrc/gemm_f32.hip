// GEMM of the fp32 configuration: fp32 MFMA (32x32x2, exact fp32 products and
// accumulation) on one 32 x 32 output tile per block.
//
// The fp32 shapes are small (tens to hundreds in every dimension), so a launch
// is bound by the latency of its chain of k tiles, not by arithmetic: small
// tiles give the most blocks, a 128-deep k tile is loaded into registers at
// once (one memory round trip per 128 of K, the next tile's loads in flight
// under the current one's products), and the four waves take a quarter of the
// k tile each, their sums meeting in LDS in wave order.
#include "gemm_epilogue.h"
#include "gemm_route.h"

namespace zl {

typedef float f32acc_t __attribute__((ext_vector_type(16)));

constexpr int FT = 32, FK = 128;  // tile edge, k depth
constexpr int FLD = FT + 4;       // LDS row stride

// One operand's 32 x 128 tile: 16 values per thread, as four groups of four
// consecutive elements of the contiguous dimension.
template <bool KMAJ>
struct F32Tile {
  float4 v[4];
  // group j of this thread: its row and k
  __device__ static inline void at(int j, int& r, int& k) {
    const int c = j * 256 + threadIdx.x;
    if (KMAJ) { r = c / (FK / 4); k = c % (FK / 4) * 4; }
    else { k = c / (FT / 4); r = c % (FT / 4) * 4; }
  }
  // p: row r0 of the operand; rows / kv: valid rows (from r0) and k.  Values
  // outside are zero.  vec: rows 16-byte aligned with strides of 4.
  __device__ inline void load(const float* p, int64_t ld, int rows, int k0, int kv, bool vec) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int r, k;
      at(j, r, k);
      k += k0;
      const int left = KMAJ ? kv - k : rows - r;  // valid elements from here
      const bool in = KMAJ ? r < rows : k < kv;
      float x[4] = {0.f, 0.f, 0.f, 0.f};
      if (in && left > 0) {
        const float* q = KMAJ ? p + (int64_t)r * ld + k : p + (int64_t)k * ld + r;
        if (vec && left >= 4) {
          const float4 f = *reinterpret_cast<const float4*>(q);
          x[0] = f.x; x[1] = f.y; x[2] = f.z; x[3] = f.w;
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) x[i] = i < left ? q[i] : 0.f;
        }
      }
      v[j] = make_float4(x[0], x[1], x[2], x[3]);
    }
  }
  __device__ inline void store(float* s) const {  // s[k][row]
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int r, k;
      at(j, r, k);
      if (KMAJ) {
        s[(k + 0) * FLD + r] = v[j].x;
        s[(k + 1) * FLD + r] = v[j].y;
        s[(k + 2) * FLD + r] = v[j].z;
        s[(k + 3) * FLD + r] = v[j].w;
      } else {
        *reinterpret_cast<float4*>(s + k * FLD + r) = v[j];
      }
    }
  }
};

template <bool AK, bool BKM>
__global__ void __launch_bounds__(256) gemm_f32_kernel(GemmDesc g, EpiArgs e) {
  __shared__ __align__(16) float lds[2 * FK * FLD];
  float* As = lds;
  float* Bs = lds + FK * FLD;
  const int nbn = (g.N + FT - 1) / FT;
  const int m0 = blockIdx.x / nbn * FT, n0 = blockIdx.x % nbn * FT;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int mr = min(FT, g.M - m0), nr = min(FT, g.N - n0);
  f32acc_t acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  F32Tile<AK> ta;
  F32Tile<BKM> tb;
  // segment 0: (A, B) over K; segment 1: (A2, B2) over K2
  for (int seg = 0; seg < 2; ++seg) {
    const int K = seg ? g.K2 : g.K;
    if (K <= 0) continue;
    const float* A = static_cast<const float*>(seg ? g.A2 : g.A);
    const float* B = static_cast<const float*>(seg ? g.B2 : g.B);
    const int64_t lda = seg ? g.lda2 : g.lda, ldb = seg ? g.ldb2 : g.ldb;
    const int ka = seg ? K : min(g.ka, K), kb = seg ? K : min(g.kb, K);
    const bool va = ((uintptr_t)A & 15) == 0 && (lda & 3) == 0;
    const bool vb = ((uintptr_t)B & 15) == 0 && (ldb & 3) == 0;
    A += AK ? (int64_t)m0 * lda : (int64_t)m0;
    B += BKM ? (int64_t)n0 * ldb : (int64_t)n0;
    ta.load(A, lda, mr, 0, ka, va);
    tb.load(B, ldb, nr, 0, kb, vb);
    for (int k0 = 0; k0 < K; k0 += FK) {
      __syncthreads();  // the previous k tile is fully read
      ta.store(As);
      tb.store(Bs);
      __syncthreads();
      if (k0 + FK < K) {
        ta.load(A, lda, mr, k0 + FK, ka, va);
        tb.load(B, ldb, nr, k0 + FK, kb, vb);
      }
      const float* as = As + (wave * (FK / 4) + (lane >> 5)) * FLD + (lane & 31);
      const float* bs = Bs + (wave * (FK / 4) + (lane >> 5)) * FLD + (lane & 31);
#pragma unroll
      for (int k = 0; k < FK / 4; k += 2)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(as[k * FLD], bs[k * FLD], acc, 0, 0, 0);
    }
  }
  __syncthreads();
  // the four waves' sums, then four consecutive columns per thread
#pragma unroll
  for (int r = 0; r < 16; ++r)
    lds[(wave * FT + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * FLD + (lane & 31)] = acc[r];
  __syncthreads();
  const int row = threadIdx.x >> 3, col = (threadIdx.x & 7) * 4;
  float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float4 f = *reinterpret_cast<const float4*>(&lds[(w * FT + row) * FLD + col]);
    s[0] += f.x; s[1] += f.y; s[2] += f.z; s[3] += f.w;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) epilogue(e, g.M, g.N, m0 + row, n0 + col + i, s[i]);
}

// The same product on the vector ALUs: one 64 x 64 output tile per block, 4 x 4
// per thread, 16 of K a step.  It moves half the operand bytes per product of
// the 32 x 32 tiles and wins once the launch fills the chip.
template <bool AK, bool BKM>
__global__ void __launch_bounds__(256) gemm_simt_kernel(GemmDesc g, EpiArgs e) {
  constexpr int BM = 64, BN = 64, BK = 16;
  __shared__ float As[BK][BM + 4];
  __shared__ float Bs[BK][BN + 4];
  const int nbn = (g.N + BN - 1) / BN;
  const int m0 = blockIdx.x / nbn * BM, n0 = blockIdx.x % nbn * BN;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  float acc[4][4] = {};
  // segment 0: (A, B) over K; segment 1: (A2, B2) over K2
  for (int seg = 0; seg < 2; ++seg) {
    const float* A = reinterpret_cast<const float*>(seg ? g.A2 : g.A);
    const float* B = reinterpret_cast<const float*>(seg ? g.B2 : g.B);
    const int64_t lda = seg ? g.lda2 : g.lda, ldb = seg ? g.ldb2 : g.ldb;
    const int K = seg ? g.K2 : g.K, ka = seg ? g.K2 : g.ka, kb = seg ? g.K2 : g.kb;
    for (int k0 = 0; k0 < K; k0 += BK) {
      for (int idx = threadIdx.x; idx < BM * BK; idx += 256) {
        int r, k;
        if (AK) { r = idx / BK; k = idx % BK; } else { r = idx % BM; k = idx / BM; }
        const int gr = m0 + r, gk = k0 + k;
        float v = 0.f;
        if (gr < g.M && gk < ka) v = AK ? A[(int64_t)gr * lda + gk] : A[(int64_t)gk * lda + gr];
        As[k][r] = v;
      }
      for (int idx = threadIdx.x; idx < BN * BK; idx += 256) {
        int r, k;
        if (BKM) { r = idx / BK; k = idx % BK; } else { r = idx % BN; k = idx / BN; }
        const int gr = n0 + r, gk = k0 + k;
        float v = 0.f;
        if (gr < g.N && gk < kb) v = BKM ? B[(int64_t)gr * ldb + gk] : B[(int64_t)gk * ldb + gr];
        Bs[k][r] = v;
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < BK; ++k) {
        float a[4], b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] = As[k][ty * 4 + i];
#pragma unroll
        for (int j = 0; j < 4; ++j) b[j] = Bs[k][tx * 4 + j];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) epilogue(e, g.M, g.N, m0 + ty * 4 + i, n0 + tx * 4 + j, acc[i][j]);
}

template <bool AK, bool BKM>
static hipError_t run_f32(const GemmDesc& g, const EpiArgs& e, hipStream_t s) {
  if (f32_large_tiles(g.M, g.N, g.K + g.K2, AK, BKM)) {
    const dim3 grid(((g.N + 63) / 64) * ((g.M + 63) / 64));
    hipLaunchKernelGGL((gemm_simt_kernel<AK, BKM>), grid, dim3(256), 0, s, g, e);
  } else {
    const dim3 grid(((g.N + FT - 1) / FT) * ((g.M + FT - 1) / FT));
    hipLaunchKernelGGL((gemm_f32_kernel<AK, BKM>), grid, dim3(256), 0, s, g, e);
  }
  return hipGetLastError();
}

hipError_t launch_gemm_f32(const GemmDesc& g, const EpiArgs& e, hipStream_t s) {
  if (g.a_kmajor) return g.b_kmajor ? run_f32<true, true>(g, e, s) : run_f32<true, false>(g, e, s);
  return g.b_kmajor ? run_f32<false, true>(g, e, s) : run_f32<false, false>(g, e, s);
}

}  // namespace zl
