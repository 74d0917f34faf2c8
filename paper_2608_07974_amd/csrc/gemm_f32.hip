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

hipError_t launch_gemm_f32(const GemmDesc& g, const EpiArgs& e, hipStream_t s) {
  const dim3 grid(((g.N + FT - 1) / FT) * ((g.M + FT - 1) / FT));
  if (g.a_kmajor && g.b_kmajor)
    hipLaunchKernelGGL((gemm_f32_kernel<true, true>), grid, dim3(256), 0, s, g, e);
  else if (g.a_kmajor)
    hipLaunchKernelGGL((gemm_f32_kernel<true, false>), grid, dim3(256), 0, s, g, e);
  else if (g.b_kmajor)
    hipLaunchKernelGGL((gemm_f32_kernel<false, true>), grid, dim3(256), 0, s, g, e);
  else
    hipLaunchKernelGGL((gemm_f32_kernel<false, false>), grid, dim3(256), 0, s, g, e);
  return hipGetLastError();
}

}  // namespace zl
