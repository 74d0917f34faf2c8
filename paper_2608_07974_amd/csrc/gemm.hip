// GEMM dispatch by type and operand layout, and the split-K reduction.
#include "gemm_epilogue.h"
#include "gemm_route.h"

namespace zl {

// Split-K reduction: C = sum over splits z = 0, 1, .. (in that order) of the
// fp32 partials, then the epilogue, for 8 consecutive columns of a row per
// thread.  RoPE also sums the partials of the 8 partner columns; the
// delta sums of a head meet across its hd / 8 consecutive lanes (rows are
// whole heads, and a head's lanes lie in one wave).  Bound by reading the
// partials; one column per thread took 9.5 us for 2 partials of 1024 x 2048.
__device__ __forceinline__ void sum_splits(const float* p, int nz, int64_t mn, bool vec, int left,
                                           float (&v)[EW]) {
#pragma unroll
  for (int k = 0; k < EW; ++k) v[k] = 0.f;
  if (vec && left >= EW) {
#pragma unroll 4
    for (int z = 0; z < nz; ++z) {
      float x[EW];
      ldv_f32(p + z * mn, x);
#pragma unroll
      for (int k = 0; k < EW; ++k) v[k] += x[k];
    }
  } else {
    for (int z = 0; z < nz; ++z)
#pragma unroll
      for (int k = 0; k < EW; ++k)
        if (k < left) v[k] += p[z * mn + k];
  }
}

__global__ void __launch_bounds__(256) splitk_reduce_kernel(const float* __restrict__ part, int nz,
                                                            int M, int N, EpiArgs e) {
  const int gpr = (N + EW - 1) / EW;  // column groups per row
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int m = (int)(i / gpr), n = (int)(i % gpr) * EW;
  if (m >= M) return;
  const int64_t mn = (int64_t)M * N;
  const bool pv = (N & 3) == 0, vec = epi_vec_ok(e);
  const float* p = part + (int64_t)m * N;
  float v[EW];
  sum_splits(p + n, nz, mn, pv, N - n, v);
  if (e.kind == EPI_ROPE && n < e.n_rot) {
    const int half = e.hd >> 1, j = n % e.hd;
    const bool lo = j < half;
    float pr[EW];
    sum_splits(p + (lo ? n + half : n - half), nz, mn, pv, EW, pr);
    int ps = e.pos[m];
    ps = ps < 0 ? 0 : (ps >= e.max_pos ? e.max_pos - 1 : ps);
    const float2* cs = e.rope + (int64_t)ps * half + (lo ? j : j - half);
#pragma unroll
    for (int k = 0; k < EW; ++k)
      v[k] = lo ? v[k] * cs[k].x - pr[k] * cs[k].y : v[k] * cs[k].x + pr[k] * cs[k].y;
  }
  float ds = 0.f;
  if (e.kind == EPI_STORE_DELTA) {
    float o[EW];
    ldv_act(e.aux, e.out_dtype, (size_t)m * e.ldaux + n, o);
#pragma unroll
    for (int k = 0; k < EW; ++k) {
      const float d = e.scale * v[k];
      ds += (e.out_dtype == BF16 ? bf16_to_f32(f32_to_bf16(d)) : d) * o[k];
    }
    const int lph = e.hd / EW;
    for (int off = 1; off < lph; off <<= 1) ds += __shfl_xor(ds, off, 64);
    if ((threadIdx.x & (lph - 1)) == 0) {
      const int b = m / e.seq, sq = m - b * e.seq, h = n / e.hd;
      e.delta[((int64_t)b * e.nheads + h) * e.seq + sq] = ds;
    }
  }
  epilogue_v(e, M, N, m, n, v, vec);
}

hipError_t launch_splitk_reduce(const float* part, int nz, int M, int N, const EpiArgs& e,
                                hipStream_t s) {
  const int64_t n = (int64_t)M * ((N + EW - 1) / EW);
  hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, part,
                     nz, M, N, e);
  return hipGetLastError();
}

// Defined per operand layout (gemm_kk.hip, gemm_kn.hip, gemm_mn.hip, gemm_mk.hip).
template <bool AK, bool BKM>
hipError_t run_layout(const GemmDesc& g, const EpiArgs& e, hipStream_t s, const char** kname);
template <bool AK, bool BKM>
hipError_t run_pair_layout(const GemmDesc& g1, const EpiArgs& e1, const GemmDesc& g2,
                           const EpiArgs& e2, hipStream_t s, bool* fused);
hipError_t launch_gemm_f32(const GemmDesc& g, const EpiArgs& e, hipStream_t s);
// Up to three products of the same M and layout, few columns each (gemm_skinny.hip).
bool skinny_ok(const GemmDesc& g, const EpiArgs& e);
hipError_t launch_gemm_skinny(const GemmDesc* g, const EpiArgs* e, int np, hipStream_t s);

static GemmShape shape_of(const GemmDesc& g) {
  return {g.M, g.N, g.K, g.a_kmajor, g.b_kmajor, g.part != nullptr, g.part_elems, false, 0};
}

bool launch_gemm_group(const GemmDesc* g, const EpiArgs* e, int np, int dtype, hipStream_t s,
                       hipError_t* err) {
  if (dtype != BF16 || np < 1 || np > 3) return false;
  GemmShape sh[3];
  for (int i = 0; i < np; ++i) {
    if (g[i].M <= 0 || g[i].N <= 0 || g[i].M != g[0].M || g[i].b_kmajor != g[0].b_kmajor ||
        !skinny_ok(g[i], e[i]))
      return false;
    sh[i] = shape_of(g[i]);
  }
  if (!skinny_better(sh, np)) return false;
  *err = launch_gemm_skinny(g, e, np, s);
  return true;
}

hipError_t launch_gemm_pair(const GemmDesc& g1, const EpiArgs& e1, const GemmDesc& g2,
                            const EpiArgs& e2, int dtype, hipStream_t s, bool* fused,
                            const char** kname) {
  *fused = false;
  if (g1.a_kmajor != g2.a_kmajor || g1.b_kmajor != g2.b_kmajor || g1.M <= 0 || g1.N <= 0 ||
      g2.M <= 0 || g2.N <= 0)
    return hipSuccess;
  if (dtype != BF16 || g1.a_kmajor || g1.b_kmajor) return hipSuccess;  // weight gradients only
  hipError_t err = run_pair_layout<false, false>(g1, e1, g2, e2, s, fused);
  if (*fused && kname) *kname = "gemm_dma_256x256_mn";
  return err;
}

hipError_t launch_gemm(const GemmDesc& g, const EpiArgs& e, int dtype, hipStream_t s,
                       const char** kname) {
  if (kname) *kname = "gemm_empty";
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (g.K2 < 0 || (g.K2 > 0 && (!g.A2 || !g.B2))) return hipErrorInvalidValue;
  if (e.kind == EPI_ROPE && (dtype != BF16 || e.hd > 128 || 128 % e.hd != 0 || !e.pos || !e.rope))
    return hipErrorInvalidValue;
  if (e.kind == EPI_LOGITS && (dtype != BF16 || !e.stats || (e.out_dtype != F32 && e.out_dtype != F16) ||
                              (e.pair && g.M % 2) || (e.zy && !e.lab)))
    return hipErrorInvalidValue;
  if (e.kind == EPI_STORE_DELTA &&
      (dtype != BF16 || !e.delta || !e.aux || e.hd < EW || e.hd > 128 || 128 % e.hd ||
       e.seq < 1 || e.nheads < 1 || e.bias || (int64_t)e.nheads * e.hd != g.N || g.M % e.seq))
    return hipErrorInvalidValue;
  if (dtype == F32) {
    if (kname) *kname = "gemm_f32_32x32";
    return launch_gemm_f32(g, e, s);
  }
  const GemmShape sh = shape_of(g);
  if (skinny_ok(g, e) && skinny_better(&sh, 1)) {
    if (kname) *kname = "gemm_skinny";
    return launch_gemm_skinny(&g, &e, 1, s);
  }
  if (g.a_kmajor && g.b_kmajor) return run_layout<true, true>(g, e, s, kname);
  if (g.a_kmajor && !g.b_kmajor) return run_layout<true, false>(g, e, s, kname);
  if (!g.a_kmajor && !g.b_kmajor) return run_layout<false, false>(g, e, s, kname);
  return run_layout<false, true>(g, e, s, kname);
}

}  // namespace zl
