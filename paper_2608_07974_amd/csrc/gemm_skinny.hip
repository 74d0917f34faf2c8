// bf16 GEMMs with few output columns (N <= 64): the LoRA products x A^T and
// dy B.  Bound by reading the tall operand once; a 128 x 128 tile multiplies
// mostly padding here (N = 8: 15/16), and needs K split over blocks to have
// enough of them, with a second launch that sums the partials (1024 x 24 x
// 2048: 11 + 5 us, 1024 x 8 x 8192: 10 + 5 us).  Here a block takes 16 or 32 whole
// rows, its eight waves take every eighth 128-wide slice of K straight from
// memory into MFMA fragments, and their sums meet in LDS in wave order.
#include "gemm_epilogue.h"

namespace zl {

typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));
typedef float facc4_t __attribute__((ext_vector_type(4)));

constexpr int SKW = 8;    // waves per block
constexpr int SKN = 64;   // most columns
constexpr int SKK = 128;  // K per wave and step

struct SkinnyProblem {
  const bf16_t* A;
  const bf16_t* B;
  int64_t lda, ldb, ldo;
  void* out;
  float scale;
  int K, N, odt;
};
struct SkinnyArgs {
  SkinnyProblem p[3];
  int M;
};

// MR: 16-row fragments per block, NF: 16-column fragments, BKM: B is [N, K]
// (else [K, N]; its elements are gathered, 2 bytes each, from a few KB that
// stay in the caches).
template <int MR, int NF, bool BKM>
__global__ void __launch_bounds__(SKW * 64) gemm_skinny_kernel(SkinnyArgs a) {
  constexpr int LD = NF * 16 + 1;
  __shared__ float red[SKW][MR * 16][LD];
  const SkinnyProblem p = a.p[blockIdx.y];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int l = lane & 15, kq = (lane >> 4) * 8;
  const int m0 = blockIdx.x * MR * 16;
  facc4_t acc[MR][NF];
#pragma unroll
  for (int i = 0; i < MR; ++i)
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[i][f] = facc4_t{0.f, 0.f, 0.f, 0.f};
  // rows past M and columns past N read the last valid one: never stored
  const bf16_t* ap[MR];
#pragma unroll
  for (int i = 0; i < MR; ++i) ap[i] = p.A + (int64_t)min(m0 + i * 16 + l, a.M - 1) * p.lda;
  int nc[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) nc[f] = min(f * 16 + l, p.N - 1);
  for (int k0 = wave * SKK; k0 < p.K; k0 += SKW * SKK) {
    // the whole slice's loads, then its products; k past K (a multiple of 8)
    // reads k 0 and counts as zero
    uint4 av[SKK / 32][MR], bv[SKK / 32][NF];
#pragma unroll
    for (int h = 0; h < SKK / 32; ++h) {
      const int k = k0 + h * 32 + kq;
      const bool in = k < p.K;
      const int kk = in ? k : 0;
      const uint32_t mask = in ? 0xffffffffu : 0u;
#pragma unroll
      for (int i = 0; i < MR; ++i) {
        const uint4 x = *reinterpret_cast<const uint4*>(ap[i] + kk);
        av[h][i] = make_uint4(x.x & mask, x.y & mask, x.z & mask, x.w & mask);
      }
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        uint4 x;
        if (BKM) {
          x = *reinterpret_cast<const uint4*>(p.B + (int64_t)nc[f] * p.ldb + kk);
        } else {
          const bf16_t* q = p.B + (int64_t)kk * p.ldb + nc[f];
          uint32_t y[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) y[i] = q[i * p.ldb];
          x = make_uint4(y[0] | (y[1] << 16), y[2] | (y[3] << 16), y[4] | (y[5] << 16),
                         y[6] | (y[7] << 16));
        }
        bv[h][f] = make_uint4(x.x & mask, x.y & mask, x.z & mask, x.w & mask);
      }
    }
#pragma unroll
    for (int h = 0; h < SKK / 32; ++h)
#pragma unroll
      for (int i = 0; i < MR; ++i)
#pragma unroll
        for (int f = 0; f < NF; ++f)
          acc[i][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8_t, av[h][i]),
                                                              __builtin_bit_cast(bf8_t, bv[h][f]),
                                                              acc[i][f], 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < MR; ++i)
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][i * 16 + 4 * (lane >> 4) + r][f * 16 + l] = acc[i][f][r];
  __syncthreads();
  for (int t = threadIdx.x; t < MR * 16 * NF * 16; t += SKW * 64) {
    const int row = t / (NF * 16), n = t % (NF * 16), m = m0 + row;
    if (m >= a.M || n >= p.N) continue;
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < SKW; ++w) s += red[w][row][n];
    st_act(p.out, p.odt, (size_t)m * p.ldo + n, p.scale * s);
  }
}

// Plain stores of a product with few columns over a K-major A, all operands
// 16-byte aligned.
bool skinny_ok(const GemmDesc& g, const EpiArgs& e) {
  return g.a_kmajor && e.kind == EPI_STORE && !e.bias && g.N <= SKN && g.K > 0 && g.K % 8 == 0 &&
         g.K2 == 0 && g.ka >= g.K && g.kb >= g.K && g.lda % 8 == 0 && ((uintptr_t)g.A & 15) == 0 &&
         (!g.b_kmajor || (g.ldb % 8 == 0 && ((uintptr_t)g.B & 15) == 0));
}

template <int MR, bool BKM>
static void skinny_go(const SkinnyArgs& a, int np, int nf, hipStream_t s) {
  const dim3 grid((a.M + MR * 16 - 1) / (MR * 16), np), blk(SKW * 64);
  if (nf <= 1) hipLaunchKernelGGL((gemm_skinny_kernel<MR, 1, BKM>), grid, blk, 0, s, a);
  else if (nf <= 2) hipLaunchKernelGGL((gemm_skinny_kernel<MR, 2, BKM>), grid, blk, 0, s, a);
  else hipLaunchKernelGGL((gemm_skinny_kernel<1, 4, BKM>), dim3((a.M + 15) / 16, np), blk, 0, s, a);
}

hipError_t launch_gemm_skinny(const GemmDesc* g, const EpiArgs* e, int np, hipStream_t s) {
  if (np < 1 || np > 3) return hipErrorInvalidValue;
  SkinnyArgs a;
  int nmax = 0;
  for (int i = 0; i < 3; ++i) {
    const GemmDesc& d = g[i < np ? i : 0];
    const EpiArgs& x = e[i < np ? i : 0];
    if (!skinny_ok(d, x) || d.M != g[0].M || d.b_kmajor != g[0].b_kmajor) return hipErrorInvalidValue;
    a.p[i] = {static_cast<const bf16_t*>(d.A), static_cast<const bf16_t*>(d.B), d.lda, d.ldb, x.ldo,
              x.out, x.scale, d.K, d.N, x.out_dtype};
    if (d.N > nmax) nmax = d.N;
  }
  a.M = g[0].M;
  const int nf = (nmax + 15) / 16;
  // 32 rows per block where 16 would give more than two blocks per CU: each
  // B fragment then serves two of A's.
  const bool two = (long)((a.M + 15) / 16) * np > 512 && nf <= 2;
  if (g[0].b_kmajor) {
    if (two) skinny_go<2, true>(a, np, nf, s);
    else skinny_go<1, true>(a, np, nf, s);
  } else {
    if (two) skinny_go<2, false>(a, np, nf, s);
    else skinny_go<1, false>(a, np, nf, s);
  }
  return hipGetLastError();
}

// ------------------------------------------------- low-rank weight gradients
// C[w, n] = sum_t Y[t, w] S[t, n] with few columns n (<= 64): the gradients of
// the LoRA factors, dB = dy^T (x A^T) and dA = (dy B)^T x (stored transposed), all
// of a projection in one launch.  Bound by reading Y once.  As 128 x 128 tiles
// each was two launches (K split, then its sum), 13 us at 1024 tokens of the
// Llama-1B widths, eleven of them per layer.  A block takes 64 columns of Y;
// its eight waves take every eighth 64 rows.  A lane reads 4 columns of 8
// rows (8-byte loads, 128 bytes per 16 lanes) and transposes them in
// registers into four MFMA fragments, of columns 4 l + j; the waves' sums
// meet in LDS in wave order.  With nz > 1 the rows are split over blocks too
// and a second launch sums the partials in order.
struct LowRankArgs {
  LowRankGrad p[4];
  int blk[5];  // first block of each problem, total
  int T, nz, rows;  // rows of one split (a multiple of SKW * 64)
  float scale;
  int acc;
  float* part;  // [block][split][64][NF * 16]
};

__device__ inline int lowrank_problem(const LowRankArgs& a, int b) {
  return b >= a.blk[2] ? (b >= a.blk[3] ? 3 : 2) : (b >= a.blk[1] ? 1 : 0);
}
__device__ inline void lowrank_store(const LowRankArgs& a, const LowRankGrad& p, int w, int n, float s) {
  if (w >= p.W || n >= p.R) return;
  float* o = p.out + (int64_t)w * p.ldw + (int64_t)n * p.ldr;
  const float v = a.scale * s;
  *o = a.acc ? *o + v : v;
}

template <int NF>
__global__ void __launch_bounds__(SKW * 64) lowrank_grad_kernel(LowRankArgs a) {
  constexpr int LD = NF * 16 + 1;
  __shared__ float red[SKW][16][LD];
  const int j0 = lowrank_problem(a, blockIdx.x);
  const LowRankGrad p = a.p[j0];
  const int w0 = ((int)blockIdx.x - a.blk[j0]) * 64;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int l = lane & 15, tq = (lane >> 4) * 8;
  const int tend = min(a.T, ((int)blockIdx.y + 1) * a.rows);
  // columns past W (a multiple of 4) and n past R read valid ones: not stored
  const bf16_t* Y = static_cast<const bf16_t*>(p.Y) + min(w0 + 4 * l, p.W - 4);
  const bf16_t* S = static_cast<const bf16_t*>(p.S);
  int nc[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) nc[f] = min(f * 16 + l, p.R - 1);
  facc4_t acc[4][NF];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[j][f] = facc4_t{0.f, 0.f, 0.f, 0.f};
  for (int t0 = (int)blockIdx.y * a.rows + wave * 64; t0 < tend; t0 += SKW * 64) {
    uint2 y[2][8];
    uint32_t sv[2][NF][8];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int t = t0 + h * 32 + tq + i;
        const int tc = min(t, a.T - 1);
        const uint32_t mask = t < tend ? 0xffffffffu : 0u;  // rows past the end count as zero
        const uint2 v = *reinterpret_cast<const uint2*>(Y + (int64_t)tc * p.ldy);
        y[h][i] = make_uint2(v.x & mask, v.y & mask);
#pragma unroll
        for (int f = 0; f < NF; ++f) sv[h][f][i] = S[(int64_t)tc * p.lds + nc[f]] & mask;
      }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      uint4 b[NF];
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        const uint32_t(&x)[8] = sv[h][f];
        b[f] = make_uint4(x[0] | (x[1] << 16), x[2] | (x[3] << 16), x[4] | (x[5] << 16),
                          x[6] | (x[7] << 16));
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        uint32_t d[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t lo = j < 2 ? y[h][2 * q].x : y[h][2 * q].y;
          const uint32_t hi = j < 2 ? y[h][2 * q + 1].x : y[h][2 * q + 1].y;
          d[q] = __builtin_amdgcn_perm(hi, lo, (j & 1) ? 0x07060302u : 0x05040100u);
        }
        const bf8_t af = __builtin_bit_cast(bf8_t, make_uint4(d[0], d[1], d[2], d[3]));
#pragma unroll
        for (int f = 0; f < NF; ++f)
          acc[j][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, __builtin_bit_cast(bf8_t, b[f]),
                                                              acc[j][f], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    __syncthreads();
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][4 * (lane >> 4) + r][f * 16 + l] = acc[j][f][r];
    __syncthreads();
    for (int t = threadIdx.x; t < 16 * NF * 16; t += SKW * 64) {
      const int row = t / (NF * 16), n = t % (NF * 16);
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < SKW; ++w) s += red[w][row][n];
      const int wl = 4 * row + j;
      if (a.nz == 1) lowrank_store(a, p, w0 + wl, n, s);
      else a.part[((int64_t)blockIdx.x * a.nz + blockIdx.y) * (64 * NF * 16) + wl * (NF * 16) + n] = s;
    }
  }
}

template <int NF>
__global__ void __launch_bounds__(256) lowrank_reduce_kernel(LowRankArgs a) {
  const int j0 = lowrank_problem(a, blockIdx.x);
  const LowRankGrad p = a.p[j0];
  const int w0 = ((int)blockIdx.x - a.blk[j0]) * 64;
  for (int t = threadIdx.x; t < 64 * NF * 16; t += 256) {
    float s = 0.f;
    for (int z = 0; z < a.nz; ++z) s += a.part[((int64_t)blockIdx.x * a.nz + z) * (64 * NF * 16) + t];
    lowrank_store(a, p, w0 + t / (NF * 16), t % (NF * 16), s);
  }
}

template <int NF>
static void lowrank_go(const LowRankArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(lowrank_grad_kernel<NF>, dim3(a.blk[4], a.nz), dim3(SKW * 64), 0, s, a);
  if (a.nz > 1) hipLaunchKernelGGL(lowrank_reduce_kernel<NF>, dim3(a.blk[4]), dim3(256), 0, s, a);
}

bool launch_lowrank_grads(const LowRankGrad* p, int np, int T, float scale, int acc, float* part,
                          size_t part_elems, int dtype, hipStream_t s, hipError_t* err) {
  if (dtype != BF16 || np < 1 || np > 4 || T < 1) return false;
  LowRankArgs a;
  int nmax = 0, b = 0;
  for (int i = 0; i < 4; ++i) {
    const LowRankGrad& q = p[i < np ? i : 0];
    if (q.W < 4 || q.W % 4 || q.ldy % 4 || (uintptr_t)q.Y % 8 || q.R < 1 || q.R > SKN) return false;
    a.p[i] = q;
    a.blk[i] = b;
    if (i < np) b += (q.W + 63) / 64;
    if (q.R > nmax) nmax = q.R;
  }
  a.blk[4] = b;
  const int nf = nmax <= 16 ? 1 : nmax <= 32 ? 2 : 4;
  // Rows are split over blocks only where the columns leave most of the chip
  // idle and each part keeps 1024 rows (128 per wave); the sum is a launch.
  int nz = b < 256 ? 256 / b : 1;
  if (nz > T / 1024) nz = T / 1024;
  const size_t one = (size_t)b * 64 * nf * 16;
  if (!part || nz < 1) nz = 1;
  if ((size_t)nz * one > part_elems) nz = part_elems / one > 1 ? (int)(part_elems / one) : 1;
  a.rows = ((T + nz - 1) / nz + SKW * 64 - 1) / (SKW * 64) * (SKW * 64);
  a.nz = (T + a.rows - 1) / a.rows;
  a.T = T; a.scale = scale; a.acc = acc; a.part = part;
  if (nf == 1) lowrank_go<1>(a, s);
  else if (nf == 2) lowrank_go<2>(a, s);
  else lowrank_go<4>(a, s);
  *err = hipGetLastError();
  return true;
}

}  // namespace zl
