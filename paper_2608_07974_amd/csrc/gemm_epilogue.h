// Epilogues of the GEMM kernels: one element, or 8 consecutive columns.
#pragma once

#include <type_traits>

#include "common.h"

namespace zl {

// f(std::integral_constant<int, i>) for i = B .. E-1: indices that are
// compile-time constants by construction, whatever the unroller decides
// (a register array indexed at run time would live in scratch memory).
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// ---------------------------------------------------------------- epilogue
// GELU (tanh form).  (1 + tanh u) / 2 = 1 / (1 + exp(-2u)): one exponential and
// one division instead of tanhf's branches, and no cancellation in 1 + tanh u
// at negative u.
__device__ inline float gelu_sig(float x) {
  const float c2 = 1.5957691216057308f;  // 2 sqrt(2/pi)
  return 1.f / (1.f + __expf(-c2 * (x + 0.044715f * x * x * x)));
}
__device__ inline float gelu_f(float x) { return x * gelu_sig(x); }
__device__ inline float gelu_grad_f(float x) {
  const float c2 = 1.5957691216057308f;
  const float s = gelu_sig(x);
  // s' = s (1 - s) 2u'; the product vanishes before x^2 can overflow it
  const float ds = s * (1.f - s);
  return s + (ds == 0.f ? 0.f : x * ds * c2 * (1.f + 3.f * 0.044715f * x * x));
}

__device__ __forceinline__ float ld_act(const void* p, int dt, size_t i) {
  if (dt == F16) return f16_to_f32(((const uint16_t*)p)[i]);
  return dt == BF16 ? bf16_to_f32(((const bf16_t*)p)[i]) : ((const float*)p)[i];
}
__device__ __forceinline__ void st_act(void* p, int dt, size_t i, float v) {
  if (dt == F16) ((uint16_t*)p)[i] = f32_to_f16(v);
  else if (dt == BF16) ((bf16_t*)p)[i] = f32_to_bf16(v);
  else ((float*)p)[i] = v;
}

__device__ __forceinline__ void epilogue(const EpiArgs& e, int M, int N, int m, int n, float acc) {
  if (m >= M || n >= N) return;
  const size_t mo = (size_t)m;
  switch (e.kind) {
    case EPI_STORE:
    case EPI_STORE_DELTA: {
      float v = e.scale * acc + (e.bias ? e.bias[n] : 0.f);
      st_act(e.out, e.out_dtype, mo * e.ldo + n, v);
      break;
    }
    case EPI_RESID: {
      float v = e.resid[mo * e.ldr + n] + acc + (e.bias ? e.bias[n] : 0.f);
      ((float*)e.out)[mo * e.ldo + n] = v;
      break;
    }
    case EPI_GELU: {
      float h = acc + (e.bias ? e.bias[n] : 0.f);
      if (e.out_dtype == BF16) h = bf16_to_f32(f32_to_bf16(h));  // as stored
      st_act(e.out2, e.out_dtype, mo * e.ldo2 + n, h);
      st_act(e.out, e.out_dtype, mo * e.ldo + n, gelu_f(h));
      break;
    }
    case EPI_GRAD: {
      float* o = (float*)e.out + mo * e.ldo + n;
      float v = e.scale * acc;
      *o = e.accumulate ? *o + v : v;
      break;
    }
    case EPI_SWIGLU_BWD: {
      float g = ld_act(e.aux, e.out_dtype, mo * e.ldaux + n);
      float u = ld_act(e.aux, e.out_dtype, mo * e.ldaux + n + e.ff);
      float sg = __builtin_amdgcn_rcpf(1.f + __expf(-g));  // hardware reciprocal (1 ulp)
      float silu = g * sg;
      float dsilu = sg * (1.f + g * (1.f - sg));
      st_act(e.out, e.out_dtype, mo * e.ldo + n, acc * u * dsilu);
      st_act(e.out, e.out_dtype, mo * e.ldo + n + e.ff, acc * silu);
      break;
    }
    case EPI_GELU_BWD: {
      float h = ld_act(e.aux, e.out_dtype, mo * e.ldaux + n);
      st_act(e.out, e.out_dtype, mo * e.ldo + n, acc * gelu_grad_f(h));
      break;
    }
    case EPI_ROPE:  // rotation already applied by the staged epilogue
    case EPI_LOGITS:  // the staged epilogue adds the row statistics
      st_act(e.out, e.out_dtype, mo * e.ldo + n, acc);
      break;
  }
}

// EW consecutive columns n .. n+EW-1 of row m.  The vector path (vec: every
// operand 16-byte aligned, every row stride a multiple of 8, checked once
// per block) loads and stores them at once (16-byte accesses for bf16) with
// the same arithmetic as epilogue(); the column tail and unaligned operands
// take the scalar path.
constexpr int EW = 8;
__device__ __forceinline__ void ldv_f32(const float* p, float (&v)[EW]) {
#pragma unroll
  for (int k = 0; k < EW; k += 4) {
    const float4 f = *reinterpret_cast<const float4*>(p + k);
    v[k] = f.x; v[k + 1] = f.y; v[k + 2] = f.z; v[k + 3] = f.w;
  }
}
__device__ __forceinline__ void unpack_bf16x8(const uint4 u, float (&v)[EW]) {
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    v[2 * k] = bf16_to_f32((bf16_t)(w[k] & 0xffff));
    v[2 * k + 1] = bf16_to_f32((bf16_t)(w[k] >> 16));
  }
}
__device__ __forceinline__ void ldv_act(const void* p, int dt, size_t i, float (&v)[EW]) {
  if (dt == BF16) {
    unpack_bf16x8(*reinterpret_cast<const uint4*>(static_cast<const bf16_t*>(p) + i), v);
  } else {
    ldv_f32(static_cast<const float*>(p) + i, v);
  }
}
// dL/dg and dL/du of SwiGLU a = silu(g) u from da, and dL/dh of GELU
__device__ __forceinline__ void swiglu_bwd8(const float (&da)[EW], const float (&g)[EW],
                                            const float (&u)[EW], float (&dg)[EW], float (&du)[EW]) {
#pragma unroll
  for (int i = 0; i < EW; ++i) {
    const float sg = __builtin_amdgcn_rcpf(1.f + __expf(-g[i]));  // hardware reciprocal (1 ulp)
    const float silu = g[i] * sg;
    const float dsilu = sg * (1.f + g[i] * (1.f - sg));
    dg[i] = da[i] * u[i] * dsilu;
    du[i] = da[i] * silu;
  }
}
// fp16 of values that are not above zero, saturating (as f32_to_f16; NaN stays NaN).
__device__ __forceinline__ void stv_f16_neg(void* p, size_t i, const float (&v)[EW]) {
  uint32_t w[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float a = v[2 * k] < -65504.f ? -65504.f : v[2 * k];
    const float b = v[2 * k + 1] < -65504.f ? -65504.f : v[2 * k + 1];
    w[k] = (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)a) |
           ((uint32_t)__builtin_bit_cast(uint16_t, (_Float16)b) << 16);
  }
  *reinterpret_cast<uint4*>(static_cast<uint16_t*>(p) + i) = make_uint4(w[0], w[1], w[2], w[3]);
}
__device__ __forceinline__ void stv_act(void* p, int dt, size_t i, const float (&v)[EW]) {
  if (dt == BF16) {
    uint32_t w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      w[k] = pack_bf16(v[2 * k], v[2 * k + 1]);
    *reinterpret_cast<uint4*>(static_cast<bf16_t*>(p) + i) = make_uint4(w[0], w[1], w[2], w[3]);
  } else if (dt == F16) {
    uint32_t w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      w[k] = (uint32_t)f32_to_f16(v[2 * k]) | ((uint32_t)f32_to_f16(v[2 * k + 1]) << 16);
    *reinterpret_cast<uint4*>(static_cast<uint16_t*>(p) + i) = make_uint4(w[0], w[1], w[2], w[3]);
  } else {
    float* q = static_cast<float*>(p) + i;
#pragma unroll
    for (int k = 0; k < EW; k += 4)
      *reinterpret_cast<float4*>(q + k) = make_float4(v[k], v[k + 1], v[k + 2], v[k + 3]);
  }
}

__device__ __forceinline__ bool epi_vec_ok(const EpiArgs& e) {
  const uintptr_t p = (uintptr_t)e.out | (uintptr_t)e.bias | (uintptr_t)e.resid |
                      (uintptr_t)e.out2 | (uintptr_t)e.aux;
  const int64_t l = e.ldo | e.ldr | e.ldo2 | e.ldaux | (int64_t)e.ff;
  return (p & 15) == 0 && (l & 7) == 0;
}

__device__ __forceinline__ void epilogue_v(const EpiArgs& e, int M, int N, int m, int n,
                                  const float (&a)[EW], bool vec) {
  if (m >= M) return;
  if (!vec || n + EW > N) {
#pragma unroll
    for (int i = 0; i < EW; ++i) epilogue(e, M, N, m, n + i, a[i]);
    return;
  }
  const size_t mo = (size_t)m;
  float v[EW], b[EW];
#pragma unroll
  for (int i = 0; i < EW; ++i) b[i] = 0.f;
  if (e.bias && (e.kind == EPI_STORE || e.kind == EPI_STORE_DELTA || e.kind == EPI_RESID ||
                 e.kind == EPI_GELU))
    ldv_f32(e.bias + n, b);
  switch (e.kind) {
    case EPI_STORE:
    case EPI_STORE_DELTA:
#pragma unroll
      for (int i = 0; i < EW; ++i) v[i] = e.scale * a[i] + b[i];
      stv_act(e.out, e.out_dtype, mo * e.ldo + n, v);
      break;
    case EPI_RESID: {
      float r[EW];
      ldv_f32(e.resid + mo * e.ldr + n, r);
#pragma unroll
      for (int i = 0; i < EW; ++i) v[i] = r[i] + a[i] + b[i];
      stv_act(e.out, F32, mo * e.ldo + n, v);
      break;
    }
    case EPI_GELU: {
      float h[EW];
#pragma unroll
      for (int i = 0; i < EW; ++i) {
        h[i] = a[i] + b[i];
        if (e.out_dtype == BF16) h[i] = bf16_to_f32(f32_to_bf16(h[i]));  // as stored
        v[i] = gelu_f(h[i]);
      }
      stv_act(e.out2, e.out_dtype, mo * e.ldo2 + n, h);
      stv_act(e.out, e.out_dtype, mo * e.ldo + n, v);
      break;
    }
    case EPI_GRAD: {
      float* o = static_cast<float*>(e.out) + mo * e.ldo + n;
#pragma unroll
      for (int i = 0; i < EW; ++i) v[i] = e.scale * a[i];
      if (e.accumulate) {
        float f[EW];
        ldv_f32(o, f);
#pragma unroll
        for (int i = 0; i < EW; ++i) v[i] = f[i] + v[i];
      }
      stv_act(o, F32, 0, v);
      break;
    }
    case EPI_SWIGLU_BWD: {
      float g[EW], u[EW], w[EW];
      ldv_act(e.aux, e.out_dtype, mo * e.ldaux + n, g);
      ldv_act(e.aux, e.out_dtype, mo * e.ldaux + n + e.ff, u);
      swiglu_bwd8(a, g, u, v, w);
      stv_act(e.out, e.out_dtype, mo * e.ldo + n, v);
      stv_act(e.out, e.out_dtype, mo * e.ldo + n + e.ff, w);
      break;
    }
    case EPI_GELU_BWD: {
      float h[EW];
      ldv_act(e.aux, e.out_dtype, mo * e.ldaux + n, h);
#pragma unroll
      for (int i = 0; i < EW; ++i) v[i] = a[i] * gelu_grad_f(h[i]);
      stv_act(e.out, e.out_dtype, mo * e.ldo + n, v);
      break;
    }
    case EPI_ROPE:  // rotation already applied by the staged epilogue
    case EPI_LOGITS:
      stv_act(e.out, e.out_dtype, mo * e.ldo + n, a);
      break;
  }
}

// C = epilogue(sum of nz fp32 partials [M, N]) (gemm.hip).
hipError_t launch_splitk_reduce(const float* part, int nz, int M, int N, const EpiArgs& e,
                                hipStream_t s);

}  // namespace zl
