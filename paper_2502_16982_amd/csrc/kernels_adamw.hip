// AdamW for the parameters that stay off Muon (RMSNorm gains, LM head, embeddings; section 2.2 of the paper), sharing
// lr and weight decay with it.  HBM-bound elementwise kernel: one launch covers up to kAdamwSlots tensors, whose
// pointers and sizes travel in the kernel arguments (no device table, no workspace); each block owns one
// 1024-element span (kAdamwSpan) of one tensor.  fp32 math, moments in fp32, one rounding to the parameter's dtype.
// Bound by memory: 22 (bf16) or 28 bytes per element.  Four elements per thread, their loads all issued before the first
// store; a launch that moves more than the memory-side cache can carry over carries the non-temporal hint.  Measured, TB/s,
// spans of 4096 loaded and stored piece by piece / these / these with the hint: 134 M elements bf16 5.2 / 5.4 / 5.8, 67 M
// fp32 5.3 / 5.5 / 6.0, 24 M bf16 6.7 / 6.9 / 6.4, 2.4 M fp32 (24 tensors) 6.0 / 6.3 / 5.4.
#include <hip/hip_runtime.h>

#include "muon_launch.h"

namespace muon {
namespace {

typedef unsigned short u16;
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// launches that move at least this many bytes use the non-temporal hint (the memory-side cache holds 256 MB)
constexpr long long kStreamBytes = 1ll << 30;

__device__ __forceinline__ float ld1(const float* p) { return *p; }
__device__ __forceinline__ float ld1(const u16* p) { return __uint_as_float(((unsigned)*p) << 16); }
__device__ __forceinline__ void st1(float* p, float v) { *p = v; }
__device__ __forceinline__ void st1(u16* p, float v) {
  const f32x2_t t = {v, 0.f};
  *p = (u16)(__builtin_bit_cast(unsigned, __builtin_convertvector(t, bf16x2_t)) & 0xffffu);
}

struct AdamwScalars {
  float lr, wd, beta1, beta2, eps;
  float inv_bc1, inv_bc2;   // 1/(1 - beta1^t), 1/(1 - beta2^t)
};

__device__ __forceinline__ void adamw_elem(float& p, float g, float& m, float& v, const AdamwScalars& h) {
  m = fmaf(h.beta1, m, (1.f - h.beta1) * g);
  v = fmaf(h.beta2, v, (1.f - h.beta2) * g * g);
  const float mhat = m * h.inv_bc1, vhat = v * h.inv_bc2;
  const float upd = mhat / (sqrtf(vhat) + h.eps);
  p = fmaf(-h.lr, fmaf(h.wd, p, upd), p);
}

// 4 consecutive elements at any alignment of the element (global memory takes such accesses).  NT: non-temporal hint.
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned int u32x2_any __attribute__((ext_vector_type(2), aligned(2)));
#define MUON_GLOBAL __attribute__((address_space(1)))
template <bool NT, typename V>
__device__ __forceinline__ V ld_any(const void* p) {
  const MUON_GLOBAL V* q = (const MUON_GLOBAL V*)p;
  if constexpr (NT) return __builtin_nontemporal_load(q);
  else return *q;
}
template <bool NT, typename V>
__device__ __forceinline__ void st_any(void* p, V v) {
  MUON_GLOBAL V* q = (MUON_GLOBAL V*)p;
  if constexpr (NT) __builtin_nontemporal_store(v, q);
  else *q = v;
}
template <bool NT>
__device__ __forceinline__ void ld4(const float* p, float* out) {
  const f32x4_any v = ld_any<NT, f32x4_any>(p);
#pragma unroll
  for (int e = 0; e < 4; ++e) out[e] = v[e];
}
template <bool NT>
__device__ __forceinline__ void ld4(const u16* p, float* out) {
  const u32x2_any v = ld_any<NT, u32x2_any>(p);
  out[0] = __uint_as_float(v.x << 16);
  out[1] = __uint_as_float(v.x & 0xffff0000u);
  out[2] = __uint_as_float(v.y << 16);
  out[3] = __uint_as_float(v.y & 0xffff0000u);
}
__device__ __forceinline__ unsigned pack2(float lo, float hi) {
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2_t));
}
template <bool NT>
__device__ __forceinline__ void st4(float* p, const float* in) { st_any<NT>(p, f32x4_any{in[0], in[1], in[2], in[3]}); }
template <bool NT>
__device__ __forceinline__ void st4(u16* p, const float* in) { st_any<NT>(p, u32x2_any{pack2(in[0], in[1]), pack2(in[2], in[3])}); }

template <bool NT, typename PT, typename GT>
__device__ __forceinline__ void adamw_span(PT* p, const GT* g, float* m, float* v, long long begin, long long numel,
                                           const AdamwScalars& h) {
  const long long i0 = begin + threadIdx.x * 4;
  if (i0 + 4 <= numel) {
    float pv[4], gv[4], mv[4], vv[4];
    ld4<NT>(m + i0, mv);
    ld4<NT>(v + i0, vv);
    ld4<NT>(p + i0, pv);
    ld4<NT>(g + i0, gv);
#pragma unroll
    for (int e = 0; e < 4; ++e) adamw_elem(pv[e], gv[e], mv[e], vv[e], h);
    st4<NT>(m + i0, mv);
    st4<NT>(v + i0, vv);
    st4<NT>(p + i0, pv);
  } else {
    for (long long i = i0; i < numel; ++i) {     // the last, partial piece of a tensor
      float pv = ld1(p + i), mv = m[i], vv = v[i];
      adamw_elem(pv, ld1(g + i), mv, vv, h);
      m[i] = mv; v[i] = vv; st1(p + i, pv);
    }
  }
}

template <bool NT>
__global__ __launch_bounds__(256) void adamw_kernel(AdamwBatch batch, AdamwScalars h) {
  // the tensor that owns this block: block_start is a prefix sum over the tensors' block counts
  int t = 0;
#pragma unroll
  for (int step = kAdamwSlots / 2; step > 0; step /= 2)
    if (t + step < batch.n && (int)blockIdx.x >= batch.block_start[t + step]) t += step;
  const long long begin = (long long)((int)blockIdx.x - batch.block_start[t]) * kAdamwSpan;
  const long long numel = batch.numel[t];
  float* m = batch.m[t];
  float* v = batch.v[t];
  const int pd = batch.p_dtype[t], gd = batch.g_dtype[t];
  if (pd == kDtypeBF16) {
    if (gd == kDtypeBF16) adamw_span<NT>(static_cast<u16*>(batch.p[t]), static_cast<const u16*>(batch.g[t]), m, v, begin, numel, h);
    else adamw_span<NT>(static_cast<u16*>(batch.p[t]), static_cast<const float*>(batch.g[t]), m, v, begin, numel, h);
  } else {
    if (gd == kDtypeBF16) adamw_span<NT>(static_cast<float*>(batch.p[t]), static_cast<const u16*>(batch.g[t]), m, v, begin, numel, h);
    else adamw_span<NT>(static_cast<float*>(batch.p[t]), static_cast<const float*>(batch.g[t]), m, v, begin, numel, h);
  }
}

}  // namespace

hipError_t launch_adamw(const AdamwBatch& batch, int n_blocks, float lr, float wd, float beta1, float beta2, float eps,
                        float inv_bc1, float inv_bc2, hipStream_t s) {
  if (n_blocks <= 0) return hipSuccess;
  AdamwScalars h{lr, wd, beta1, beta2, eps, inv_bc1, inv_bc2};
  long long bytes = 0;
  for (int t = 0; t < batch.n; ++t)
    bytes += batch.numel[t] * (16 + (batch.p_dtype[t] == kDtypeBF16 ? 4 : 8) + (batch.g_dtype[t] == kDtypeBF16 ? 2 : 4));
  if (bytes >= kStreamBytes) adamw_kernel<true><<<n_blocks, 256, 0, s>>>(batch, h);
  else adamw_kernel<false><<<n_blocks, 256, 0, s>>>(batch, h);
  return hipGetLastError();
}

}  // namespace muon
