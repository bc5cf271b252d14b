// Shared device-side helpers for the population-step kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pbt {

typedef uint16_t bf16_t;  // raw bfloat16 bits

// Round-to-nearest-even float -> bfloat16 (NaN kept quiet).
// float -> bf16, round to nearest even: the matrix-core generation has a conversion instruction
// (v_cvt_pk_bf16_f32), which the compiler emits for these casts
__device__ __forceinline__ bf16_t f2bf(float f) { return __builtin_bit_cast(bf16_t, (__bf16)f); }
// two at once: lo in bits 0..15, hi in bits 16..31
__device__ __forceinline__ uint32_t f2bf_pair(float lo, float hi) {
  typedef __attribute__((ext_vector_type(2))) float f32x2_t;
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
__device__ __forceinline__ float bf2f(bf16_t h) { return __uint_as_float(((uint32_t)h) << 16); }
// double -> bf16 with a single round-to-nearest-even: first to float with round-to-odd (truncate
// toward zero, then set the last bit if anything was lost), which the final rounding cannot mistake.
__device__ __forceinline__ bf16_t d2bf(double v) {
  float f = (float)v;
  const double back = (double)f;
  if (back != v) {
    uint32_t b = __float_as_uint(f);
    if (fabs(back) > fabs(v)) b -= 1u;  // step toward zero (f is finite and non-zero here)
    f = __uint_as_float(b | 1u);
  }
  return f2bf(f);
}

// bf16(x * s) with a single round-to-nearest-even of the exact product, in float arithmetic: hi = fl(x s) and the
// exact remainder lo = x s - hi (one fma).  Rounding hi to bf16 can only differ from rounding the exact product
// when hi sits exactly half way between two bf16 values; the sign of lo then says on which side the product lies.
// (Products so small that lo could underflow take the double route.)
__device__ __forceinline__ bf16_t bf16_times_float(bf16_t x, float s) {
  const float xf = bf2f(x);
  const float hi = xf * s;
  const uint32_t b = __float_as_uint(hi);
  if ((b & 0xffffu) != 0x8000u) return f2bf(hi);
  if ((b & 0x7f800000u) < (40u << 23)) return d2bf((double)xf * (double)s);
  const float lo = fmaf(xf, s, -hi);
  if (lo == 0.f) return f2bf(hi);                                  // a true tie: to even
  const bool away = (lo > 0.f) == (hi > 0.f);                      // the product is larger in magnitude than hi
  return (bf16_t)((b >> 16) + (away ? 1u : 0u));
}

// eight values, rounded to bf16, times 0 (keeping the sign) or the scale by their keep bits, rounded once more
__device__ __forceinline__ uint4 keep_times_scale(const float* a, uint32_t bits, float scale) {
  uint32_t out[4], tie = 0;
  float x[8];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t r = f2bf_pair(a[2 * q], a[2 * q + 1]);
    x[2 * q] = __uint_as_float(r << 16);
    x[2 * q + 1] = __uint_as_float(r & 0xffff0000u);
    const float lo = x[2 * q] * scale, hi = x[2 * q + 1] * scale;
    // (the rounded product rounds wrongly only where it lies half way between two bf16 values: bf16_times_float looks into those)
    tie |= ((__float_as_uint(lo) & 0xffffu) == 0x8000u || (__float_as_uint(hi) & 0xffffu) == 0x8000u) ? 1u << q : 0u;
    const uint32_t keep = (((bits >> (2 * q)) & 1u) ? 0xffffu : 0x8000u) | (((bits >> (2 * q + 1)) & 1u) ? 0xffff0000u : 0x80000000u);
    // (x * 0 keeps the sign: of the value itself, which the scale does not change)
    out[q] = f2bf_pair(lo, hi) & keep;
  }
  if (tie) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if ((tie >> q) & 1u) {
        uint32_t w = 0;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const bf16_t b = (bf16_t)(__float_as_uint(x[2 * q + e]) >> 16);
          const bf16_t y = (bits >> (2 * q + e)) & 1u ? bf16_times_float(b, scale) : (bf16_t)(b & 0x8000u);
          w |= (uint32_t)y << (16 * e);
        }
        out[q] = w;
      }
  }
  return make_uint4(out[0], out[1], out[2], out[3]);
}

enum { ACT_NONE = 0, ACT_RELU = 1, ACT_GELU = 2, ACT_LEAKY_RELU = 3, ACT_TANH = 4 };

// Standard normal CDF Phi(z) and density phi(z) for GELU and its derivative, from ONE exponential:
// erf(x) = 1 - (a1 t + ... + a5 t^5) exp(-x^2), t = 1/(1 + p x), x >= 0 (Abramowitz & Stegun
// 7.1.26, |error| <= 1.5e-7), with x = |z|/sqrt(2) so that exp(-x^2) = exp(-z^2/2) is also what
// phi(z) needs.  About a dozen instructions instead of a library erff call per element, which
// matters in GEMM epilogues that touch 8 million elements per layer (the correctly rounded reciprocal was a third of it: held-out pass
// of the wide MLPs 2.86 -> 2.66 ms without, the same error, 2.7e-7 at most against double).
__device__ __forceinline__ void normal_cdf_pdf(float z, float& cdf, float& pdf) {
  // (clamped where exp(-x^2) is long zero, so that the reciprocal's argument is finite: one Newton step on the estimate, not a division)
  const float x = fminf(fabsf(z) * 0.70710678118654752f, 1e9f);
  const float q = fmaf(0.3275911f, x, 1.f), t0 = __builtin_amdgcn_rcpf(q), t = fmaf(fmaf(-q, t0, 1.f), t0, t0);
  const float e = __expf(-x * x);
  float poly = fmaf(1.061405429f, t, -1.453152027f);
  poly = fmaf(poly, t, 1.421413741f);
  poly = fmaf(poly, t, -0.284496736f);
  poly = fmaf(poly, t, 0.254829592f);
  const float half_erfc = 0.5f * poly * t * e;          // 0.5 * erfc(|z| / sqrt 2)
  cdf = z >= 0.f ? 1.f - half_erfc : half_erfc;
  pdf = 0.39894228040143268f * e;
}

// Activation and its derivative as functions of the pre-activation z.
__device__ __forceinline__ float act_fwd(float z, int kind) {
  switch (kind) {
    case ACT_RELU: return z > 0.f ? z : 0.f;
    case ACT_GELU: { float c, p; normal_cdf_pdf(z, c, p); return z * c; }
    case ACT_LEAKY_RELU: return z > 0.f ? z : 0.2f * z;
    case ACT_TANH: return tanhf(z);
    default: return z;
  }
}
__device__ __forceinline__ float act_bwd(float z, int kind) {
  switch (kind) {
    case ACT_RELU: return z > 0.f ? 1.f : 0.f;
    case ACT_GELU: { float c, p; normal_cdf_pdf(z, c, p); return fmaf(z, p, c); }
    case ACT_LEAKY_RELU: return z > 0.f ? 1.f : 0.2f;
    case ACT_TANH: { float t = tanhf(z); return 1.f - t * t; }
    default: return 1.f;
  }
}

// The same for eight values with the choice of the activation taken once, outside the element loop (inside
// it the compiler keeps a branch ladder per element).
__device__ __forceinline__ void act_fwd8(const float* z, float* a, int kind) {
  switch (kind) {
    case ACT_RELU:
#pragma unroll
      for (int e = 0; e < 8; ++e) a[e] = z[e] > 0.f ? z[e] : 0.f;
      break;
    case ACT_GELU:
#pragma unroll
      for (int e = 0; e < 8; ++e) { float c, p; normal_cdf_pdf(z[e], c, p); a[e] = z[e] * c; }
      break;
    case ACT_LEAKY_RELU:
#pragma unroll
      for (int e = 0; e < 8; ++e) a[e] = z[e] > 0.f ? z[e] : 0.2f * z[e];
      break;
    case ACT_TANH:
#pragma unroll
      for (int e = 0; e < 8; ++e) a[e] = tanhf(z[e]);
      break;
    default:
#pragma unroll
      for (int e = 0; e < 8; ++e) a[e] = z[e];
  }
}
// d[e] = v[e] * act'(z[e])
__device__ __forceinline__ void act_bwd_scale8(const float* v, const float* z, float* d, int kind) {
  switch (kind) {
    case ACT_RELU:
#pragma unroll
      for (int e = 0; e < 8; ++e) d[e] = v[e] * (z[e] > 0.f ? 1.f : 0.f);
      break;
    case ACT_GELU:
#pragma unroll
      for (int e = 0; e < 8; ++e) { float c, p; normal_cdf_pdf(z[e], c, p); d[e] = v[e] * fmaf(z[e], p, c); }
      break;
    case ACT_LEAKY_RELU:
#pragma unroll
      for (int e = 0; e < 8; ++e) d[e] = v[e] * (z[e] > 0.f ? 1.f : 0.2f);
      break;
    case ACT_TANH:
#pragma unroll
      for (int e = 0; e < 8; ++e) { const float t = tanhf(z[e]); d[e] = v[e] * (1.f - t * t); }
      break;
    default:
#pragma unroll
      for (int e = 0; e < 8; ++e) d[e] = v[e] * 1.f;
  }
}

// Sum (largest) over the 64 lanes of a wavefront, all of them active; every lane receives it.  The butterfly order is fixed (distances 32, 16, ... 1),
// so the result does not depend on scheduling.  Each stage is one or two vector instructions: halves and rows of 16 lanes change places, inside a row the
// rotation by 8 or 4 reaches a lane with the partner's value.  (Through __shfl_xor they were six LDS permutations in
// series: with them, and without the next row's loads ahead, the backward LayerNorm of 6 members' 720 x 192 took 10.8 us, 8.4 now.)
template <class Op>
__device__ __forceinline__ float wave_butterfly(float v, Op op) {
  const auto f = [](uint32_t u) { return __uint_as_float(u); };
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = op(f(h[0]), f(h[1]));
  const auto g = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = op(f(g[0]), f(g[1]));
  v = op(v, f(__builtin_amdgcn_mov_dpp(__float_as_uint(v), 0x128, 0xf, 0xf, true)));   // row_ror:8
  v = op(v, f(__builtin_amdgcn_mov_dpp(__float_as_uint(v), 0x124, 0xf, 0xf, true)));   // row_ror:4
  v = op(v, f(__builtin_amdgcn_mov_dpp(__float_as_uint(v), 0x4e, 0xf, 0xf, true)));    // quad_perm [2, 3, 0, 1]
  return op(v, f(__builtin_amdgcn_mov_dpp(__float_as_uint(v), 0xb1, 0xf, 0xf, true)));  // quad_perm [1, 0, 3, 2]
}
__device__ __forceinline__ float wave_sum(float v) {
  return wave_butterfly(v, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float wave_max(float v) {
  return wave_butterfly(v, [](float a, float b) { return fmaxf(a, b); });
}

}  // namespace pbt
