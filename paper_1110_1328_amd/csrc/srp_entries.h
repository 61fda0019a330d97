// Plane entries of sparse sign random projections: the generator, the entries
// themselves (FP64), and about the entries (the hardware's fp32 functions).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace blsh {

// ---------------------------------------------------------------------------
// Philox-4x32-10 (Salmon et al., SC 2011) and the plane entries
// ---------------------------------------------------------------------------
__device__ inline uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
    const uint32_t lo0 = 0xD2511F53u * c.x, hi0 = __umulhi(0xD2511F53u, c.x);
    const uint32_t lo1 = 0xCD9E8D57u * c.z, hi1 = __umulhi(0xCD9E8D57u, c.z);
    c = make_uint4(hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0);
  }
  return c;
}

// The plane entries of hashes 4 q .. 4 q + 3 at coordinate `term`.
__device__ inline void srp_gauss4(uint32_t term, uint32_t q, uint32_t k0, uint32_t k1, double g[4]) {
  const uint4 w = philox4x32_10(make_uint4(term, q, 0u, 0u), k0, k1);
  const double two32 = 4294967296.0, two_pi = 6.283185307179586476925286766559;
  const double r0 = sqrt(-2.0 * log((double(w.x) + 0.5) / two32)), r1 = sqrt(-2.0 * log((double(w.z) + 0.5) / two32));
  double s1, c1, s3, c3;   // one argument reduction for each sine-cosine pair
  sincos(two_pi * ((double(w.y) + 0.5) / two32), &s1, &c1);
  sincos(two_pi * ((double(w.w) + 0.5) / two32), &s3, &c3);
  g[0] = double(float(r0 * c1));
  g[1] = double(float(r0 * s1));
  g[2] = double(float(r1 * c3));
  g[3] = double(float(r1 * s3));
}

// The plane entry of hash h at coordinate `term`.
__device__ inline double srp_gauss1(uint32_t term, uint32_t h, uint32_t k0, uint32_t k1) {
  const uint4 w = philox4x32_10(make_uint4(term, h >> 2, 0u, 0u), k0, k1);
  const double two32 = 4294967296.0, two_pi = 6.283185307179586476925286766559;
  const double u = (double(h & 2 ? w.z : w.x) + 0.5) / two32, a = (double(h & 2 ? w.w : w.y) + 0.5) / two32;
  double sn, cs;
  sincos(two_pi * a, &sn, &cs);
  const double radius = sqrt(-2.0 * log(u));
  return double(float(radius * (h & 1 ? sn : cs)));
}

// 2-byte storage of a plane entry (Section 4.3): g in (-8, 8) becomes the
// integer floor((g + 8) 2^16 / 16), saturating outside; the code is read back
// as the middle of its cell of width 2^-12 (error at most 2^-13).  Both steps
// are exact in FP64 for every fp32 entry.
__device__ inline uint32_t q16_code(double g) {
  const double c = floor((g + 8.0) * 4096.0);
  return uint32_t(fmin(fmax(c, 0.0), 65535.0));
}

__device__ inline double q16_value(uint32_t code) { return (double(code) + 0.5) * (1.0 / 4096.0) - 8.0; }

// ---------------------------------------------------------------------------
// About the entries
// ---------------------------------------------------------------------------
// |g' - g| over every Philox word: the radius is off by at most 5.76e-7 and the sine
// and cosine by 2.69e-7 (measured over all 2^32 words, test_gpu_bounds.py), the radius is
// below 6.764, and the product and the entry's own rounding to fp32 add at most 4.8e-7:
// 2.87e-6 of the 3.81e-6 allowed.
constexpr float kFastErr = 0x1p-18f;
constexpr float kUnit = 4800.f;          // |g| < 6.77: codes within 16 bits

__device__ inline float srp_fast_radius(uint32_t w) {
  // sqrt(-2 ln u), u = (w + 0.5) 2^-32; near 1 from t = 1 - u, which fp32 holds to its last bit
  const float u = __builtin_fmaf(float(w), 0x1p-32f, 0x1p-33f), t = __builtin_fmaf(float(~w), 0x1p-32f, 0x1p-33f);
  const float near_one = t * (1.f + t * (0.5f + t * (1.f / 3.f + t * (0.25f + t * (0.2f + t * (1.f / 6.f))))));
  const float l = t < 0.0625f ? near_one : -0.69314718f * __builtin_amdgcn_logf(u);
  return __builtin_amdgcn_sqrtf(2.f * l);
}

// About the entry of hash h at coordinate `term`.
__device__ inline float srp_fast1(uint32_t term, uint32_t h, uint32_t k0, uint32_t k1) {
  const uint4 w = philox4x32_10(make_uint4(term, h >> 2, 0u, 0u), k0, k1);
  const float a = __builtin_fmaf(float(h & 2 ? w.w : w.y), 0x1p-32f, 0x1p-33f);
  return srp_fast_radius(h & 2 ? w.z : w.x) * (h & 1 ? __builtin_amdgcn_sinf(a) : __builtin_amdgcn_cosf(a));
}

// About the entries of hashes 4 q .. 4 q + 3 at coordinate `term`.
__device__ inline void srp_fast4(uint32_t term, uint32_t q, uint32_t k0, uint32_t k1, float g[4]) {
  const uint4 w = philox4x32_10(make_uint4(term, q, 0u, 0u), k0, k1);
  const float r0 = srp_fast_radius(w.x), r1 = srp_fast_radius(w.z);
  const float a0 = __builtin_fmaf(float(w.y), 0x1p-32f, 0x1p-33f), a1 = __builtin_fmaf(float(w.w), 0x1p-32f, 0x1p-33f);
  // (the hardware's sine and cosine take revolutions)
  g[0] = r0 * __builtin_amdgcn_cosf(a0);
  g[1] = r0 * __builtin_amdgcn_sinf(a0);
  g[2] = r1 * __builtin_amdgcn_cosf(a1);
  g[3] = r1 * __builtin_amdgcn_sinf(a1);
}

}  // namespace blsh
