// Device-side helpers shared by the libqcf kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace qcf {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// bfloat16 <-> float32.  Widening is exact; narrowing rounds to nearest, ties
// to even (the hardware conversion on gfx950).
__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) {
  return __builtin_bit_cast(uint16_t, (__bf16)f);
}
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return (uint32_t)f2bf(lo) | ((uint32_t)f2bf(hi) << 16);
}

// 16-byte vector <-> floats for the two storage types.
template <typename T> struct Vec16;
template <> struct Vec16<float> {
  static constexpr int N = 4;
  __device__ static void unpack(const uint4& v, float* f) {
    f[0] = __uint_as_float(v.x); f[1] = __uint_as_float(v.y);
    f[2] = __uint_as_float(v.z); f[3] = __uint_as_float(v.w);
  }
  __device__ static uint4 pack(const float* f) {
    return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]),
                      __float_as_uint(f[3]));
  }
};
template <> struct Vec16<uint16_t> {
  static constexpr int N = 8;
  __device__ static void unpack(const uint4& v, float* f) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[2 * i] = __uint_as_float(w[i] << 16);
      f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
  __device__ static uint4 pack(const float* f) {
    return make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]),
                      pack_bf16x2(f[6], f[7]));
  }
};

__device__ __forceinline__ uint4 ld16(const void* p) { return *reinterpret_cast<const uint4*>(p); }
__device__ __forceinline__ void st16(void* p, const uint4& v) { *reinterpret_cast<uint4*>(p) = v; }

// The same 16-byte accesses with the non-temporal hint, for streams that should
// not displace cache lines that the next kernels of a step read again.
typedef uint32_t u32x4_nt __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 ld16_nt(const void* p) {
  const u32x4_nt x = __builtin_nontemporal_load(reinterpret_cast<const u32x4_nt*>(p));
  return make_uint4(x[0], x[1], x[2], x[3]);
}
__device__ __forceinline__ void st16_nt(void* p, const uint4& v) {
  const u32x4_nt x = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(x, reinterpret_cast<u32x4_nt*>(p));
}

// Rotary frequencies omega_j = theta^(-2j/d), as the factors theta^(-2^(i+1)/d) of j's bits i
// (formed on the host once per launch: omega_j is then at most five float64 products, within
// 1e-15 of the power, where a float64 pow per angle was most of a block's start).
// kBig: angles of 2^52 and more can occur, which takes theta < kBigTheta (positions are 32-bit).
constexpr double kBigTheta = 1e-6;
template <bool kBig>
struct RopeFreq {
  double f[6];
};
template <bool kBig>
inline RopeFreq<kBig> rope_freq(double theta, int d) {
  RopeFreq<kBig> r;
  for (int i = 0; i < 6; ++i) r.f[i] = pow(theta, -2.0 * (double)(1 << i) / (double)d);
  return r;
}

// The (cos, sin) of pos * omega_j, formed in float64 and rounded to float32.  The angle is reduced
// by multiples of pi/2 (two-part constant, one fused multiply-add each: exact to float64 rounding
// for angles below 2^52; kernels of their own send larger ones through the library, whose code in
// every kernel cost assembly 0.5%) and both functions come from their Taylor series on [-pi/4, pi/4] (first omitted terms below 1e-16).  With the
// library's pow and sincos a block's start took longer: assembling a 32K-token request 58.7 ->
// 56.1 us, a layer recompute of 10 x 512 tokens ~1 us less in each of its two rotations.
template <bool kBig>
__device__ __forceinline__ float2 rope_cs(double pos, int j, const RopeFreq<kBig>& fr) {
  double x = pos;
#pragma unroll
  for (int i = 0; i < 6; ++i) x = (j >> i) & 1 ? x * fr.f[i] : x;
  if (kBig && !(fabs(x) < 0x1p52)) {  // (infinity, NaN: NaN)
    double s, c;
    sincos(x, &s, &c);
    return make_float2((float)c, (float)s);
  }
  const double k = rint(x * 0x1.45f306dc9c883p-1);  // 2 / pi
  double r = fma(-k, 0x1.921fb54442d18p+0, x);
  r = fma(-k, 0x1.1a62633145c07p-54, r);
  const double z = r * r;
  double s = -1.0 / 1307674368000.0;  // 1 / 15!
  s = fma(s, z, 1.0 / 6227020800.0);
  s = fma(s, z, -1.0 / 39916800.0);
  s = fma(s, z, 1.0 / 362880.0);
  s = fma(s, z, -1.0 / 5040.0);
  s = fma(s, z, 1.0 / 120.0);
  s = fma(s, z, -1.0 / 6.0);
  s = fma(s * z, r, r);
  double c = 1.0 / 20922789888000.0;  // 1 / 16!
  c = fma(c, z, -1.0 / 87178291200.0);
  c = fma(c, z, 1.0 / 479001600.0);
  c = fma(c, z, -1.0 / 3628800.0);
  c = fma(c, z, 1.0 / 40320.0);
  c = fma(c, z, -1.0 / 720.0);
  c = fma(c, z, 1.0 / 24.0);
  c = fma(c, z, -0.5);
  c = fma(c, z, 1.0);
  const double kq = k * 0.25;
  const int q = (int)((kq - floor(kq)) * 4.0);  // quadrant
  const float sf = (float)s, cf = (float)c;
  const float co = q & 1 ? sf : cf, si = q & 1 ? cf : sf;
  return make_float2((q + 1) & 2 ? -co : co, q & 2 ? -si : si);
}

// One rotate-half pair (x1, x2) turned by the angle whose (cos, sin) is cs:
// (x1 cos - x2 sin, x1 sin + x2 cos), each a product plus one fused
// multiply-add in float32.  Every kernel that rotates keys or queries uses
// this form, so a key rotated by one kernel equals the same key rotated by
// another bit for bit.
__device__ __forceinline__ void rope_pair(float x1, float x2, float2 cs, float& y1, float& y2) {
  y1 = fmaf(x1, cs.x, -(x2 * cs.y));
  y2 = fmaf(x1, cs.y, x2 * cs.x);
}

// Wave-wide reductions (64 lanes).
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ int wave_max_i(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ int wave_min_i(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
  return v;
}

// Number of set bits of `mask` in lanes below the calling lane.
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

}  // namespace qcf
