// Shared device helpers for the gfx950 kernels: storage types, vector loads, wave reductions.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace otas {

typedef __bf16 bf16_t;
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kWave = 64;

template <typename T> struct Vec;          // 16-byte vector of the storage type
template <> struct Vec<float> {
  static constexpr int N = 4;
  floatx4 v;
  __device__ float get(int i) const { return v[i]; }
  __device__ void set(int i, float f) { v[i] = f; }
};
template <> struct Vec<bf16_t> {
  static constexpr int N = 8;
  bf16x8 v;
  __device__ float get(int i) const { return (float)v[i]; }
  __device__ void set(int i, float f) { v[i] = (bf16_t)f; }   // round to nearest even (v_cvt_pk_bf16_f32)
};

template <typename T> __device__ inline Vec<T> load_vec(const T* p) {
  return *reinterpret_cast<const Vec<T>*>(p);
}
template <typename T> __device__ inline void store_vec(T* p, const Vec<T>& v) {
  *reinterpret_cast<Vec<T>*>(p) = v;
}

template <typename T> struct alignas(4 * sizeof(T)) Quad { T x[4]; };   // 4 consecutive elements, one load
template <typename T> struct alignas(8 * sizeof(T)) Oct { T x[8]; };    // 8 consecutive elements, one load

__device__ inline float to_float(float x) { return x; }
__device__ inline float to_float(bf16_t x) { return (float)x; }
template <typename T> __device__ inline floatx4 load4(const T* p) {   // four elements widened
  const Quad<T> v = *reinterpret_cast<const Quad<T>*>(p);
  return floatx4{to_float(v.x[0]), to_float(v.x[1]), to_float(v.x[2]), to_float(v.x[3])};
}
template <typename T> __device__ inline T from_float(float x);
template <> __device__ inline float from_float<float>(float x) { return x; }
template <> __device__ inline bf16_t from_float<bf16_t>(float x) { return (bf16_t)x; }

// Exchanges between the lanes of a wave in registers.  A __shfl is a round trip through the LDS pipe (over 100 clocks),
// and the reductions below are chains of them that nothing covers; these take a VALU instruction each.  All 64 lanes active.
// Same bits; ViT-B pass of one query with r = 16 540 -> 529 us, of 64 1.992 -> 1.974 ms (MI355X).
struct LaneHalves { float lo, hi; };
// lo: in both halves of the wave the lower half's value, hi: the upper half's.
__device__ inline LaneHalves wave_halves(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ inline float xor32_sum(float v) { const LaneHalves h = wave_halves(v); return h.lo + h.hi; }
__device__ inline float xor32_max(float v) { const LaneHalves h = wave_halves(v); return fmaxf(h.lo, h.hi); }
__device__ inline float xor16_sum(float v) {   // rows of 16 lanes: 0 with 1, 2 with 3
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Data-parallel-primitive controls inside a row of 16 lanes.
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141;
constexpr int dpp_ror(int n) { return 0x120 + n; }
template <int CTRL> __device__ inline float dpp_sum(float v) {   // v + the value of the lane the control names
  return v + __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xF, 0xF, true));
}

// Butterfly reduction over the 64 lanes of a wave (partners 32, 16, 8, 4, 2, 1 apart): every lane ends with the same
// value, and the order of additions does not depend on which lanes hold data.  From the step over 8 lanes on the values
// repeat inside a row with the period reached, so that a rotation by half of it meets the butterfly's partner's value.
__device__ inline float wave_sum(float v) {
  v = xor16_sum(xor32_sum(v));
  v = dpp_sum<dpp_ror(8)>(v);
  v = dpp_sum<dpp_ror(4)>(v);
  v = dpp_sum<dpp_ror(2)>(v);
  return dpp_sum<dpp_ror(1)>(v);
}

// Exact GELU: 0.5 x (1 + erf(x / sqrt 2)).
__device__ inline float gelu_exact(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752440f)); }

// The same GELU for results that are rounded to bf16 afterwards, written as
//   0.5 x (1 + erf(x / sqrt 2)) = max(x, 0) - |x| Phi(-|x|),   Phi = the standard normal distribution function.
// log2 Phi(-u) is smooth and close to a parabola: a polynomial of degree 6 in u on [0, 6] (least squares on a
// fine grid, re-weighted until the error of u Phi(-u) is flat) reproduces u Phi(-u) to 5e-8; beyond u = 6 the
// term is below 6e-9 and u is clamped (in the polynomial and in the product).  Evaluated in fp32 the whole function is within 3e-7 of the exact one
// over [-8, 8], four orders below half a bf16 unit of a result of size 1, for six multiply-adds and one exp2 --
// against a reciprocal, an exp2 and eleven other instructions for erf by formula 7.1.26 of Abramowitz & Stegun
// (same accuracy), which this replaces: transcendentals run at quarter rate, and in the GEMM epilogue of the
// MLP's first linear this function is all the ALU work there is.
__device__ inline float gelu_bf16(float x) {
  const float u = fminf(fabsf(x), 6.0f);
  float p = fmaf(3.30306029e-05f, u, -7.68667320e-04f);
  p = fmaf(p, u, 8.07889923e-03f);
  p = fmaf(p, u, -5.34093268e-02f);
  p = fmaf(p, u, -4.58772987e-01f);
  p = fmaf(p, u, -1.15120113e+00f);
  p = fmaf(p, u, -9.99993145e-01f);
  const float relu = __builtin_amdgcn_fmed3f(x, 0.0f, 3.0e38f);   // max(x, 0) in one instruction
  return fmaf(-u, __builtin_amdgcn_exp2f(p), relu);   // u, not |x|: beyond 6 the term stays 6e-9 (also for infinities)
}

}  // namespace otas
