// Complex arithmetic and storage formats for the Wilson-Dirac kernels.
//
// Fields are stored as arrays of complex pairs in one of four storage
// formats (FP64, FP32, FP16, BF16). Kernels load a pair, convert it to the
// compute type (double or float) and convert back when storing.
// Conversions from a wider to a narrower format round to nearest even.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dw {

template <typename T>
struct cplx {
  T re, im;
};

template <typename T>
__host__ __device__ __forceinline__ cplx<T> mk(T r, T i) { return cplx<T>{r, i}; }
template <typename T>
__host__ __device__ __forceinline__ cplx<T> operator+(cplx<T> a, cplx<T> b) { return {a.re + b.re, a.im + b.im}; }
template <typename T>
__host__ __device__ __forceinline__ cplx<T> operator-(cplx<T> a, cplx<T> b) { return {a.re - b.re, a.im - b.im}; }
template <typename T>
__host__ __device__ __forceinline__ cplx<T> operator-(cplx<T> a) { return {-a.re, -a.im}; }
template <typename T>
__host__ __device__ __forceinline__ cplx<T> operator*(cplx<T> a, cplx<T> b) {
  return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
template <typename T>
__host__ __device__ __forceinline__ cplx<T> operator*(T s, cplx<T> a) { return {s * a.re, s * a.im}; }
template <typename T>
__host__ __device__ __forceinline__ cplx<T>& operator+=(cplx<T>& a, cplx<T> b) { a.re += b.re; a.im += b.im; return a; }
template <typename T>
__host__ __device__ __forceinline__ cplx<T>& operator-=(cplx<T>& a, cplx<T> b) { a.re -= b.re; a.im -= b.im; return a; }
template <typename T>
__host__ __device__ __forceinline__ cplx<T> conj(cplx<T> a) { return {a.re, -a.im}; }
// conj(a) * b
template <typename T>
__host__ __device__ __forceinline__ cplx<T> cdot(cplx<T> a, cplx<T> b) {
  return {a.re * b.re + a.im * b.im, a.re * b.im - a.im * b.re};
}
template <typename T>
__host__ __device__ __forceinline__ T norm2(cplx<T> a) { return a.re * a.re + a.im * a.im; }
// acc += a b and acc -= a b as four fused multiply-adds (one rounding per term)
template <typename T>
__host__ __device__ __forceinline__ void cmac(cplx<T>& acc, cplx<T> a, cplx<T> b) {
  acc.re = fma(a.re, b.re, acc.re);
  acc.re = fma(-a.im, b.im, acc.re);
  acc.im = fma(a.re, b.im, acc.im);
  acc.im = fma(a.im, b.re, acc.im);
}
// acc += conj(a) b
template <typename T>
__host__ __device__ __forceinline__ void cmacj(cplx<T>& acc, cplx<T> a, cplx<T> b) {
  acc.re = fma(a.re, b.re, acc.re);
  acc.re = fma(a.im, b.im, acc.re);
  acc.im = fma(a.re, b.im, acc.im);
  acc.im = fma(-a.im, b.re, acc.im);
}
// acc += a b or conj(a) b. CHAIN: every product chained into the sum by fused
// multiply-adds, four instructions, each rounding at the size of the sum. Else the
// product is formed apart and added, six instructions and the smaller error: FP32
// operator 5.09e-8 instead of 5.15e-8 of the norm (with the clover term 5.29e-8, 5.39e-8),
// FP64 preconditioner with the clover term 1.83e-16 instead of 1.87e-16 (2x4x4x4
// blocks). Chains serve where the fields' 16 bits round far more than either (24^3x48 FP16
// operator with the clover term, 4 sides: 212 -> 193 us), and in the two-thread
// preconditioner, where the sums are short enough to come out no worse.
template <bool CHAIN, typename T>
__host__ __device__ __forceinline__ void cmadd(cplx<T>& acc, cplx<T> a, cplx<T> b) {
  if constexpr (CHAIN) cmac(acc, a, b);
  else acc += a * b;
}
template <bool CHAIN, typename T>
__host__ __device__ __forceinline__ void cmaddj(cplx<T>& acc, cplx<T> a, cplx<T> b) {
  if constexpr (CHAIN) cmacj(acc, a, b);
  else acc += cdot(a, b);
}
template <typename T>
__host__ __device__ __forceinline__ void cmsub(cplx<T>& acc, cplx<T> a, cplx<T> b) {
  acc.re = fma(-a.re, b.re, acc.re);
  acc.re = fma(a.im, b.im, acc.re);
  acc.im = fma(-a.re, b.im, acc.im);
  acc.im = fma(-a.im, b.re, acc.im);
}
// multiply by +i and -i
template <typename T>
__host__ __device__ __forceinline__ cplx<T> mul_i(cplx<T> a) { return {-a.im, a.re}; }
template <typename T>
__host__ __device__ __forceinline__ cplx<T> mul_mi(cplx<T> a) { return {a.im, -a.re}; }

// ---- sums over a wavefront ---------------------------------------------------
// FP64 sums stay in registers: data-parallel-primitive moves instead of LDS
// permutes (two permutes and a wait on the LDS per step; a chain of six steps
// took about 700 cycles that way).
template <int CTRL, int ROWS, bool ZERO>
__device__ __forceinline__ double dpp64(double old, double v) {
  const int lo = __builtin_amdgcn_update_dpp(__double2loint(old), __double2loint(v), CTRL, ROWS, 0xf, ZERO);
  const int hi = __builtin_amdgcn_update_dpp(__double2hiint(old), __double2hiint(v), CTRL, ROWS, 0xf, ZERO);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double lane_value(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}
// sum over the 64 lanes, in every lane (fixed order: rows of 16, then the rows)
__device__ __forceinline__ double wave_total(double a) {
  a += dpp64<0x111, 0xf, false>(0.0, a);  // row_shr:1
  a += dpp64<0x112, 0xf, false>(0.0, a);  // row_shr:2
  a += dpp64<0x114, 0xf, false>(0.0, a);  // row_shr:4
  a += dpp64<0x118, 0xf, false>(0.0, a);  // row_shr:8
  a += dpp64<0x142, 0xa, false>(0.0, a);  // row_bcast:15 into rows 1 and 3
  a += dpp64<0x143, 0xc, false>(0.0, a);  // row_bcast:31 into rows 2 and 3
  return lane_value(a, 63);
}
// largest value over the 64 lanes, in every lane
__device__ __forceinline__ double wave_largest(double a) {
  a = fmax(a, dpp64<0x111, 0xf, false>(a, a));
  a = fmax(a, dpp64<0x112, 0xf, false>(a, a));
  a = fmax(a, dpp64<0x114, 0xf, false>(a, a));
  a = fmax(a, dpp64<0x118, 0xf, false>(a, a));
  a = fmax(a, dpp64<0x142, 0xa, false>(a, a));
  a = fmax(a, dpp64<0x143, 0xc, false>(a, a));
  return lane_value(a, 63);
}
// sum over each group of four lanes, in all of them
__device__ __forceinline__ double quad_total(double a) {
  a += dpp64<0xb1, 0xf, true>(0.0, a);  // lanes 1, 0, 3, 2
  a += dpp64<0x4e, 0xf, true>(0.0, a);  // lanes 2, 3, 0, 1
  return a;
}

// ---- storage formats -------------------------------------------------------

struct __attribute__((aligned(16))) s64 { double x, y; };
struct __attribute__((aligned(8))) s32 { float x, y; };
struct __attribute__((aligned(4))) s16 { _Float16 x, y; };
struct __attribute__((aligned(4))) sbf { uint16_t x, y; };
// whether products with a field stored as S are chained (cmadd): the 16-bit formats
template <typename S>
constexpr bool chain_of = sizeof(S) == 4;

__host__ __device__ __forceinline__ float bf16_to_f32(uint16_t h) {
  uint32_t u = (uint32_t)h << 16;
  float f;
  __builtin_memcpy(&f, &u, 4);
  return f;
}

// round to nearest even; NaN stays NaN
__host__ __device__ __forceinline__ uint16_t f32_to_bf16(float f) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_bit_cast(uint16_t, (__bf16)f);  // one conversion instruction
#endif
  uint32_t u;
  __builtin_memcpy(&u, &f, 4);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

template <typename S>
struct storage_traits;

template <>
struct storage_traits<s64> {
  template <typename T>
  __device__ static __forceinline__ cplx<T> load(const s64& s) { return {(T)s.x, (T)s.y}; }
  template <typename T>
  __device__ static __forceinline__ s64 store(cplx<T> c) { return s64{(double)c.re, (double)c.im}; }
};
template <>
struct storage_traits<s32> {
  template <typename T>
  __device__ static __forceinline__ cplx<T> load(const s32& s) { return {(T)s.x, (T)s.y}; }
  template <typename T>
  __device__ static __forceinline__ s32 store(cplx<T> c) { return s32{(float)c.re, (float)c.im}; }
};
template <>
struct storage_traits<s16> {
  template <typename T>
  __device__ static __forceinline__ cplx<T> load(const s16& s) { return {(T)(float)s.x, (T)(float)s.y}; }
  template <typename T>
  __device__ static __forceinline__ s16 store(cplx<T> c) { return s16{(_Float16)(float)c.re, (_Float16)(float)c.im}; }
};
template <>
struct storage_traits<sbf> {
  template <typename T>
  __device__ static __forceinline__ cplx<T> load(const sbf& s) { return {(T)bf16_to_f32(s.x), (T)bf16_to_f32(s.y)}; }
  template <typename T>
  __device__ static __forceinline__ sbf store(cplx<T> c) { return sbf{f32_to_bf16((float)c.re), f32_to_bf16((float)c.im)}; }
};

template <typename T, typename S>
__device__ __forceinline__ cplx<T> ld(const S* p) { return storage_traits<S>::template load<T>(*p); }

// Streaming (non-temporal) load and store of one complex pair: for data read
// or written once per kernel, so that it does not evict reused data from
// the caches. The pair moves as one vector of its own size.
template <int BYTES> struct nt_vec;
template <> struct nt_vec<16> { typedef double type __attribute__((ext_vector_type(2))); };
template <> struct nt_vec<8> { typedef float type __attribute__((ext_vector_type(2))); };
template <> struct nt_vec<4> { typedef uint32_t type; };

template <typename S>
__device__ __forceinline__ S ld_nt_raw(const S* p) {
  using V = typename nt_vec<sizeof(S)>::type;
  const V v = __builtin_nontemporal_load(reinterpret_cast<const V*>(p));
  S s;
  __builtin_memcpy(&s, &v, sizeof(S));
  return s;
}
template <typename T, typename S>
__device__ __forceinline__ cplx<T> ld_nt(const S* p) { return storage_traits<S>::template load<T>(ld_nt_raw(p)); }
template <typename T, typename S>
__device__ __forceinline__ void st_nt(S* p, cplx<T> c) {
  using V = typename nt_vec<sizeof(S)>::type;
  const S s = storage_traits<S>::template store<T>(c);
  V v;
  __builtin_memcpy(&v, &s, sizeof(S));
  __builtin_nontemporal_store(v, reinterpret_cast<V*>(p));
}
template <typename T, typename S>
__device__ __forceinline__ void st(S* p, cplx<T> c) { *p = storage_traits<S>::template store<T>(c); }

}  // namespace dw
