// Shared device/host helpers of the mpsl library: complex arithmetic on
// double2/float2 storage, status handling.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <string>

#include "../../include/mpsl.h"

namespace mpsl {

// Storage type of one complex number in precision T.
template <typename T> struct cvec;
template <> struct cvec<double> { using type = double2; };
template <> struct cvec<float> { using type = float2; };
template <typename T> using cv_t = typename cvec<T>::type;

// Register-side complex number.
template <typename T> struct cx {
  T re, im;
};

template <typename T> __host__ __device__ inline cx<T> mk(T r, T i) { return cx<T>{r, i}; }
template <typename T> __host__ __device__ inline cx<T> ld(const cv_t<T> &v) { return cx<T>{v.x, v.y}; }
template <typename T> __host__ __device__ inline cv_t<T> st(const cx<T> &v) {
  cv_t<T> o;
  o.x = v.re;
  o.y = v.im;
  return o;
}
template <typename T> __host__ __device__ inline cx<T> operator+(cx<T> a, cx<T> b) { return {a.re + b.re, a.im + b.im}; }
template <typename T> __host__ __device__ inline cx<T> operator-(cx<T> a, cx<T> b) { return {a.re - b.re, a.im - b.im}; }
template <typename T> __host__ __device__ inline cx<T> operator*(cx<T> a, cx<T> b) {
  return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
template <typename T> __host__ __device__ inline cx<T> operator*(T s, cx<T> a) { return {s * a.re, s * a.im}; }
template <typename T> __host__ __device__ inline cx<T> conj(cx<T> a) { return {a.re, -a.im}; }
// acc += a * b
template <typename T> __host__ __device__ inline void cmac(cx<T> &acc, cx<T> a, cx<T> b) {
  acc.re = fma(a.re, b.re, acc.re);
  acc.re = fma(-a.im, b.im, acc.re);
  acc.im = fma(a.re, b.im, acc.im);
  acc.im = fma(a.im, b.re, acc.im);
}

// sin and cos of r, |r| <= pi / 4, by their Taylor series (terms up to r^9
// and r^10 in FP32, r^17 and r^18 in FP64: the first term left out is at most
// 1.8e-9 and 1.2e-10 in FP32, 8.4e-20 and 3.3e-21 in FP64).
__device__ inline void sincos_quarter(float r, float &s, float &c) {
  const float r2 = r * r;
  s = r * (1.0f + r2 * (-1.0f / 6 + r2 * (1.0f / 120 + r2 * (-1.0f / 5040 + r2 * (1.0f / 362880)))));
  c = 1.0f + r2 * (-0.5f + r2 * (1.0f / 24 + r2 * (-1.0f / 720 + r2 * (1.0f / 40320 + r2 * (-1.0f / 3628800)))));
}
__device__ inline void sincos_quarter(double r, double &s, double &c) {
  const double r2 = r * r;
  double ps = 1.0 / 355687428096000.0, pc = 1.0 / 6402373705728000.0;  // 1/17!, 1/18!
  ps = 1.0 / 1307674368000.0 - r2 * ps;   // 1/15!
  ps = 1.0 / 6227020800.0 - r2 * ps;      // 1/13!
  ps = 1.0 / 39916800.0 - r2 * ps;        // 1/11!
  ps = 1.0 / 362880.0 - r2 * ps;          // 1/9!
  ps = 1.0 / 5040.0 - r2 * ps;
  ps = 1.0 / 120.0 - r2 * ps;
  ps = 1.0 / 6.0 - r2 * ps;
  s = r * (1.0 - r2 * ps);
  pc = 1.0 / 20922789888000.0 - r2 * pc;  // 1/16!
  pc = 1.0 / 87178291200.0 - r2 * pc;     // 1/14!
  pc = 1.0 / 479001600.0 - r2 * pc;       // 1/12!
  pc = 1.0 / 3628800.0 - r2 * pc;         // 1/10!
  pc = 1.0 / 40320.0 - r2 * pc;
  pc = 1.0 / 720.0 - r2 * pc;
  pc = 1.0 / 24.0 - r2 * pc;
  pc = 0.5 - r2 * pc;
  c = 1.0 - r2 * pc;
}

// x with its sign bit flipped where s = 2^31 (s = 0: unchanged).
__device__ inline float flip_sign(float x, unsigned s) { return __uint_as_float(__float_as_uint(x) ^ s); }
__device__ inline double flip_sign(double x, unsigned s) {
  return __hiloint2double(static_cast<int>(static_cast<unsigned>(__double2hiint(x)) ^ s), __double2loint(x));
}

// e^{a + i b} in the matvec precision.  The phase b (up to |lambda| times the
// strip width) is reduced in FP64 to r = b - k pi/2, |r| <= pi/4, with a
// two-term pi/2 (Cody and Waite); sin and cos of r come from the series
// above in T and are rotated by k quarter turns; exp(a) in T.  In FP32 the
// relative error is ~2e-7 (the result is rounded to FP32 anyway); in FP64 a
// few units in the last place.  No large-argument path: every lane runs the
// same instructions.
template <typename T> __device__ inline cx<T> cexpT(double a, double b) {
  constexpr double kHalfPiHi = 1.5707963267948966, kHalfPiLo = 6.123233995736766e-17;
  constexpr double kRound = 6755399441055744.0;  // 1.5 2^52: the sum's low bits are the nearest integer
  const double km = fma(b, 0.6366197723675814, kRound), k = km - kRound;
  const double r = fma(-k, kHalfPiLo, fma(-k, kHalfPiHi, b));
  T sr, cr;
  sincos_quarter(static_cast<T>(r), sr, cr);
  const unsigned qd = static_cast<unsigned>(__double2loint(km));
  const T sn = flip_sign((qd & 1) ? cr : sr, (qd & 2) << 30);
  const T cs = flip_sign((qd & 1) ? sr : cr, ((qd + 1) & 2) << 30);
  const T e = exp(static_cast<T>(a));
  return {e * cs, e * sn};
}

// Orders on the matrix cores and on the vector units: full 16-order tiles go
// to the MFMAs; a remainder of one or two orders (p = 16: 33 = 2 x 16 + 1,
// p = 8: 17 = 16 + 1) is accumulated on the vector units instead of a tile of
// which it would fill at most 2/16; a longer remainder gets a padded tile.
template <int P> struct OrderSplit {
  static constexpr int NF = P / 16;
  static constexpr int REM = P - 16 * NF;
  static constexpr bool VALU_REM = REM > 0 && REM <= 2;
  static constexpr int NT = VALU_REM ? NF : (P + 15) / 16;  // MFMA tiles
  static constexpr int NV = VALU_REM ? REM : 0;             // vector-unit orders, slots 16 NT ..
};

// One 16x16x4 matrix-core multiply-accumulate in precision T, D = A B + C.
// Operand layout (both precisions): lane i supplies A[i % 16][i / 16] and
// B[i / 16][i % 16]; result register j of lane i is D[row(i, j)][i % 16],
// row = 4 (i / 16) + j for f32 and i / 16 + 4 j for f64 (measured on gfx950
// with one-hot operands).
template <typename T> struct mfma4;
template <> struct mfma4<float> {
  typedef float v4 __attribute__((ext_vector_type(4)));
  static __device__ inline v4 mac(float a, float b, v4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  static __device__ inline int row(int lane, int j) { return 4 * (lane >> 4) + j; }
};
template <> struct mfma4<double> {
  typedef double v4 __attribute__((ext_vector_type(4)));
  static __device__ inline v4 mac(double a, double b, v4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
  static __device__ inline int row(int lane, int j) { return (lane >> 4) + 4 * j; }
};

}  // namespace mpsl

#define MPSL_HIP_TRY(ctx, call)                                                              \
  do {                                                                                       \
    hipError_t e_ = (call);                                                                  \
    if (e_ != hipSuccess) {                                                                  \
      (ctx)->err = std::string("HIP error in ") + #call + ": " + hipGetErrorString(e_);      \
      return MPSL_EHIP;                                                                      \
    }                                                                                        \
  } while (0)
