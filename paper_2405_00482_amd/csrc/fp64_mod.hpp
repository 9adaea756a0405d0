// Exact modular arithmetic on binary64 for primes q < 2^48 (gfx950 VALU).
//
// Residues are integers held exactly in IEEE-754 binary64 (|x| < 2^53).  On
// CDNA4 the FP64 FMA and round-to-integer instructions issue at full rate,
// while a 64x64-bit integer product costs many 32-bit multiply steps, so the
// ring arithmetic of RNS-CKKS is carried out with this exact scheme:
//
//   h = a*b (rounded), l = fma(a, b, -h)          =>  a*b = h + l exactly
//   k = rint(h * (1/q))                           (quotient estimate)
//   r = fma(-k, q, h) + l                         =>  r = a*b - k*q exactly
//
// fma(-k, q, h) is exact because its result is an integer of magnitude below
// 2^53, and r + l is exact for the same reason.  The quotient estimate has
// relative error below 3 * 2^-53, so with |a*b/q| < 2^50 (e.g. |a| <= 2^51,
// |b| <= q/2 + 1) k is within 0.875 of a*b/q and |r| < q.  Every function
// states the input range it needs and the output range it gives.
// Compile with -ffp-contract=off: contraction would change h and break the
// identity a*b = h + l.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pvfl {

struct ModQ {
  double q;     // the prime, exact
  double qinv;  // 1/q rounded to nearest
};

// a*b mod q as some representative r with |r| < q.
// Needs |a*b/q| < 2^50 (e.g. |a| <= 4q, |b| <= q/2 + 1).
__device__ __forceinline__ double mulmod(double a, double b, ModQ m) {
  double h = a * b;
  double l = __builtin_fma(a, b, -h);
  double k = __builtin_rint(h * m.qinv);
  double r = __builtin_fma(-k, m.q, h);
  return r + l;
}

// Sums of products with one reduction.  The pair (hi, lo) holds an exact sum
// of integer products a*b: hi lives in one binade [2^e, 2^(e+1)) around an
// offset C that is a multiple of q, so that every product is rounded to the
// same grid 2^(e-52),
//   h' = fma(a, b, hi),   lo += fma(a, b, hi - h'),   hi = h'
// where hi - h' is exact (a multiple of the grid, below 2^53 of its steps) and
// so is the rounding error fma(a, b, hi - h') (an integer of magnitude <=
// 2^(e-53)).  Four operations for a product and its sum instead of the seven
// of mulmod and an addition, plus one acc_fold for the whole sum.
// acc_offset(q, x): C for sums of magnitude below 0.43 * 2^(2b + x), where
// 2^b is the power of two above q.  C/2^e lies in [1.43, 1.5], hence the 0.43.
__device__ __forceinline__ double acc_offset(double q, int x) {
  const int b = __builtin_amdgcn_frexp_exp(q);
  int e = 2 * b + x;
  if (e < 52) e = 52;  // the grid stays at whole numbers, so that C is a multiple of q
  const double kappa = __builtin_trunc(6755399441055744.0 / q);  // 1.5 * 2^52 / q
  return __builtin_ldexp(kappa * q, e - 52);
}
__device__ __forceinline__ void acc_first(double a, double b, double c, double& hi, double& lo) {
  hi = __builtin_fma(a, b, c);
  lo = __builtin_fma(a, b, c - hi);
}
__device__ __forceinline__ void acc_mac(double a, double b, double& hi, double& lo) {
  const double h = __builtin_fma(a, b, hi);
  lo += __builtin_fma(a, b, hi - h);
  hi = h;
}
// hi + lo mod q.  The quotient estimate is within 0.5 + |hi/q| 2^-52 of hi/q,
// so the result's magnitude is below (0.5 + 2^(e+1-52)/q) q + |lo|.
__device__ __forceinline__ double acc_fold(double hi, double lo, ModQ m) {
  const double k = __builtin_rint(hi * m.qinv);
  return __builtin_fma(-k, m.q, hi) + lo;
}

// centred representative, |r| <= (q+1)/2, for any integer |x| < 2^53.
__device__ __forceinline__ double reduce(double x, ModQ m) {
  double k = __builtin_rint(x * m.qinv);
  return __builtin_fma(-k, m.q, x);
}

// least non-negative residue in [0, q), for any integer |x| < 2^52.
__device__ __forceinline__ double canon(double x, ModQ m) {
  double r = reduce(x, m);
  r = (r < 0.0) ? r + m.q : r;
  return (r >= m.q) ? r - m.q : r;
}

// u64 in [0, 2^52) <-> binary64, two instructions each way.
__device__ __forceinline__ double u64_to_f64(uint64_t x) {
  return __longlong_as_double((long long)(x | 0x4330000000000000ull)) - 4503599627370496.0;
}
__device__ __forceinline__ uint64_t f64_to_u64(double c) {  // c integer in [0, 2^52)
  return (uint64_t)__double_as_longlong(c + 4503599627370496.0) & 0x000FFFFFFFFFFFFFull;
}

// signed 64-bit integer -> centred residue (|m| may be up to 2^63).
__device__ __forceinline__ double i64_to_res(int64_t v, ModQ m, double two32_mod) {
  // v = hi * 2^32 + lo with lo in [0, 2^32): both parts exact in binary64
  int64_t hi = v >> 32;
  double lo = (double)(uint32_t)(v & 0xffffffffll);
  double h = reduce((double)hi, m);
  double t = mulmod(h, two32_mod, m);
  return reduce(t + lo, m);
}

}  // namespace pvfl
