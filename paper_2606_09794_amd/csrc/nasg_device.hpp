// Device-side building blocks of the NASGabor / SH-3 evaluators (gfx950).
//
// - storage decode for float32 / bfloat16 lobe parameters, and the
//   nontemporal (streaming) accesses for data used once,
// - reductions over the `P` consecutive lanes that share a primitive, done
//   with DPP row operations (no LDS, no atomics, fixed order),
// - the per-lobe normaliser (Section 5.1) and its log-derivatives, in FP64
//   and, for the range of lam and lam (1 + a) where nothing cancels badly,
//   in FP32.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nasg {

constexpr double kPi = 3.141592653589793238462643383279502884;
constexpr double kInvTwoPi = 0.159154943091895335768883763372514362;

// ---------------------------------------------------------------- storage
// Data that a launch touches once is accessed nontemporally: the streaming
// cache policy keeps it from displacing what is still to be reused (the
// cameras, the log table). The appearance kernels do so in their streaming
// flavour (ONCE), used where it is safe and pays: one lane per primitive, so
// that a wave's access covers whole cache lines (with P lanes a wave covers
// part of a line, e.g. 4 x 64/P bytes of a colour-weight row, its neighbour
// the rest, and a streamed line can be gone before the second part is read
// or be written out twice), and a launch that reads every lobe record and
// writes every output once (all views in one chunk, no accumulation onto
// earlier results; otherwise later chunks, or the accumulating caller's next
// launch, read the same data again and it should stay cached).
typedef float f32x4_nt __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_nt __attribute__((ext_vector_type(2)));

template <class T>
__device__ inline T load_once(const T* p) {
  return __builtin_nontemporal_load(p);
}
template <class T>
__device__ inline void store_once(T v, T* p) {
  __builtin_nontemporal_store(v, p);
}
template <bool NT, class T>
__device__ inline T load_if(const T* p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  return *p;
}
template <bool NT, class T>
__device__ inline void store_if(T v, T* p) {
  if constexpr (NT) {
    __builtin_nontemporal_store(v, p);
  } else {
    *p = v;
  }
}

template <bool BF16>
struct Store;

template <>
struct Store<false> {
  using Raw4 = f32x4_nt;
  using Raw1 = float;
  __device__ static inline float4 wide(Raw4 v) { return make_float4(v.x, v.y, v.z, v.w); }
  __device__ static inline float wide(Raw1 v) { return v; }
  template <bool ONCE>
  __device__ static inline Raw4 raw4(const void* p, int64_t idx) {
    return load_if<ONCE>(reinterpret_cast<const Raw4*>(p) + idx);
  }
  template <bool ONCE>
  __device__ static inline Raw1 raw1(const void* p, int64_t idx) {
    return load_if<ONCE>(reinterpret_cast<const float*>(p) + idx);
  }
};

template <>
struct Store<true> {
  using Raw4 = u32x2_nt;   // four bfloat16 values packed little-endian in 8 bytes
  using Raw1 = uint16_t;
  __device__ static inline float4 wide(Raw4 u) {
    return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u),
                       __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u));
  }
  __device__ static inline float wide(Raw1 u) {
    return __uint_as_float(static_cast<uint32_t>(u) << 16);
  }
  template <bool ONCE>
  __device__ static inline Raw4 raw4(const void* p, int64_t idx) {
    return load_if<ONCE>(reinterpret_cast<const Raw4*>(p) + idx);
  }
  template <bool ONCE>
  __device__ static inline Raw1 raw1(const void* p, int64_t idx) {
    return load_if<ONCE>(reinterpret_cast<const uint16_t*>(p) + idx);
  }
};

// ---------------------------------------------------------- lane-group sums
// All-reduce over aligned groups of P consecutive lanes (P <= 16, one DPP row).
// Call only where every lane of the wavefront is active: DPP reads an
// inactive lane as zero.
// quad_perm [1,0,3,2] and [2,3,0,1] give the quad sum; row_half_mirror pairs
// the two quads of a half-row; row_mirror pairs the two half-rows.

// The neighbour's value through a DPP move with zero fill (bound_ctrl), the
// form the compiler folds into the consuming add (v_add_f32_dpp).
template <int CTRL>
__device__ inline float dpp_f(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}

template <int P>
__device__ inline float group_sum(float x) {
  static_assert(P == 1 || P == 2 || P == 4 || P == 8 || P == 16, "lanes per primitive");
  if constexpr (P >= 2) x += dpp_f<0xB1>(x);
  if constexpr (P >= 4) x += dpp_f<0x4E>(x);
  if constexpr (P >= 8) x += dpp_f<0x141>(x);
  if constexpr (P >= 16) x += dpp_f<0x140>(x);
  return x;
}

// ------------------------------------------------- FP64 envelope helpers
// The envelope exponent X = ln(p E) reaches |X| ~ 1e2 where G still matters,
// and exp amplifies an absolute error of X into a relative error of G, so X
// is formed in FP64. The helpers below are purpose-built for that: a few FP64
// fused multiply-adds each (FP64 FMA issues at the non-packed FP32 rate on
// CDNA4), relative error ~1e-13, inputs restricted to the ranges that occur.

// a * b + c as a three-address v_fma_f64. Used in the once-per-lobe code,
// where the compiler otherwise picks the two-address form with a hoisted
// coefficient as the accumulator and copies it before every step.
__device__ __forceinline__ double fma3(double a, double b, double c) {
  double d;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}

constexpr double kLn2Hi = 0.693145751953125;               // 2^-11 multiple
constexpr double kLn2Lo = 1.4286068203094172321214581765680755e-06;
constexpr double kLog2e = 1.442695040888963407359924681001892137;

// 1/x for x > 0 normal: the hardware estimate (relative error < 5e-8
// measured on gfx950) plus one Newton step (error ~ its square, ~2e-15).
__device__ inline double rcp64(double x) {
  const double y = __builtin_amdgcn_rcp(x);
  return fma(y, fma(-x, y, 1.0), y);
}

// 1/sqrt(x) and sqrt(x) for x > 0 normal: the hardware estimate and one
// Newton step, y1 = y + y (1 - x y^2)/2 (relative error ~ 1.5 times the
// square of the estimate's).
__device__ inline double rsqrt64(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(0.5 * y, e, y);
}
__device__ inline double sqrt64(double x) { return x * rsqrt64(x); }

// ---------------------------------------- envelope helpers (per lobe-view)
// Where G is above the FP32 range floor, |X| <= ~1e2. A relative error eps of
// ln kappa or of e^B then moves X by at most ~2e2 eps (the derivative of X
// with respect to ln kappa is about X / ln kappa, and e^B - 1 enters as
// 2 lam (e^B - 1) with lam (1 - e^B) <= ~50), so eps ~ 1e-10 keeps G
// relatively accurate to ~1e-8. Near kappa = 1, where that derivative grows
// to 2 lam (1 + tau) ~ 2e6, ln kappa keeps an absolute error ~1e-16.

// The path works in base 2 (log2 kappa, powers of two), so that splitting an
// exponent into integer and fraction costs a rounding and an exact difference,
// no product with log2(e) or ln 2; those constants are folded into the
// per-lobe factors.

constexpr double kLn2 = 0.693147180559945309417232121458176568;

// One bucket of the log2 table: log2(e)/c (rounded, as inv_c log2(e) times a
// rho = 1 + O(1e-16)) and -log2 of rho/c.
struct alignas(16) LogEntry {
  double inv_c;
  double l2c;
};
constexpr int kLogBits = 7;
constexpr int kLogEntries = 1 << kLogBits;

// log2 kappa for kappa in (0, 1], from a 128-entry table in LDS. kappa = m 2^e
// with m in [1/2, 1); the top seven mantissa bits of m select c (the bucket
// centre; c = 1 for the top bucket); r = (m/c - 1) log2(e) in one rounding,
// less `dkap`, log2(e) times the known rounding error of kappa itself (kappa
// as computed minus its exact value; it matters only in the top bucket, where
// r = (kappa - 1) log2(e)); |r| <= log2(e)/256 and log2 kappa = e + log2 c +
// log2(1 + r/log2(e)), the last summed to r^4 (truncation (r/log2(e))^5/5 <=
// 1.8e-13; relative to the fourth power over 5 in the top bucket, so log2
// kappa stays relatively accurate however close kappa is to 1).
__device__ inline int log_bucket(double m) {
  return (__double2hiint(m) >> (20 - kLogBits)) & (kLogEntries - 1);
}
// A constant held in a vector register the compiler cannot see through, so
// that a polynomial step with two constant operands (a coefficient times the
// variable plus a coefficient) still encodes as one fused multiply-add: the
// hardware takes at most one scalar operand besides literals, and without it
// the compiler copies the second constant into a register before every use.
__device__ __forceinline__ double vreg_const(double c) {
  double r;
  asm volatile("v_mov_b64 %0, %1" : "=v"(r) : "s"(c));
  return r;
}

// a * b + c with b or c a scalar operand (the one the encoding allows besides
// vector registers), so that no copy of a constant is made.
__device__ __forceinline__ double fma_vsv(double a, double b, double c) {
  double d;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "s"(b), "v"(c));
  return d;
}
__device__ __forceinline__ double fma_vvs(double a, double b, double c) {
  double d;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
  return d;
}

constexpr double kLog2C3 = kLn2 * kLn2 / 3.0;   // of r^3 in log2(1 + r/log2(e))
__device__ inline double log2_finish(double m, int e, const LogEntry& t, double dkap,
                                     double c3 = kLog2C3) {
  const double r = fma(m, t.inv_c, -kLog2e) - dkap;
  double p = fma_vsv(r, -0.25 * kLn2 * kLn2 * kLn2, c3);
  p = fma_vvs(p, r, -0.5 * kLn2);
  const double lp = fma(p, r * r, r);
  return static_cast<double>(e) + (t.l2c + lp);
}

// Nearest int of an integral double, saturated at the int range (the
// conversion instruction's own behaviour, spelled out so that out-of-range
// values are defined).
__device__ __forceinline__ int sat_int(double n) {
  int r;
  asm("v_cvt_i32_f64 %0, %1" : "=v"(r) : "v"(n));
  return r;
}

// 2^B and 2^B - 1 for B <= 0 on the envelope path: B = n + r exactly, |r| <=
// 1/2, 2^r - 1 = r q(r) with q the Taylor series of (2^r - 1)/r to r^7
// (relative truncation (r ln2)^8/9! <= 6e-10 at |r| = 1/2, far smaller near
// B = 0 where 2 lam (2^B - 1) is large). 2^B - 1 is formed as 2^B - 1, an
// absolute error ~1e-16. A very negative B gives 0 (n saturates).
constexpr double kLn2P2 = kLn2 * kLn2, kLn2P4 = kLn2P2 * kLn2P2;
constexpr double kExp2C8 = kLn2P4 * kLn2P4 / 40320.0;   // ln2^8 / 8!
__device__ inline void env_exp2(double B, double& eb, double& em1, double c8 = kExp2C8) {
  const double n = rint(B);
  const double r = B - n;
  double q = fma(c8, r, kLn2P4 * kLn2P2 * kLn2 / 5040.0);
  q = fma(q, r, kLn2P4 * kLn2P2 / 720.0);
  q = fma(q, r, kLn2P4 * kLn2 / 120.0);
  q = fma(q, r, kLn2P4 / 24.0);
  q = fma(q, r, kLn2P2 * kLn2 / 6.0);
  q = fma(q, r, kLn2P2 / 2.0);
  q = fma(q, r, kLn2);
  eb = ldexp(fma(r, q, 1.0), sat_int(n));
  em1 = eb - 1.0;
}

// e^B and e^B - 1 for B <= 0: B = n ln2 + r, |r| <= ln2/2, e^r - 1 = r q(r)
// with q the Taylor series of (e^r - 1)/r to r^9/10! (truncation ~3e-13).
// For |B| <= ln2/2 (n = 0) e^B - 1 is the series value r q(r) itself, so it
// keeps its relative accuracy however small B is; otherwise it is e^B - 1
// (|e^B - 1| >= 0.29 there). B below -1400 is clamped (e^-1400 underflows FP64
// to 0 either way).
template <bool THREE_ADDR = false>
__device__ inline void exp_em1(double B, double& eb, double& em1) {
  auto mad = [](double x, double y, double z) { return THREE_ADDR ? fma3(x, y, z) : fma(x, y, z); };
  B = fmax(B, -1400.0);
  const double n = rint(B * kLog2e);
  double r = fma(-n, kLn2Hi, B);
  r = fma(-n, kLn2Lo, r);
  double q = 1.0 / 3628800.0;          // 1/10!
  q = mad(q, r, 1.0 / 362880.0);
  q = mad(q, r, 1.0 / 40320.0);
  q = mad(q, r, 1.0 / 5040.0);
  q = mad(q, r, 1.0 / 720.0);
  q = mad(q, r, 1.0 / 120.0);
  q = mad(q, r, 1.0 / 24.0);
  q = mad(q, r, 1.0 / 6.0);
  q = mad(q, r, 0.5);
  q = fma(q, r, 1.0);
  eb = ldexp(fma(r, q, 1.0), static_cast<int>(n));
  em1 = n == 0.0 ? r * q : eb - 1.0;
}

// 2^y as float for y <= 0 in FP64: its nearest integer n and the exact rest
// |f| <= 1/2, then the hardware base-2 exponential of f and an exact
// power-of-two scale. Very negative y gives 2^f with n saturated far below the
// FP32 range: 0.
__device__ inline float exp2_neg(double y) {
  const double n = rint(y);
  const float p = __builtin_amdgcn_exp2f(static_cast<float>(y - n));
  return ldexpf(p, sat_int(n));
}

// Half phase of the carrier in units of pi, reduced to r in [-1/2, 1/2] (exact):
// cos(pi r) = pi v (1 + uc) and sin(pi r) = 2 r (1 + us) with v = 1/4 - r^2 formed
// as b (1 - b), b = 1/2 - |r|, so that both are relatively accurate next to their
// zeros. uc = v + O(v^2) and us = 2 v + O(v^2) are at most 0.28 and 0.58 and vanish
// at the cosine's zeros, so FP32 holds them: own Remez fits with the leading
// coefficients fixed at 1 and 2, 1.9e-9 and 1.0e-8 relative to cosine and sine,
// 3e-8 and 6e-8 at most (rms 6e-9 and 1.3e-8) with their FP32 rounding.
__device__ __forceinline__ double quarter_less_sq(double r) {
  const double b = 0.5 - fabs(r);
  return fma(-b, b, b);
}
__device__ __forceinline__ float cos_pi_u(float v) {
  float u = fmaf(v, 0.007639229607417381f, 0.06514647357787971f);
  u = fmaf(u, v, 0.35506860612312846f);
  return v * fmaf(u, v, 1.f);
}
__device__ __forceinline__ float sin_pi_u(float v) {
  float u = fmaf(v, 0.03848935620413844f, 0.2604881783097619f);
  u = fmaf(u, v, 1.0652133403459647f);
  return v * fmaf(u, v, 2.f);
}

// cos(2 pi r) in FP32 for |r| <= 1/2, r exact: the sine of 2 pi (1/4 - |r|), so that
// it is relatively accurate next to its zeros (own Remez fit, 5.3e-9 relative,
// 1.7e-7 with FP32 rounding).
__device__ inline float cos_two_pi(double r) {
  const float w = static_cast<float>(0.25 - fabs(r));
  const float z = w * w;
  float p = fmaf(z, 39.710918145200566f, -76.57499218217357f);
  p = fmaf(p, z, 81.60223124273418f);
  p = fmaf(p, z, -41.34167747839161f);
  p = fmaf(p, z, 6.283185273790786f);
  return w * p;
}

// sin(2 pi t) and cos(2 pi t) in FP64 for any t: t is reduced to the nearest
// integer and quarter turn, leaving |r| <= pi/4 for the Taylor series
// (sine to r^13, cosine to r^14; truncation below 1e-14). Scalar constants: only
// lobes with a fast carrier come here, and in vector registers the dozen would be
// kept through the lobe loops.
__device__ inline void sincos_turns(double t, double& s, double& c) {
  constexpr double kTwoPi = 6.283185307179586476925286766559005768;
  const double f = t - rint(t);
  const double qd = rint(4.0 * f);
  const double r = (f - 0.25 * qd) * kTwoPi;
  const double z = r * r;
  double ps = 1.0 / 6227020800.0;      // 1/13!
  ps = fma_vvs(ps, z, -1.0 / 39916800.0);
  ps = fma_vvs(ps, z, 1.0 / 362880.0);
  ps = fma_vvs(ps, z, -1.0 / 5040.0);
  ps = fma_vvs(ps, z, 1.0 / 120.0);
  ps = fma_vvs(ps, z, -1.0 / 6.0);
  const double sr = fma(ps * z, r, r);
  double pc = 1.0 / 87178291200.0;     // 1/14!
  pc = fma_vvs(pc, z, -1.0 / 479001600.0);
  pc = fma_vvs(pc, z, 1.0 / 3628800.0);
  pc = fma_vvs(pc, z, -1.0 / 40320.0);
  pc = fma_vvs(pc, z, 1.0 / 720.0);
  pc = fma_vvs(pc, z, -1.0 / 24.0);
  pc = fma_vvs(pc, z, 0.5);
  const double cr = fma(-pc, z, 1.0);
  const int q = static_cast<int>(qd) & 3;
  s = (q == 0) ? sr : (q == 1) ? cr : (q == 2) ? -sr : -cr;
  c = (q == 0) ? cr : (q == 1) ? -sr : (q == 2) ? -cr : sr;
}

// ------------------------------------------- activations (paper's stored values)
// They feed the lobe frame and the lobe parameters, whose errors the envelope
// amplifies by up to lam (1 + a). Polynomials are Taylor series economised on
// |r| <= ln2/2.

// e^B, B clamped to [-1400, 700] (beyond, e^B is 0 or overflows FP64 either
// way): 2^n e^r, (e^r - 1)/r to degree 10 (error 2.5e-17).
__device__ inline double exp_full(double B) {
  B = fmin(fmax(B, -1400.0), 700.0);
  const double n = rint(B * kLog2e);
  double r = fma(-n, kLn2Hi, B);
  r = fma(-n, kLn2Lo, r);
  double q = 2.5100376916201744e-08;
  q = fma_vvs(q, r, 2.761379705043833e-07);
  q = fma_vvs(q, r, 2.7557268477824867e-06);
  q = fma_vvs(q, r, 2.4801536406057835e-05);
  q = fma_vvs(q, r, 0.00019841269863042323);
  q = fma_vvs(q, r, 0.0013888888905873068);
  q = fma_vvs(q, r, 0.008333333333330063);
  q = fma_vvs(q, r, 0.041666666666651364);
  q = fma_vvs(q, r, 0.16666666666666669);
  q = fma(q, r, 0.5);
  q = fma(q, r, 1.0);
  return ldexp(fma(r, q, 1.0), static_cast<int>(n));
}

// e^B = num / den for B <= 0 (clamped to -1400): with c = r coth(r/2), even in
// r, e^r = (c + r)/(c - r), so that the one division of tanh, sech and the
// logistic serves the exponential too. c to r^10 (error 6e-18).
__device__ inline void exp_frac(double B, double& num, double& den) {
  B = fmax(B, -1400.0);
  const double n = rint(B * kLog2e);
  double r = fma(-n, kLn2Hi, B);
  r = fma(-n, kLn2Lo, r);
  const double z = r * r;
  double c = fma_vvs(4.143774697636149e-08, z, -1.653406021796854e-06);
  c = fma_vvs(c, z, 6.613756471747488e-05);
  c = fma_vvs(c, z, -0.002777777777756467);
  c = fma_vvs(c, z, 0.1666666666666666);
  c = fma(c, z, 2.0);
  num = ldexp(c + r, static_cast<int>(n));
  den = c - r;
}

// tanh u and sech u (= +sqrt(1 - tanh^2 u)) from q = e^{-|u|} = num/den:
// tanh|u| = (1 - q)(1 + q)/(1 + q^2), sech u = 2 q/(1 + q^2); no overflow.
__device__ inline void tanh_sech(double u, double& t, double& s) {
  double num, den;
  exp_frac(-fabs(u), num, den);
  const double inv = rcp64(fma(num, num, den * den));
  t = copysign((den - num) * (den + num) * inv, u);
  s = 2.0 * num * den * inv;
}

// tanh u and its derivative sech^2 u, for a value rounded to FP32.
__device__ inline void tanh_f32(double u, float& t, float& dt) {
  double num, den;
  exp_frac(-2.0 * fabs(u), num, den);
  const double inv = rcp64(den + num);
  t = static_cast<float>(copysign((den - num) * inv, u));
  dt = static_cast<float>(4.0 * (num * inv) * (den * inv));
}

// k = 20 (tanh u + 1) = 40/(1 + e^{-2u}) and dk/du = 20 sech^2 u
// = 80 t/(1 + t)^2 with t = e^{-2|u|} (no overflow, no cancellation).
__device__ inline void k_activation(double u, double& k, float& dk) {
  double num, den;
  exp_frac(-2.0 * fabs(u), num, den);
  const double inv = rcp64(den + num);
  k = 40.0 * (u >= 0.0 ? den : num) * inv;
  dk = static_cast<float>(80.0 * (num * inv) * (den * inv));
}

// ------------------------------------------------------------- normaliser

struct LobeNorm {
  float n;        // normaliser value
  float dl, da;   // d ln N / d lambda, d ln N / d a
  float dk;       // d ln N / d k, and (pi/2) d ln N / d zeta (both zero for the
  double dz;      // NASG normaliser), the latter in FP64: see lobe_norm_f32
};

// Psi(Lam, k) = 2 Lam e^{-Lam} S(r) / (1 - e^{-2 Lam}) of the closed-form
// integral (Section 5.1), r = Lam^2 - k^2, S(r) = sinh(sqrt r)/sqrt r (continued
// to r < 0 as sin(sqrt -r)/sqrt -r), and its partials in Lam and k.
//
// r > 1: with s = sqrt r and delta = Lam - s = k^2 / (Lam + s),
//   Psi = (Lam/s) e^{-delta} (1 - e^{-2s}) / (1 - e^{-2 Lam}),
//   d ln Psi/dLam = -k^2/(Lam s^2) + (delta/s)(1 + 2g) + 2 (g - g_Lam),
//   d ln Psi/dk   = (k/s)(1/s - 1 - 2g),    g = e^{-2s}/(1 - e^{-2s}),
//   g - g_Lam = -e^{-2s} expm1(-2 delta) / ((1 - e^{-2s})(1 - e^{-2 Lam})):
//   every term vanishes with k instead of cancelling (Psi = 1 and both
//   partials are 0 at k = 0), which keeps the partials relatively accurate
//   where 1/(1 + cos(zeta) Psi) amplifies them (zeta near pi).
// |r| <= 1: power series of S and S' (to r^9/19!); r < -1: sin t / t with
//   t = sqrt(-r); then Psi and its partials from F = e^{-Lam} S and
//   F' = e^{-Lam} S' directly (no small-k cancellation there: k is close to
//   Lam or above it).
// The two exponentials are shared by the branches: e^{-delta} or e^{-Lam},
// and e^{-2s} or e^{-2 Lam}.
__device__ inline void psi_partials(double L, double k, double iL, double& psi,
                                    double& dpsi_dL, double& dpsi_dk) {
  const double r = (L - k) * (L + k);
  const bool hyp = r > 1.0;
  const double ar = fmax(fabs(r), 1.0);
  const double is = rsqrt64(ar);                   // 1/s, s = sqrt|r| (where |r| > 1)
  const double s = ar * is;
  const double delta = k * k * rcp64(L + s);
  double e1, e1m1, e2, e2m1;
  exp_em1<true>(hyp ? -delta : -L, e1, e1m1);      // e^{-delta} or e^{-Lam}
  exp_em1<true>(hyp ? -2.0 * s : -2.0 * L, e2, e2m1);   // e^{-2s} or e^{-2 Lam}
  if (hyp) {
    const double Ds = -e2m1;                       // 1 - e^{-2s}
    const double e2L = e2 * e1 * e1;               // e^{-2 Lam} = e^{-2s} e^{-2 delta}
    const double DL = 1.0 - e2L;
    const double iDD = rcp64(Ds * DL);
    const double g = e2 * DL * iDD;
    psi = L * is * e1 * Ds * Ds * iDD;
    const double dlnL = fma(-k * k * iL, is * is, delta * is * fma(2.0, g, 1.0)) -
                        2.0 * e2 * e1m1 * (2.0 + e1m1) * iDD;
    const double dlnk = k * is * (is - 1.0 - 2.0 * g);
    dpsi_dL = psi * dlnL;
    dpsi_dk = psi * dlnk;
  } else {
    double F, dF;
    if (!(fabs(r) > 1.0)) {
      // 1/(2n+1)! for n = 0..9
      constexpr double c[10] = {1.0, 1.0 / 6.0, 1.0 / 120.0, 1.0 / 5040.0, 1.0 / 362880.0,
                                1.0 / 39916800.0, 1.0 / 6227020800.0, 1.0 / 1307674368000.0,
                                1.0 / 355687428096000.0, 1.0 / 121645100408832000.0};
      double sr = c[9], ds = 9.0 * c[9];
#pragma unroll
      for (int n = 8; n >= 1; --n) {
        sr = fma3(sr, r, c[n]);
        ds = fma3(ds, r, n * c[n]);
      }
      sr = fma(sr, r, c[0]);
      F = e1 * sr;
      dF = e1 * ds;
    } else {
      double sn, cs;
      sincos_turns(s * kInvTwoPi, sn, cs);
      F = e1 * sn * is;
      dF = e1 * fma(-s, cs, sn) * 0.5 * is * is * is;
    }
    const double iD = rcp64(-e2m1);                // 1 / (1 - e^{-2 Lam})
    psi = 2.0 * L * F * iD;
    const double dF_dL = fma(2.0 * L, dF, -F);
    dpsi_dL = (2.0 * F + 2.0 * L * dF_dL) * iD - 4.0 * L * F * e2 * iD * iD;
    dpsi_dk = -4.0 * L * k * dF * iD;
  }
}

// Normaliser of one lobe and the log-derivatives the backward pass needs.
// mode 0: 1 / closed-form integral (Section 5.1; the phase multiplies Psi by
//         cos zeta): I = pi (1 - e^{-2 lam}) / (lam sqrt(1+a)) B,
//         B = 1 + cos(zeta) Psi, which FP64 keeps relatively accurate down to
//         B ~ 1e-9 (zeta within ~5e-5 of pi with Psi -> 1);
// mode 1: NASG normaliser lambda sqrt(1+a) / (2 pi (1 - e^{-2 lambda})).
// UNIT: whether n comes times pi^2, the unit of the kernels' carrier.
template <bool UNIT = false>
__device__ inline LobeNorm lobe_norm(double lam, double a, double kd, double zd, int mode) {
  constexpr double unit = UNIT ? kPi * kPi : 1.0;
  double e2l, em1_2l;
  exp_em1<true>(-2.0 * lam, e2l, em1_2l);
  const double dlam = -em1_2l;                    // 1 - e^{-2 lam}, relatively accurate
  const double sq = sqrt64(1.0 + a);
  const double idl = rcp64(dlam);
  const double il = rcp64(lam);
  const double ia = rcp64(1.0 + a);
  // d/dlam ln(lam / (1 - e^{-2 lam})) = 1/lam - 2 e^{-2 lam} / (1 - e^{-2 lam})
  const double dl_base = il - 2.0 * e2l * idl;
  const double da_base = 0.5 * ia;
  LobeNorm out;
  if (mode == 1) {
    out.n = static_cast<float>(lam * sq * idl * (0.5 / kPi * unit));
    out.dl = static_cast<float>(dl_base);
    out.da = static_cast<float>(da_base);
    out.dk = 0.f;
    out.dz = 0.0;
    return out;
  }
  const double L = lam * (1.0 + a);
  double psi, dpsi_dL, dpsi_dk;
  psi_partials(L, kd, il * ia, psi, dpsi_dL, dpsi_dk);
  double sz, cz;
  sincos_turns(zd * kInvTwoPi, sz, cz);
  const double B = fma(cz, psi, 1.0);
  const double iB = rcp64(B);
  const double czB = cz * iB;
  out.n = static_cast<float>(lam * sq * idl * iB * (1.0 / kPi * unit));
  out.dl = static_cast<float>(dl_base - czB * dpsi_dL * (1.0 + a));
  out.da = static_cast<float>(da_base - czB * dpsi_dL * lam);
  out.dk = static_cast<float>(-czB * dpsi_dk);
  out.dz = (0.5 * kPi) * (sz * psi * iB);
  return out;
}

// ------------------------------------------------ normaliser, FP32 fast path
// The same normaliser and log-derivatives in FP32 for lam >= 1/2 and
// Lam = lam (1 + a) >= 3/2, the range every lobe of a trained model or a
// log-uniform draw in [1, 1e3] falls in; smaller lam or Lam take the FP64
// code above. In that range nothing below cancels by more than a factor of a
// few, so FP32 keeps N relatively accurate to ~1e-6 and the log-derivatives
// to ~1e-6 of their size. That is not enough for the one in zeta: where Psi is
// near 1 (a carrier that hardly turns across the lobe) it cancels the carrier's
// own d ln c/d zeta = -tan(theta/2), by factors of thirty and more, and so it is
// formed in FP64 as tan(zeta/2) (1 - rho), rho = (1 - Psi)/B, whose error is that
// of rho alone (rho >= 1/2, where 1 - rho would cancel: no such cancellation
// there, and the FP32 form serves). The others:
// - 1 - e^{-2 lam} >= 0.63 and d/dlam ln(lam / (1 - e^{-2 lam})) >= 0.84;
// - B = 1 + cos(zeta) Psi is formed as (1 - Psi) + Psi (1 + cos zeta), with
//   sin zeta, cos zeta and 1 + cos zeta each relatively accurate (the phase
//   is reduced in FP64): for 0 <= Psi <= 1 two terms of one sign, for Psi < 0
//   (|Psi| < 0.22) B >= 0.78, so B keeps its relative accuracy as zeta -> pi
//   and k -> 0 drive it to 0, and the k and zeta log-derivatives keep theirs
//   next to the zeros of cos zeta and sin zeta;
// - where Lam^2 - k^2 > 1, with s, delta, g as in psi_partials and
//   m = 1 - e^{-delta} (relatively accurate),
//     1 - Psi = [m (1 + e^{-delta} e^{-2s}) - delta e^{-delta} (1 - e^{-2s})/s]
//               / (1 - e^{-2 Lam}),
//   whose two terms (~delta and ~delta/s) differ by at least a factor s >= 3/2
//   for small k, and the log-derivatives are those of psi_partials with
//   1 - e^{-2 delta} = m (2 - m): every term vanishes with k;
// - elsewhere (|Lam^2 - k^2| <= 1, or k^2 > Lam^2 + 1) k >= 1.1, Psi <= 0.83,
//   and Psi and its partials come from e^{-Lam} S(r) and e^{-Lam} S'(r) as in
//   psi_partials: S and S' by their series to r^6/13! (both positive there),
//   or, where k^2 > Lam^2 + 1, sin t / t and its derivative in FP64, since
//   they cross zero and the k and zeta gradients scale with them.

__device__ inline float exp_f(float x) { return __builtin_amdgcn_exp2f(x * 1.44269504088896341f); }

// e^x - 1 for x <= 0, relatively accurate: the Taylor series to x^8/8! for
// x > -1/2 (truncation below 1e-8 relative), e^x - 1 below (|e^x - 1| >= 0.39).
__device__ inline float expm1_neg_f(float x) {
  float p = 1.f / 40320.f;
  p = fmaf(p, x, 1.f / 5040.f);
  p = fmaf(p, x, 1.f / 720.f);
  p = fmaf(p, x, 1.f / 120.f);
  p = fmaf(p, x, 1.f / 24.f);
  p = fmaf(p, x, 1.f / 6.f);
  p = fmaf(p, x, 0.5f);
  p = fmaf(p, x, 1.f);
  return x > -0.5f ? p * x : exp_f(x) - 1.f;
}

// lam, a, k as the caller holds them (FP64 for the paper's activated values),
// rounded to FP32 here except where the sine branch needs them exact.
template <bool UNIT>
__device__ inline LobeNorm lobe_norm_f32(double lamd, double ad, double kd, double zd, int mode) {
  constexpr double unit = UNIT ? kPi * kPi : 1.0;
  const float lam = static_cast<float>(lamd), a = static_cast<float>(ad), k = static_cast<float>(kd);
  const float e2l = exp_f(-2.f * lam);
  const float idl = __builtin_amdgcn_rcpf(1.f - e2l);
  const float il = __builtin_amdgcn_rcpf(lam);
  const float opa = 1.f + a;
  const float ia = __builtin_amdgcn_rcpf(opa);
  const float sq = opa * __builtin_amdgcn_rsqf(opa);
  const float dl_base = il - 2.f * e2l * idl;
  const float da_base = 0.5f * ia;
  LobeNorm out;
  if (mode == 1) {
    out.n = lam * sq * idl * static_cast<float>(0.5 / kPi * unit);
    out.dl = dl_base;
    out.da = da_base;
    out.dk = 0.f;
    out.dz = 0.0;
    return out;
  }
  const float L = lam * opa;
  const float r = (L - k) * (L + k);
  const bool hyp = r > 1.f;
  const float ar = fmaxf(fabsf(r), 1.f);
  const float is = __builtin_amdgcn_rsqf(ar);          // 1/s
  const float s = ar * is;
  const float delta = k * k * __builtin_amdgcn_rcpf(L + s);
  const float e1 = exp_f(hyp ? -delta : -L);           // e^{-delta} or e^{-Lam}
  const float e2 = exp_f(hyp ? -2.f * s : -2.f * L);   // e^{-2s} or e^{-2 Lam}
  float psi, om, dPL, dPk;
  if (hyp) {
    const float Ds = 1.f - e2;
    const float iDs = __builtin_amdgcn_rcpf(Ds);
    const float iDL = __builtin_amdgcn_rcpf(1.f - e2 * e1 * e1);
    const float g = e2 * iDs;
    psi = L * is * e1 * Ds * iDL;
    const float m = -expm1_neg_f(-delta);              // 1 - e^{-delta}
    om = (m * fmaf(e1, e2, 1.f) - delta * e1 * Ds * is) * iDL;
    const float dlnL = fmaf(-k * k * il * ia, is * is, delta * is * fmaf(2.f, g, 1.f)) +
                       2.f * e2 * (m * (2.f - m)) * iDL * iDs;
    const float dlnk = k * is * (is - 1.f - 2.f * g);
    dPL = psi * dlnL;
    dPk = psi * dlnk;
  } else {
    float S, dS;
    if (!(fabsf(r) > 1.f)) {
      // S(r) = sum r^n/(2n+1)! and S'(r), n <= 6
      S = 1.f / 6227020800.f;
      dS = 6.f / 6227020800.f;
      S = fmaf(S, r, 1.f / 39916800.f);
      dS = fmaf(dS, r, 5.f / 39916800.f);
      S = fmaf(S, r, 1.f / 362880.f);
      dS = fmaf(dS, r, 4.f / 362880.f);
      S = fmaf(S, r, 1.f / 5040.f);
      dS = fmaf(dS, r, 3.f / 5040.f);
      S = fmaf(S, r, 1.f / 120.f);
      dS = fmaf(dS, r, 2.f / 120.f);
      S = fmaf(S, r, 1.f / 6.f);
      dS = fmaf(dS, r, 1.f / 6.f);
      S = fmaf(S, r, 1.f);
    } else {
      // sin t / t and its derivative in r, t = sqrt(k^2 - Lam^2), in FP64:
      // S'(r) = (sin t - t cos t)/(2 t^3) and S itself cross zero, and both
      // must stay relatively accurate there (the k and zeta gradients scale
      // with them); FP32 rounding of t alone would move them by ~1e-6 t
      const double Ld = lamd * (1.0 + ad);
      const double t2 = (kd - Ld) * (kd + Ld);
      const double it = rsqrt64(t2);
      const double t = t2 * it;
      double sn, cs;
      sincos_turns(t * kInvTwoPi, sn, cs);
      S = static_cast<float>(sn * it);
      dS = static_cast<float>(fma(-t, cs, sn) * (0.5 * it * it * it));
    }
    const float F = e1 * S;
    const float dF = e1 * dS;
    const float iD = __builtin_amdgcn_rcpf(1.f - e2);
    psi = 2.f * L * F * iD;
    om = 1.f - psi;
    const float dF_dL = fmaf(2.f * L, dF, -F);
    dPL = fmaf(2.f, F, 2.f * L * dF_dL) * iD - 4.f * L * F * e2 * iD * iD;
    dPk = -4.f * L * k * dF * iD;
  }
  // zeta, reduced as the carrier's half phase: its cosine from that offset, sin zeta
  // and 1 + cos zeta from the half angle's sine and cosine
  const double zh = zd * kInvTwoPi;
  const double r0 = zh - rint(zh);
  const double v0 = quarter_less_sq(r0);
  const float vf = static_cast<float>(v0);
  const float uc = cos_pi_u(vf), us = sin_pi_u(vf);
  const double ch = fma(v0, static_cast<double>(uc), v0);
  const double sh = fma(r0, static_cast<double>(us), r0);
  const float cz = cos_two_pi(r0);
  const float opc = static_cast<float>((2.0 * kPi * kPi) * (ch * ch));
  const float B = fmaf(psi, opc, om);
  const float iB = __builtin_amdgcn_rcpf(B);
  const float czB = cz * iB;
  out.n = lam * sq * idl * iB * static_cast<float>(1.0 / kPi * unit);
  out.dl = dl_base - czB * dPL * opa;
  out.da = da_base - czB * dPL * lam;
  out.dk = -czB * dPk;
  // d ln N/d zeta = sin(zeta) Psi/B = tan(zeta/2) (1 - (1 - Psi)/B)
  const float rho = om * iB;
  // (sh/ch = (pi/2) tan(zeta/2), 4 pi sh ch = sin zeta)
  out.dz = rho < 0.5f ? sh * rcp64(ch) * (1.0 - static_cast<double>(rho))
                      : (2.0 * kPi * kPi) * (sh * ch) * static_cast<double>(psi * iB);
  return out;
}

// The FP64 normaliser as a called function: it runs only for the rare lobes
// outside the FP32 range, and kept out of line its FP64 temporaries do not
// count against the calling kernel's register budget.
template <bool UNIT>
__device__ __noinline__ LobeNorm lobe_norm_outlined(double lam, double a, double kd, double zd,
                                                    int mode) {
  return lobe_norm<UNIT>(lam, a, kd, zd, mode);
}

// The normaliser by the FP32 path where it applies, by the FP64 one elsewhere.
template <bool UNIT>
__device__ inline LobeNorm lobe_norm_any(double lam, double a, double kd, double zd, int mode) {
  const float lf = static_cast<float>(lam), af = static_cast<float>(a);
  if (lf >= 0.5f && lf * (1.f + af) >= 1.5f) return lobe_norm_f32<UNIT>(lam, a, kd, zd, mode);
  return lobe_norm_outlined<UNIT>(lam, a, kd, zd, mode);
}

}  // namespace nasg
