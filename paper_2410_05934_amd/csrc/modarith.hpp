// modarith.hpp -- exact modular arithmetic for the gfx950 NTT kernels.
//
// Three arithmetic classes, chosen per modulus when a plan is built:
//
//   ArF64S  q < 2^32, 32-bit words.  Values are held in fp64 registers as
//           exact integers.  A product x*w is split exactly into h + l with
//           one multiply and one FMA; the quotient c = rint(h/q) is
//           estimated in fp64 and r = (h - c*q) + l is then exact (all terms
//           are integers below 2^53).  Inputs may be lazily reduced: for
//           q < 2^32 the bounds stay far below 2^53 for any N <= 2^16, so no
//           intermediate reduction is needed inside a transform.
//   ArF64L  q < 2^50 - 2^10, 64-bit words, the same fp64 scheme.  A group of
//           up to four butterfly stages keeps every value below 2^53 when its
//           inputs are centred (|x| <= q/2 + 2); a centred reduction
//           x - q*rint(x/q) follows every such group.
//   ArI64   q < 2^62, 64-bit words: Shoup multiplication with a precomputed
//           companion w' = floor(w * 2^64 / q) and Harvey's lazy butterflies
//           (forward values in [0, 4q), inverse values in [0, 2q)).
//
// fp64 is used because gfx950 runs fp64 FMA at full vector rate while 64-bit
// integer multiplies cost several quarter-rate 32-bit partial products.  The
// results are exact integers in every class; no floating-point rounding ever
// reaches an output.
//
// Everything here is __host__ __device__ so that the same code can be checked
// exhaustively on the CPU against 128-bit integer arithmetic.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#ifndef __HIP_DEVICE_COMPILE__
#include <cmath>
#endif

namespace nttk {

#define NTT_HD __host__ __device__ __forceinline__

NTT_HD double fma_rn(double a, double b, double c) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_fma(a, b, c);
#else
  return std::fma(a, b, c);
#endif
}
NTT_HD double rint_rn(double a) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_rint(a);
#else
  return std::nearbyint(a);
#endif
}
NTT_HD double as_double(uint64_t x) {
  union { uint64_t u; double d; } c;
  c.u = x;
  return c.d;
}
NTT_HD uint64_t as_u64(double x) {
  union { uint64_t u; double d; } c;
  c.d = x;
  return c.u;
}
NTT_HD uint64_t mulhi64(uint64_t a, uint64_t b) {
#ifdef __HIP_DEVICE_COMPILE__
  return __umul64hi(a, b);
#else
  return (uint64_t)(((unsigned __int128)a * b) >> 64);
#endif
}

// One device instruction each; everything built on them is the same code on both sides.
NTT_HD uint32_t mulhi32(uint32_t a, uint32_t b) {
#ifdef __HIP_DEVICE_COMPILE__
  return __umulhi(a, b);
#else
  return (uint32_t)(((uint64_t)a * b) >> 32);
#endif
}
// Low 32 bits of (hi 2^32 + lo) >> (s mod 32).
NTT_HD uint32_t funnel32(uint32_t hi, uint32_t lo, uint32_t s) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_amdgcn_alignbit(hi, lo, s);
#else
  return (uint32_t)((((uint64_t)hi << 32) | lo) >> (s & 31u));
#endif
}

constexpr double kTwo52 = 4503599627370496.0;  // 2^52

// Largest modulus (exclusive) of the ArF64L class.  Four inverse (GS) stages
// double the sum side from centred inputs (|x| <= q/2 + 2) to 8q + 32, which
// must stay below 2^53; the forward chain (four CT stages from |x| < q, each
// adding at most q/2 + |x| (q/2) 3 2^-53) stays lower.  2^10 of margin below
// 2^50 covers the rounding terms.  Larger moduli take the integer class.
constexpr uint64_t kF64LBound = (1ull << 50) - (1ull << 10);

// x*w - c*q exactly, with c = rint(RN(x*w) * RN(1/q)).  The quotient estimate
// carries three roundings (the product, 1/q and their product), so
// |result| <= (1/2 + e)*q with e <= |x*w/q| * 3 * 2^-53.  Taking it from the
// high part costs no operation per twiddle (x * (w/q) needs w/q, one product for
// every twiddle used once) and no register to hold it: products of 2 x 36 x 2^16
// polynomials 86.3 -> 83.8 us, a CMux step 16.3 -> 15.9 us.
NTT_HD double f64_mulmod(double x, double w, double q, double qinv) {
  const double h = x * w;
  const double l = fma_rn(x, w, -h);
  const double c = rint_rn(h * qinv);
  const double r = fma_rn(-c, q, h);
  return r + l;
}

// x w mod q for x, w < q < 2^50 - 2^10 given wq = w/q: the exact value of
// x w - c q with c the rounded quotient, in (-7/8 q, 7/8 q).
NTT_HD double f64_mulmod_pre(double x, double w, double wq, double q) {
  const double h = x * w;
  const double l = fma_rn(x, w, -h);
  const double c = rint_rn(x * wq);
  return fma_rn(-c, q, h) + l;
}

// The ModDown step on a reduced sum r in [0, p): (x - r) s mod p for the
// residue x in [0, p), with s < p < 2^50 - 2^10 and sq = s / p.  |x - r| < p,
// so the product is exact as for non-negative operands.
NTT_HD double f64_sub_scale(double x, double r, double s, double sq, double p) {
  const double v = f64_mulmod_pre(x - r, s, sq, p);
  return v < 0.0 ? v + p : v;
}

// General product of two lazily-reduced operands (neither is a table entry).
NTT_HD double f64_mulmod2(double x, double y, double q, double qinv) {
  return f64_mulmod(x, y, q, qinv);
}

// Centred representative: |result| <= q/2 + 2 for |x| < 2^53.
NTT_HD double f64_center(double x, double q, double qinv) {
  const double c = rint_rn(x * qinv);
  return fma_rn(-c, q, x);
}

// Canonical representative in [0, q) for |x| < 2^53.
NTT_HD double f64_canon(double x, double q, double qinv) {
  double r = f64_center(x, q, qinv);
  r = r < 0.0 ? r + q : r;
  return r;
}

// Shoup: y*w mod q in [0, 2q) for any y < 2^64, q < 2^63.  From 32-bit
// halves, with nq = 2^64 - q accumulated into the low product: the two
// low halves share one multiply-add chain and no 64-bit subtraction (with its
// carry through a mask register) follows.  With the sign selects below a
// butterfly of the forward rows went from 66 to 58 instructions and from seven
// wait states to two; products of 3 x 11 limbs of 2^14 at 60 bits 42.1 -> 37.8 us.
NTT_HD uint64_t shoup_mul_n(uint64_t y, uint64_t w, uint64_t ws, uint64_t nq) {
  const uint32_t yl = (uint32_t)y, yh = (uint32_t)(y >> 32);
  const uint32_t sl = (uint32_t)ws, sh = (uint32_t)(ws >> 32);
  const uint64_t t1 = (uint64_t)yl * sh + mulhi32(yl, sl);
  const uint64_t t2 = (uint64_t)yh * sl + (uint32_t)t1;
  const uint64_t h = (uint64_t)yh * sh + (t1 >> 32) + (t2 >> 32);
  const uint32_t hl = (uint32_t)h, hh = (uint32_t)(h >> 32);
  const uint32_t nl = (uint32_t)nq, nh = (uint32_t)(nq >> 32);
  const uint64_t acc = (uint64_t)hl * nl + (uint64_t)yl * (uint32_t)w;
  const uint32_t hi = (uint32_t)(acc >> 32) + yl * (uint32_t)(w >> 32) + yh * (uint32_t)w +
                      hl * nh + hh * nl;
  return ((uint64_t)hi << 32) | (uint32_t)acc;
}
NTT_HD uint64_t shoup_mul(uint64_t y, uint64_t w, uint64_t ws, uint64_t q) {
  return shoup_mul_n(y, w, ws, 0 - q);
}

// x - m for x in [m, 2^63 + m), else x (x < m), given nm = 2^64 - m: one 64-bit
// add and a select on the sign of the difference.
NTT_HD uint64_t cond_sub_n(uint64_t x, uint64_t nm) {
  const uint64_t d = x + nm;
  return (int64_t)d < 0 ? x : d;
}

// Low 64 bits of (hi 2^64 + lo) >> s, s = 0 .. 63, from 32-bit funnel shifts: a
// pointwise kernel with a 64-bit vector shift whose amount lay in the last register of
// the wave's allocation (v39 of 40) returned wrong words once several workgroups shared
// a compute unit, and which register the compiler picks cannot be chosen in the source,
// so no kernel shifts 64 bits by a vector register (test_device_code_host.py reads the
// built code for it).
NTT_HD uint64_t shr128(uint64_t lo, uint64_t hi, uint32_t s) {
  const uint32_t w0 = (uint32_t)lo, w1 = (uint32_t)(lo >> 32), w2 = (uint32_t)hi, w3 = (uint32_t)(hi >> 32);
  const bool up = s >= 32;
  const uint32_t x0 = up ? w1 : w0, x1 = up ? w2 : w1, x2 = up ? w3 : w2;
  return ((uint64_t)funnel32(x2, x1, s) << 32) | funnel32(x1, x0, s);
}

// Barrett-style product of two operands in [0, q), q < 2^62, b = bit length
// of q, mu = floor(2^(2b) / q).  Result in [0, q).
NTT_HD uint64_t barrett_mul(uint64_t a, uint64_t b, uint64_t q, uint64_t mu, uint32_t qbits) {
  const uint64_t lo = a * b;
  const uint64_t hi = mulhi64(a, b);
  // t = floor(P / 2^(qbits-1)) < 2^(qbits+1)
  const uint64_t t = shr128(lo, hi, qbits - 1);
  // e = floor(t * mu / 2^(qbits+1))
  const uint64_t plo = t * mu;
  const uint64_t phi = mulhi64(t, mu);
  const uint64_t e = shr128(plo, phi, qbits + 1);
  uint64_t r = lo - e * q;  // in [0, 3q)
  r = r >= q ? r - q : r;
  r = r >= q ? r - q : r;
  return r;
}

// ---------------------------------------------------------------------------
// Per-modulus constants as the kernels see them.
struct LimbDev {
  uint64_t q;
  union { double qd; uint64_t nq; };       // fp64 classes: q;   ArI64: 2^64 - q
  union { double qinv; uint64_t nq2; };    // fp64 classes: 1/q; ArI64: 2^64 - 2q
  const void* twf;  // forward table, index k -> psi^brv(k)  (double or TwI64)
  const void* twi;  // inverse table, index k -> psi^-brv(k)
  // N^-1 folded into the last inverse stage: (u+v)*ninv, (u-v)*ninvw
  double ninv_d, ninvw_d;                  // centred, fp64 classes
  uint64_t ninv, ninv_s, ninvw, ninvw_s;   // Shoup pairs, ArI64
  uint64_t bmu;                            // Barrett constant, ArI64
  uint32_t qbits;
  uint32_t cls;
};

struct TwI64 {
  uint64_t w, ws;
};

// The constants of modulus q that depend on its class alone.
inline void set_limb_modulus(LimbDev& d, uint64_t q, uint32_t cls) {
  d.q = q;
  if (cls == 2) {
    d.nq = 0 - q;
    d.nq2 = 0 - 2 * q;
  } else {
    d.qd = (double)q;
    d.qinv = 1.0 / (double)q;
  }
  d.cls = cls;
  d.qbits = 64 - __builtin_clzll(q);
  d.bmu = (uint64_t)(((unsigned __int128)1 << (2 * d.qbits)) / q);
}

// ---------------------------------------------------------------------------
// Arithmetic classes used as kernel template parameters.

struct ArF64S {
  using W = uint32_t;
  using V = double;
  using TW = double;
  static constexpr int kCls = 0;
  static constexpr const char* kName = "f64s";
  static constexpr bool kCenterRounds = false;
  double q, qinv;
  NTT_HD explicit ArF64S(const LimbDev& d) : q(d.qd), qinv(d.qinv) {}
  NTT_HD V from_word(W x) const { return (double)x; }
  NTT_HD W to_word(V x) const { return (W)f64_canon(x, q, qinv); }
  NTT_HD V from_raw(W x) const { return (double)(int32_t)x; }
  NTT_HD W to_raw(V x) const { return (W)(int32_t)f64_center(x, q, qinv); }
  NTT_HD void center(V& x) const { (void)x; }
  NTT_HD void ct(V& x, V& y, TW w) const {
    const double t = f64_mulmod(y, w, q, qinv);
    const double a = x;
    x = a + t;
    y = a - t;
  }
  NTT_HD void gs(V& x, V& y, TW w) const {
    const double a = x, b = y;
    x = a + b;
    y = f64_mulmod(a - b, w, q, qinv);
  }
  NTT_HD void gs_fold(V& x, V& y, TW w, const LimbDev& d) const {
    (void)w;
    const double a = x, b = y;
    x = f64_mulmod(a + b, d.ninv_d, q, qinv);
    y = f64_mulmod(a - b, d.ninvw_d, q, qinv);
  }
  NTT_HD V mul(V x, V y) const {
    return f64_mulmod2(f64_center(x, q, qinv), f64_center(y, q, qinv), q, qinv);
  }
  // Multiply-accumulate: a transform's value as an operand, its product with a
  // canonical word, the sum of up to eight products on a folded sum, the fold.
  // Any |f| < 2^12 q and 2^20 terms stay far below 2^53: nothing to reduce.
  NTT_HD V mac_operand(V x) const { return x; }
  NTT_HD V mac_term(V f, V k) const { return f64_mulmod(f, k, q, qinv); }
  NTT_HD V mac_add(V a, V t) const { return a + t; }
  NTT_HD V mac_fold(V a) const { return f64_center(a, q, qinv); }
  // A gadget digit (|d| <= 2^31; top digits are not negative) as a value.
  NTT_HD V from_digit(uint32_t d, bool top) const { return top ? (double)d : (double)(int32_t)d; }
};

struct ArF64L {
  using W = uint64_t;
  using V = double;
  using TW = double;
  static constexpr int kCls = 1;
  static constexpr const char* kName = "f64l";
  static constexpr bool kCenterRounds = true;
  double q, qinv;
  NTT_HD explicit ArF64L(const LimbDev& d) : q(d.qd), qinv(d.qinv) {}
  // Words below 2^52 become doubles exactly through the 2^52 exponent trick.
  NTT_HD V from_word(W x) const { return as_double(x | 0x4330000000000000ull) - kTwo52; }
  NTT_HD W to_word(V x) const {
    const double r = f64_canon(x, q, qinv);
    return as_u64(r + kTwo52) & 0x000FFFFFFFFFFFFFull;
  }
  NTT_HD V from_raw(W x) const { return as_double(x); }
  NTT_HD W to_raw(V x) const { return as_u64(f64_center(x, q, qinv)); }
  NTT_HD void center(V& x) const { x = f64_center(x, q, qinv); }
  NTT_HD void ct(V& x, V& y, TW w) const {
    const double t = f64_mulmod(y, w, q, qinv);
    const double a = x;
    x = a + t;
    y = a - t;
  }
  NTT_HD void gs(V& x, V& y, TW w) const {
    const double a = x, b = y;
    x = a + b;
    y = f64_mulmod(a - b, w, q, qinv);
  }
  NTT_HD void gs_fold(V& x, V& y, TW w, const LimbDev& d) const {
    (void)w;
    const double a = x, b = y;
    x = f64_mulmod(a + b, d.ninv_d, q, qinv);
    y = f64_mulmod(a - b, d.ninvw_d, q, qinv);
  }
  NTT_HD V mul(V x, V y) const {
    return f64_mulmod2(f64_center(x, q, qinv), f64_center(y, q, qinv), q, qinv);
  }
  // Multiply-accumulate: a transform's value as an operand, its product with a
  // canonical word, the sum of up to eight products on a folded sum, the fold.
  // |f| <= q (centred, or a canonical word) and k in [0, q): |term| <= 7/8 q, and
  // q/2 + 2 plus eight of them stay below 2^53.
  NTT_HD V mac_operand(V x) const { return f64_center(x, q, qinv); }
  NTT_HD V mac_term(V f, V k) const { return f64_mulmod(f, k, q, qinv); }
  NTT_HD V mac_add(V a, V t) const { return a + t; }
  NTT_HD V mac_fold(V a) const { return f64_center(a, q, qinv); }
  NTT_HD V from_digit(uint32_t d, bool top) const { return top ? (double)d : (double)(int32_t)d; }
};

struct ArI64 {
  using W = uint64_t;
  using V = uint64_t;
  using TW = TwI64;
  static constexpr int kCls = 2;
  static constexpr const char* kName = "i64";
  static constexpr bool kCenterRounds = false;
  uint64_t q, q2, nq, nq2, mu;
  uint32_t qbits;
#if defined(__HIP_DEVICE_COMPILE__) || defined(NTT_LIMB_NEGATIONS)
  // -q and -2q read, not formed here: a product with a visible negation is turned back
  // into a product with q and a subtraction
  NTT_HD explicit ArI64(const LimbDev& d)
      : q(d.q), q2(2 * d.q), nq(d.nq), nq2(d.nq2), mu(d.bmu), qbits(d.qbits) {}
#else
  NTT_HD explicit ArI64(const LimbDev& d)
      : q(d.q), q2(2 * d.q), nq(0 - d.q), nq2(0 - 2 * d.q), mu(d.bmu), qbits(d.qbits) {}
#endif
  NTT_HD V from_word(W x) const { return x; }
  // x in [0, 4q): q < 2^62, so every difference below lies in (-2^63, 2^63).
  NTT_HD W to_word(V x) const { return cond_sub_n(cond_sub_n(x, nq2), nq); }
  NTT_HD V from_raw(W x) const { return x; }
  NTT_HD W to_raw(V x) const { return x; }
  NTT_HD void center(V& x) const { (void)x; }
  // Forward (Harvey): x, y in [0, 4q) -> outputs in [0, 4q).
  NTT_HD void ct(V& x, V& y, TW w) const {
    const uint64_t a = cond_sub_n(x, nq2);
    const uint64_t t = shoup_mul_n(y, w.w, w.ws, nq);
    x = a + t;
    y = a + q2 - t;
  }
  // Inverse (Harvey): x, y in [0, 2q) -> outputs in [0, 2q).
  NTT_HD void gs(V& x, V& y, TW w) const {
    const uint64_t a = x, b = y;
    x = cond_sub_n(a + b, nq2);
    y = shoup_mul_n(a + q2 - b, w.w, w.ws, nq);
  }
  NTT_HD void gs_fold(V& x, V& y, TW w, const LimbDev& d) const {
    (void)w;
    const uint64_t a = x, b = y;
    x = shoup_mul_n(a + b, d.ninv, d.ninv_s, nq);
    y = shoup_mul_n(a + q2 - b, d.ninvw, d.ninvw_s, nq);
  }
  NTT_HD V mul(V x, V y) const { return barrett_mul(to_word(x), to_word(y), q, mu, qbits); }
  // Operands in [0, q) (products of mul) -> sum in [0, q).
  NTT_HD V add(V x, V y) const {
    const uint64_t s = x + y;
    return s >= q ? s - q : s;
  }
  // Multiply-accumulate on canonical values.
  NTT_HD V mac_operand(V x) const { return to_word(x); }
  NTT_HD V mac_term(V f, V k) const { return barrett_mul(f, k, q, mu, qbits); }
  NTT_HD V mac_add(V a, V t) const { return add(a, t); }
  NTT_HD V mac_fold(V a) const { return a; }
  NTT_HD V from_digit(uint32_t d, bool top) const {
    return top || !(d >> 31) ? (V)d : q - (V)(0u - d);
  }
};

}  // namespace nttk
