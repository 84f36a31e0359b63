"""Host checks of the device arithmetic's 32-bit-halves forms and of the sums that are
reduced only every eight terms (csrc/modarith.hpp, csrc/decompose.hpp), compiled with
g++ as the kernels inline them (the integer class reads its negated moduli from the
limb's constants, as on the device) against 128-bit integers, at the worst cases:

  * Shoup products and the Harvey butterflies for every operand range they take, 64-bit
    shifts through 32-bit funnels at every amount, conditional subtractions by sign;
  * eight products of up to 7/8 q on a folded sum (multiply-accumulate, external
    product) and eight of the basis conversions stay exact integers below 2^53 at the
    largest fp64 modulus, for the operands that make them largest;
  * gadget digits as values of every class, up to 32-bit bases.
"""
import os
import shutil
import subprocess

import pytest

from paper_2410_05934_amd import synth

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2410_05934_amd", "csrc")
ROCM_INC = "/opt/rocm/include"

DRIVER = r"""
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>
#include "modarith.hpp"
#include "decompose.hpp"
using namespace nttk;
typedef __int128 i128;
typedef unsigned __int128 u128;
typedef unsigned long long ull;

static long fails = 0, checks = 0;
#define CHECK(cond, ...)                                                        \
  do {                                                                          \
    ++checks;                                                                   \
    if (!(cond)) {                                                              \
      if (fails++ < 12) { std::printf("FAIL line %d: ", __LINE__);              \
                          std::printf(__VA_ARGS__); std::printf("\n"); }        \
    }                                                                           \
  } while (0)
static i128 md(i128 a, i128 q) { i128 r = a % q; return r < 0 ? r + q : r; }
static bool int53(double v) { return std::fabs(v) < 9007199254740992.0 && v == std::nearbyint(v); }
static const long double U = 1.0L / 9007199254740992.0L;  // 2^-53

static LimbDev limb(uint64_t q, uint32_t cls) {
  LimbDev d;
  std::memset(&d, 0, sizeof(d));
  set_limb_modulus(d, q, cls);
  return d;
}

static void check_integer_class(uint64_t q, std::mt19937_64& rng) {
  const LimbDev ld = limb(q, 2);
  CHECK(ld.nq + q == 0 && ld.nq2 + 2 * q == 0, "negated moduli");
  const ArI64 ar(ld);
  std::uniform_int_distribution<uint64_t> dq(0, q - 1), d64;
  auto some = [&](uint64_t top, int n) {
    std::vector<uint64_t> v = {0, 1, top - 1, top / 2, top / 2 + 1};
    for (uint64_t m : {q, 2 * q, 3 * q}) for (uint64_t x : {m - 1, m, m + 1}) if (x < top) v.push_back(x);
    for (uint64_t x : {0xffffffffull, 0x100000000ull, 0xffffffff00000000ull, 0xfffffffeffffffffull})
      if (x < top) v.push_back(x);
    std::uniform_int_distribution<uint64_t> d(0, top - 1);
    for (int i = 0; i < n; ++i) v.push_back(d(rng));
    return v;
  };
  std::vector<uint64_t> ys = some(~0ull, 200), ws = some(q, 60);
  ys.push_back(~0ull);
  for (uint64_t w : ws) {
    const uint64_t s = (uint64_t)(((u128)w << 64) / q);
    for (uint64_t y : ys) {
      const uint64_t r = shoup_mul_n(y, w, s, ld.nq);
      CHECK(r < 2 * q && (u128)r % q == (u128)y * w % q && r == y * w - mulhi64(y, s) * q,
            "shoup q=%llu y=%llu w=%llu", (ull)q, (ull)y, (ull)w);
    }
  }
  for (uint64_t x : some(4 * q, 300)) {
    const uint64_t c = cond_sub_n(x, ld.nq2);
    CHECK(c == (x >= 2 * q ? x - 2 * q : x), "conditional subtraction x=%llu", (ull)x);
    CHECK(ar.to_word(x) == x % q, "to_word x=%llu", (ull)x);
  }
  for (uint64_t w : {(uint64_t)0, (uint64_t)1, q - 1, q / 2, dq(rng), dq(rng)}) {
    const TwI64 tw = {w, (uint64_t)(((u128)w << 64) / q)};
    for (uint64_t x : some(4 * q, 40))
      for (uint64_t y : some(4 * q, 40)) {
        uint64_t X = x, Y = y;
        ar.ct(X, Y, tw);
        const i128 t = (i128)((u128)y * w % q);
        CHECK(X < 4 * q && Y < 4 * q && md((i128)X - x - t, q) == 0 && md((i128)Y - x + t, q) == 0, "ct");
        if (x < 2 * q && y < 2 * q) {
          X = x; Y = y;
          ar.gs(X, Y, tw);
          CHECK(X < 2 * q && Y < 2 * q && md((i128)X - x - y, q) == 0 &&
                    md((i128)Y - ((i128)x - (i128)y) * (i128)w, q) == 0, "gs");
        }
        CHECK(ar.mac_term(x % q, y % q) == (uint64_t)((u128)(x % q) * (y % q) % q), "product");
      }
  }
}

static void check_shifts(std::mt19937_64& rng) {
  std::uniform_int_distribution<uint64_t> d;
  for (int i = 0; i < 400; ++i) {
    const uint64_t lo = i == 0 ? 0 : i == 1 ? ~0ull : d(rng), hi = i == 2 ? 0 : i == 1 ? ~0ull : d(rng);
    for (uint32_t s = 0; s < 64; ++s)
      CHECK(shr128(lo, hi, s) == (uint64_t)((((u128)hi << 64) | lo) >> s), "shift by %u", s);
  }
}

// A folded sum and eight more products, each operand pair chosen (of many) to make its
// product as large as it gets, all of one sign; then the fold.
template <class Term, class Fold>
static long double eight_terms(uint64_t q, Term term, Fold fold, double start, std::mt19937_64& rng) {
  long double most = 0;
  for (int sign : {1, -1}) {
    double acc = sign * start;
    i128 sum = (i128)acc;
    for (int i = 0; i < 8; ++i) {
      double best = 0;
      i128 exact = 0;
      for (int k = 0; k < 4000; ++k) {
        i128 e;
        const double t = term(rng, &e);
        CHECK(int53(t) && md((i128)t - e, q) == 0, "product not exact");
        if (k == 0 || sign * t > sign * best) { best = t; exact = e; }
      }
      // analytic: the quotient's three roundings move it by at most 3 2^-53 of itself
      CHECK(std::fabs((long double)best) <= (long double)q * (0.5L + (long double)q * 3 * U * (1 + U)), "term bound");
      acc += best;
      sum += exact;
      most = std::max(most, (long double)std::fabs(acc));
      CHECK(int53(acc), "sum of %d terms left 2^53", i + 1);
    }
    const double r = fold(acc);
    CHECK(md((i128)r - sum, q) == 0 && std::fabs(r) <= (double)(q / 2 + 2), "fold");
  }
  return most / q;
}

int main(int argc, char** argv) {
  if (argc == 2) { std::printf("%llu\n", (ull)kF64LBound); return 0; }
  uint64_t Q[5];
  for (int i = 0; i < 5; ++i) Q[i] = std::strtoull(argv[i + 1], nullptr, 10);
  const uint64_t qL = Q[0], q32 = Q[1], q62 = Q[2], q56 = Q[3], qs = Q[4];
  std::mt19937_64 rng(2468);
  for (uint64_t q : {q62, q56, qL, qs}) check_integer_class(q, rng);
  check_shifts(rng);

  const long double lq = (long double)qL;
  // whatever the operands: half a modulus and eight terms
  CHECK(lq / 2 + 2 + 8 * lq * (0.5L + lq * 3 * U * (1 + U)) < 1 / U, "eight terms at the class bound");
  CHECK((double)kF64LBound * 7.5 + 2 < 9007199254740992.0, "eight terms of 7/8 q at the class bound");
  long double m[3];
  {  // multiply-accumulate: canonical words, or a centred transform value, times a key word
    const ArF64L ar(limb(qL, 1));
    std::uniform_int_distribution<uint64_t> near(qL - (1 << 20), qL - 1), any(0, qL - 1);
    auto words = [&](std::mt19937_64& r, i128* e) {
      const uint64_t f = r() & 1 ? near(r) : any(r), k = r() & 1 ? near(r) : any(r);
      *e = (i128)f * k;
      return ar.mac_term(ar.from_word(f), ar.from_word(k));
    };
    auto fold = [&](double a) { return ar.mac_fold(a); };
    m[0] = eight_terms(qL, words, fold, (double)(qL / 2 + 2), rng);
    std::uniform_int_distribution<int64_t> c(-(int64_t)(qL / 2 + 2), (int64_t)(qL / 2 + 2));
    auto centred = [&](std::mt19937_64& r, i128* e) {
      const int64_t f = c(r);
      const uint64_t k = near(r);
      *e = (i128)f * k;
      return ar.mac_term((double)f, ar.from_word(k));
    };
    m[1] = eight_terms(qL, centred, fold, (double)(qL / 2 + 2), rng);
    for (int i = 0; i < 20000; ++i) {  // what publishes a transform's value
      const double x = (double)(int64_t)(rng() >> 11) * (i & 1 ? 1 : -1);
      const double f = ar.mac_operand(x);
      CHECK(md((i128)f - (i128)x, qL) == 0 && std::fabs(f) <= (double)(qL / 2 + 2), "mac_operand");
    }
  }
  {  // basis conversion: t below the source modulus, w below the target's, w / p given
    const double p = (double)qL, pinv = 1.0 / p;
    std::uniform_int_distribution<uint64_t> near(qL - (1 << 20), qL - 1), any(0, qL - 1);
    auto term = [&](std::mt19937_64& r, i128* e) {
      const uint64_t t = r() & 1 ? near(r) : any(r), w = r() & 1 ? near(r) : any(r);
      *e = (i128)t * w;
      return f64_mulmod_pre((double)t, (double)w, (double)w * pinv, p);
    };
    auto fold = [&](double a) { return std::fma(-std::nearbyint(a * pinv), p, a); };
    m[2] = eight_terms(qL, term, fold, (double)(qL / 2 + 2), rng);
    for (uint64_t small : {(uint64_t)3, (uint64_t)65537, q32}) {  // targets far below the source
      const double sp = (double)small;
      for (int i = 0; i < 20000; ++i) {
        const uint64_t t = near(rng), w = rng() % small;
        const double v = f64_mulmod_pre((double)t, (double)w, (double)w * (1.0 / sp), sp);
        CHECK(int53(v) && md((i128)v - (i128)t * w, small) == 0 && std::fabs(v) < 0.875 * sp + 1, "small target");
      }
    }
  }
  {  // 32-bit moduli: a transform's unreduced value (below 2^12 q) times a word, 2^20 of them
    const ArF64S ar(limb(q32, 0));
    std::uniform_int_distribution<int64_t> d(-((int64_t)q32 << 12), (int64_t)q32 << 12);
    long double most = 0;
    for (int i = 0; i < 200000; ++i) {
      const int64_t f = i < 2 ? (i ? -((int64_t)q32 << 12) : (int64_t)q32 << 12) : d(rng);
      const uint32_t k = i % 3 ? (uint32_t)(rng() % q32) : (uint32_t)(q32 - 1);
      const double t = ar.mac_term(ar.mac_operand((double)f), ar.from_word(k));
      CHECK(int53(t) && md((i128)t - (i128)f * k, q32) == 0, "32-bit product");
      most = std::max(most, (long double)std::fabs(t));
    }
    CHECK(most * (1 << 20) < 1 / U, "2^20 terms of the 32-bit class");
  }
  // gadget digits as values: congruent to the digit, no larger than half a base
  struct Combo { uint64_t q; int levels, beta; } combos[] = {
      {q32, 3, 11}, {q32, 2, 17}, {q32, 2, 32}, {qs, 1, 32}, {qs, 2, 9}, {qs, 2, 32},
      {qL, 2, 26}, {qL, 2, 32}, {q62, 2, 32}, {q62, 4, 16}};
  for (const Combo& c : combos) {
    const uint64_t off = digit_offset(c.levels, c.beta);
    const bool small = c.q < (1ull << 32);
    for (int i = 0; i < 20000; ++i) {
      const uint64_t x = i == 0 ? 0 : i == 1 ? c.q - 1 : i == 2 ? c.q / 2 : rng() % c.q;
      for (int j = 0; j < c.levels; ++j) {
        const bool top = j + 1 == c.levels;
        const uint32_t d = digit_bits(x, j, top, c.beta, off);
        const uint64_t want = signed_digit<uint64_t>(x, j, c.levels, c.beta, off, c.q);
        const i128 v = top ? (i128)d : (i128)(int32_t)d;
        CHECK(md(v, c.q) == (i128)want % c.q && v <= (i128)1 << 31 && v >= -((i128)1 << 31), "digit bits");
        const double l = ArF64L(limb(c.q, 1)).from_digit(d, top);
        CHECK((i128)l == v, "fp64 digit");
        if (small) CHECK((i128)ArF64S(limb(c.q, 0)).from_digit(d, top) == v, "32-bit digit");
        CHECK(ArI64(limb(c.q, 2)).from_digit(d, top) == want, "integer digit");
      }
    }
  }
  std::printf("largest sums: words %.3Lf q, centred %.3Lf q, conversion %.3Lf q\n", m[0], m[1], m[2]);
  std::printf("%s %ld checks, %ld failures\n", fails ? "FAILED" : "ok", checks, fails);
  return fails ? 1 : 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(ROCM_INC),
                    reason="g++ or the HIP headers not available")
def test_halves_forms_and_eight_term_sums(tmp_path):
    src, exe = tmp_path / "arith.cpp", tmp_path / "arith"
    src.write_text(DRIVER)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__",
                           "-DNTT_LIMB_NEGATIONS", f"-I{ROCM_INC}", f"-I{CSRC}", str(src), "-o", str(exe)])
    bound = int(subprocess.run([str(exe), "bound"], capture_output=True, text=True, check=True).stdout)
    q = [synth.primes_below(bound, 1 << 17, 1)[0], synth.primes_below(1 << 32, 1 << 17, 1)[0],
         synth.primes_below(1 << 62, 1 << 17, 1)[0], synth.latency_prime(), 65537]
    out = subprocess.run([str(exe), *map(str, q)], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout + out.stderr
    print(out.stdout)
