// bconv_rules.hpp -- which form a basis conversion takes and the grid of the
// few-source kernel: host arithmetic on sizes alone.
#pragma once

#include <cstdint>

namespace nttk {

// What a conversion kernel does around the sum (the template argument MODE).
constexpr int kBconvPlain = 0;  // y_j
constexpr int kBconvUp = 1;     // y_j, and the source residues copied beside them
constexpr int kBconvDown = 2;   // (x_j - y_j) s_j mod p_j

constexpr uint32_t kBconvBlock = 256;
constexpr int kFewUnroll = 4;  // targets a thread of the few-source kernel has in flight

// Register sizes the few-source kernel is built for.
inline uint32_t few_size(uint32_t L) { return L <= 8 ? L : L <= 16 ? (L + 1u) & ~1u : 0u; }

// Whether a call whose shape the matrix cores take by default (more than 8 sources)
// still runs on the vector units: with few targets the matrix form's one or two owner
// waves finish every output while its digit waves wait, and large calls fill the chip
// without it.  Vector over matrix time, over rotating buffers of some 700 MB in all:
//   conversion, up to 16 sources (few-source kernel), up to 4 targets from 2^15
//     coefficients per target on: 3 x 2^15 coefficients, 1 target from 9 / 16 sources
//     0.74 / 0.91, 3 from 16 1.06; 4 x 2^16, 4 targets 0.80 / 0.99 (below: 2^14, 1 target
//     1.05 / 1.37); up to 8 targets of up to 10 sources from 3 x 2^16 on (0.94);
//   ModUp the same while sources x targets is up to 40 (3 x 2^16: 4 targets from 9 / 12
//     sources 0.91 / 1.04; 4 x 2^16, 2 from 16 1.03, 8 from 9 1.04);
//   ModDown, whose outputs cost the owners more, up to 8 targets from 2^16 coefficients on
//     (3 x 2^15: 8 targets from 9 / 16 sources 0.63 / 0.84, 12 from 9 / 12 0.95 / 1.05),
//     and at any number from 2^18 on for up to 12 sources (4 x 2^16: 12 / 36 targets from
//     9 sources 0.86 / 0.89, from 12 0.97 / 1.02; 3 x 2^16: 0.97 / 1.02 and 1.12 / 1.14);
//   more sources (the kernel that re-reads them), ModDown from 3 x 2^16 on: 17 sources
//     0.84 / 1.01 for 1 / 4 targets, 24 1.03 for 2 (4 x 2^16 0.72 / 0.85, 0.87), 36 1.15;
//     above 36, where the matrix form cannot load ahead, 4 x 2^16 0.76 / 0.81 for 1 / 4
//     from 40; other conversions from 2^19 on only (17 and 20 sources to 2 0.91 / 0.92).
inline bool vector_first(int mode, bool few, uint32_t L, uint32_t M, uint32_t total) {
  if (mode == kBconvDown)
    return few ? (M <= 4 && total >= M << 15) || (M <= 8 && total >= 1u << 16) ||
                     (L <= 12 && total >= 4u << 16)
               : total >= 3u << 16 && (L > 36 ? M <= 4 : L <= 24 && L * M <= 68);
  if (!few) return L <= 20 && M <= 2 && total >= 8u << 16;
  if (mode == kBconvUp && L * M > 40) return false;
  return (M <= 4 && total >= M << 15) || (M <= 8 && L <= 10 && mode == kBconvPlain && total >= 3u << 16);
}

struct FewGrid {
  uint32_t blocks, rows, per;  // grid x (coefficients), grid y, targets per grid row
};

// Grid rows of the few-source kernel: enough to put about eight waves on every
// SIMD when one coefficient per thread does not, each row at least kFewUnroll
// targets.  (ModDown 24 + 8 limbs of 4 x 2^16: 37.2 us with four waves, 32.6 with
// eight, 35.0 with sixteen.)
inline FewGrid few_grid(uint32_t total, uint32_t M) {
  const uint32_t want = (uint32_t)((2048ull * 256u + total - 1u) / total);
  const uint32_t most = (M + kFewUnroll - 1) / kFewUnroll;
  const uint32_t rows = want < most ? want : most;
  FewGrid g;
  g.blocks = (uint32_t)(((uint64_t)total + kBconvBlock - 1) / kBconvBlock);
  g.per = (M + rows - 1) / rows;
  g.rows = (M + g.per - 1) / g.per;
  return g;
}

}  // namespace nttk
