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
// without it.  Vector over matrix time:
//   up to 16 sources (few-source kernel): up to 4 targets from 2^15 coefficients per
//     target on (conversion from 9 / 16 sources, 4 x 2^16 coefficients: 1 target 0.47 /
//     0.62, 4 0.68 / 0.90; 2^14: 1.05 / 1.37, 1.44 / 1.93), and up to 8 targets of up
//     to 10 sources from 3 x 2^16 on (9 sources, 8 targets 0.81, ModUp 0.89); ModDown,
//     whose outputs cost the owners more, up to 8 targets from 2^16 coefficients on (4 x
//     2^16: 8 targets 0.75 / 1.05, 12 0.98 / 1.32; 2^15: 1.13 / 1.46);
//   more sources, ModDown from 3 x 2^16 coefficients on (the kernel that re-reads them):
//     17 sources 0.64 .. 0.94 for 1 .. 4 targets, 24 0.96 / 1.03 / 1.34 for 1 / 2 / 4,
//     36 1.13 / 1.54 for 1 / 4; above 36, where the matrix form cannot load ahead, 4 x
//     2^16: 0.74 / 0.93 for 1 / 4.
inline bool vector_first(int mode, bool few, uint32_t L, uint32_t M, uint32_t total) {
  if (few)
    return (M <= 4 && total >= M << 15) ||
           (M <= 8 && (mode == kBconvDown ? total >= 1u << 16 : L <= 10 && total >= 3u << 16));
  return mode == kBconvDown && total >= 3u << 16 && (L > 36 ? M <= 4 : L <= 24 && L * M <= 68);
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
