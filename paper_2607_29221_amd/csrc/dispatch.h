// Which kernel form a call takes: rules on sizes, types and alignment alone,
// free of HIP so that they can be compiled and checked on the host.
#pragma once

#include <stdint.h>

namespace mosaic {

// A launch holds fewer than 2^32 threads.
constexpr int64_t kMaxGridThreads = (int64_t(1) << 32) - 256;

// ---------------------------------------------------------------------------
// Mask pass (elementwise.hip)

enum MaskRoute { MASK_QUAD, MASK_QUAD_RAGGED, MASK_TURN, MASK_GENERAL };

struct MaskShape {
  int64_t rows, cols;
  bool has_x, x_row, x_turned;        // plaintext; its rows contiguous (x_cs == 1), its columns (x_rs == 1)
  bool aligned;                       // every row of x, u and out on a lane's alignment, cols % 4 == 0
  bool has_noise, noise_transposed;
  bool digits;                        // digits are written
};

// Workgroups per row of mask_quad_kernel (1024 columns each).
inline int64_t mask_quad_slices(const MaskShape& a) {
  const int64_t lanes = a.digits ? 64 * ((a.cols + 63) / 64) / 4 : 4 * ((a.cols + 15) / 16);
  return (lanes + 255) / 256;
}

inline MaskRoute mask_route(const MaskShape& a, int64_t cus) {
  // Contiguous rows take mask_quad_kernel, its ragged form unless every row of
  // every operand starts on a lane's own alignment (16 bytes of words, 4 of
  // int8) and ends with a whole lane. The ragged form gives a row a workgroup
  // of its own, whose 256 threads draw noise whether the row has columns for
  // them or not: short rows take the general kernel, which packs 16 columns of
  // many rows into a workgroup, unless the rows are so few that it leaves the
  // chip idle. Device time, general / ragged: words + u + noise to digits
  // 65027 x 129 68 / 85 us, 43919 x 191 61 / 68, 32640 x 257 61 / 46; uniform
  // sample 2796202 x 3 31 / 1573, 15420 x 17 11 / 12, 4161 x 63 11 / 5.8,
  // 3276 x 5 5.6 / 4.7.
  const bool fits = a.rows <= kMaxGridThreads / 256 / mask_quad_slices(a);
  if ((!a.has_x || a.x_row) && !(a.has_noise && a.noise_transposed) && fits) {
    if (a.aligned) return MASK_QUAD;
    if (a.cols >= 192 || a.rows <= (a.cols >= 16 ? 24 : 8) * cus) return MASK_QUAD_RAGGED;
    return MASK_GENERAL;
  }
  // Transposed plaintext and transposed noise (or one of them alone): tiles
  // turned through LDS. What remains for the general kernel is one of them
  // transposed and the other not, and plaintext with two strides.
  const int64_t tiles_j = (a.cols + 63) / 64;
  if ((!a.has_x || a.x_turned) && (!a.has_noise || a.noise_transposed) &&
      (a.rows + 63) / 64 <= kMaxGridThreads / 256 / tiles_j)
    return MASK_TURN;
  return MASK_GENERAL;
}

}  // namespace mosaic
