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
  // Transposed plaintext and transposed noise (or one of them alone): tiles of
  // 64 x 64 turned through LDS, unless a side is so short that most of a tile
  // is empty. That counts once there are more tiles than compute units; and
  // where the rows are not a multiple of four, every lane's four noise elements
  // lie across Philox blocks (two, of a sparse stream three). Device time,
  // general / turned: uniform sample 1 x 2^20 8 / 71 us, 33 x 262144 24 / 29,
  // 48 x 262144 34 / 23; sparse 65 x 512 7.3 / 10.3, 1 x 4096 6.9 / 9.8; int8 + u
  // 2^20 x 3 13 / 43, 262144 x 16 13 / 15, 20 x 262144 20 / 14; dgauss 4 x 4096 10.0 /
  // 5.3. What remains for the general kernel besides is one of plaintext and
  // noise transposed and the other not, and plaintext with two strides.
  const int64_t tiles_i = (a.rows + 63) / 64, tiles_j = (a.cols + 63) / 64;
  if ((a.has_x && !a.x_turned) || (a.has_noise && !a.noise_transposed) || tiles_i > kMaxGridThreads / 256 / tiles_j)
    return MASK_GENERAL;
  const bool few = tiles_i * tiles_j <= cus;
  const int64_t min_rows = !a.has_noise ? (few ? 2 : 12) : a.rows % 4 != 0 ? 128 : few ? 4 : 32;
  return a.cols >= (few ? 6 : 17) && a.rows >= min_rows ? MASK_TURN : MASK_GENERAL;
}

}  // namespace mosaic
