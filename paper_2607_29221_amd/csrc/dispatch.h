// Which kernel form a call takes: rules on sizes, types and alignment alone,
// free of HIP so that they can be compiled and checked on the host.
#pragma once

#include <stdint.h>

#include <initializer_list>

namespace mosaic {

// A launch holds fewer than 2^32 threads (along its first dimension): the
// runtime takes a larger one without an error and runs the remainder modulo
// 2^32 only.
constexpr int64_t kMaxGridThreads = (int64_t(1) << 32) - 256;

// Cuts rows x units (the units of a row side by side, such as the blocks of a
// rotation) into launches of at most `most` units: whole rows, or parts of one
// row where a row has more. f(row0, rows, unit0, units) returns true to go on.
template <class F>
inline void for_each_launch(int64_t rows, int64_t units, int64_t most, F f) {
  const int64_t per_u = units < most ? units : most, per_r = units < most ? most / units : 1;
  for (int64_t r = 0; r < rows; r += per_r)
    for (int64_t u = 0; u < units; u += per_u)
      if (!f(r, rows - r < per_r ? rows - r : per_r, u, units - u < per_u ? units - u : per_u)) return;
}

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

// ---------------------------------------------------------------------------
// Products of one or two rows of A by dot products (ring_gemv.hip): which of
// them are ahead of the matrix-core kernels, in M, N and the padded inner
// dimension Kp. All kernels stream B, at 5-6 TB/s beyond a few megabytes, so
// the dot products gain what stands around the stream, and lose where a wave's
// own chain is long (long rows, too few of them to hide it) or its fixed cost
// per two rows of B is (many short rows). A wave's sums fit 32 bits and its
// LDS a compute unit's up to 6144 columns. Device time, B beyond the last-level
// cache.

constexpr int64_t kGemvMaxN = 8 * (kMaxGridThreads / 256);   // a workgroup of 256 threads per 8 rows of B

// Store: the matrix-core kernel clears C first (a launch of its own) and adds
// partial sums. One row, matrix cores / dot products: 4096 x 1536 9.5 / 7.3 us,
// 8192 x 3072 22.6 / 19.3, 1024 x 4096 7.4 / 7.0, 3072 x 5120 15.5 / 14.3; but 200 x 4096
// 5.8 / 6.2, 1024 x 5120 8.7 / 9.4, 2048 x 5120 11.8 / 12.1, 28672 x 128 7.0 / 8.5. Two rows
// gain up to 2048 columns (8192 x 1536 13.9 / 12.3; 6656 x 4096 20.7 / 22.1) and
// lose on many short rows sooner (16384 x 256 7.8 / 8.1, 28672 x 512 warm 13.4 / 13.8).
inline bool gemv_takes_store(int64_t M, int64_t N, int64_t Kp) {
  if (Kp <= 0 || N > kGemvMaxN || (N > 8192 && Kp < 512)) return false;
  if (M == 2) return Kp <= 2048;
  return M == 1 && (Kp <= 3072 || (Kp <= 4096 && N >= 1024) || (Kp <= 6144 && N >= 3072));
}

// Unmask from ring words. One row: 64 x 6144 17.3 / 8.2 us, 4096 x 1536 9.6 / 7.8, 28672
// x 6144 135 / 119; two rows: 4096 x 1536 9.6 / 8.6, 28672 x 2048 54 / 42. A single
// chunk of 64 columns is behind with either: 16384 x 64 5.6 / 6.6 and 5.7 / 7.9.
inline bool gemv_takes_unmask(int64_t M, int64_t N, int64_t Kp) {
  if (Kp < 128 || N > kGemvMaxN) return false;
  return (M == 1 && Kp <= 6144) || (M == 2 && Kp <= 2048);
}

// Unmask from ring words of 3 to 16 rows (ring_gemm_skinny.hip): 16-row tiles of
// B and waves per workgroup. One tile and four waves while that leaves no
// compute unit a second round. Beyond, two waves halve the reads of A and the
// sums to add, which is most of the time with a short inner dimension, but a
// long one is left with too few loads in flight. Beyond 48 columns of the
// output per unit: two tiles, on two waves up to 3072 columns of the inner
// dimension (four / two waves, factors beyond the last-level cache: 8 x 14336 at
// 704 17.8 / 15.3 us, 16 x 14336 at 1536 28.7 / 26.3, 10 x 28672 at 2560 58 / 55;
// at 4096 61 / 71, and at 64 5.9 / 6.5). From 16 to 48, for up to 8 rows: one tile on
// two waves, beyond 32 per unit up to 6144 (8 x 11008 at 1536 24.9 / 20.5, at 4096
// 57 / 48; 3 x 12288 at 8192 91 / 98), below it up to 1024 (8 x 5003 at 704 11.7 /
// 10.8; at 2560 19.8 / 21.2). With more rows there the reads of A count most and two tiles share
// them on four waves (16 x 8192 at 1536: 17.2, else 19.2-19.5).
enum UnmaskWordsForm { UNMASK_1_TILE_4_WAVES, UNMASK_2_TILES_4_WAVES, UNMASK_1_TILE_2_WAVES, UNMASK_2_TILES_2_WAVES };

inline UnmaskWordsForm unmask_words_form(int64_t M, int64_t N, int64_t Kp, int64_t cus) {
  if (N <= 16 * cus) return UNMASK_1_TILE_4_WAVES;
  if (N > 48 * cus) return Kp >= 128 && Kp <= 3072 ? UNMASK_2_TILES_2_WAVES : UNMASK_2_TILES_4_WAVES;
  return M <= 8 && Kp <= (N > 32 * cus ? 6144 : 1024) ? UNMASK_1_TILE_2_WAVES : UNMASK_2_TILES_4_WAVES;
}

// ---------------------------------------------------------------------------
// Tiled ring product (ring_gemm.hip): its form and split.
//
// The forms and what a product is estimated to take in each, in microseconds
// on a chip of `cus` compute units. All of it follows from two rates. A compute
// unit by itself takes 0.58 us for a stage (32 columns of the inner dimension)
// of a 128 x 128 tile; with every unit busy on uniform digits the chip is
// power-limited to 0.96 us a stage. The estimates rank the forms and are no
// predictions: over 3100 products of 65-4096 rows, 1000-28672 columns and 16-512
// stages half of them are within 7% of the time measured from 96 stages on
// (nine in ten within 22%, the low side where rows of odd length or pitch or
// few rows against many columns cost memory time) and within 14% below.
//
// FORM_128, 128 x 128 tiles: whole rounds at 0.96 us a stage, the last round at
// what its tiles leave of the power, 7 us a round for the prologue and the
// epilogue.
// FORM_128 with its last round split along K (not for the unmask epilogue,
// which needs whole products): that round's tiles run as k pieces each, added
// into C atomically, at 5 us per million words added, and C cleared first for
// a store. Only a round that would leave at least half of the units idle: a
// last round on three quarters of them runs at higher clocks, and splitting it
// measured no faster.
// FORM_64K, 64 x 128 tiles, two groups of waves splitting the stages: for
// products of at most one tile per unit. A tile costs a unit 0.45 us a stage,
// so a short product on few units takes two thirds of FORM_128's time (200 x
// 4608 x 1536 unmask: 23 against 34 us; 200 x 6144 x 4096: 57 against 80 us
// whole, 66 split in two).
// FORM_64, 64 x 128 tiles, two workgroups to a unit: half the work per tile
// and no common rounds, so products of one and a bit, or two and a bit, rounds
// of FORM_128 waste less of the last (333 x 14336 x 1536 unmask: 76 against
// 91 us; 1024 x 6144 x 1536: 80 against 92 us), but 1.5 times the operand
// traffic. Two tiles on a unit take 0.43 us a stage each when the stages are
// many (192 x 14336 x 8192, one and a third tiles per unit: 252 us against 240
// with FORM_128, 448 x 6539 x 8192 220 / 213), and a few tiles left over after
// whole turns of the units another 0.15 (640 x 6539 x 4096, 2.03 tiles per unit: 170
// against 151 us; 448 x 14336 x 2560, 3.06: 158 / 149). From eight whole rounds of
// FORM_128 on a partial last one matters less than the estimates' error and
// the traffic decides (28672 x 8192 x 1536, 56 rounds: 3050-3100 us, with
// FORM_128 2780).
enum GemmForm { FORM_128, FORM_64K, FORM_64 };

struct GemmPlan {
  GemmForm form;
  int64_t split_tiles;       // tiles of the last round that run as pieces
  int split_k;               // pieces of each
};

inline GemmPlan choose_plan(int64_t M, int64_t N, int64_t stages, int64_t cus, bool store, bool unmask) {
  const int64_t tn = (N + 127) / 128;
  const int64_t t128 = ((M + 127) / 128) * tn, t64 = ((M + 63) / 64) * tn;
  const double S = (double)stages, full = (double)(t128 / cus);
  const int64_t tail = t128 % cus;
  const double whole = full * (0.96 * S + 7.0) + 2.0;
  const auto round = [&](double share) { return (share * 0.96 > 0.58 ? share * 0.96 : 0.58) * S + 7.0; };

  GemmPlan plan{FORM_128, 0, 1};
  double best = whole + (tail > 0 ? round((double)tail / (double)cus) : 0.0);
  if (!unmask && tail > 0 && 2 * tail < cus) {
    for (int k : {2, 3, 4, 6, 8}) {
      if (stages / 2 < 2 * (int64_t)k) break;            // a piece keeps at least two stage pairs
      const double rounds = (double)((tail * k + cus - 1) / cus);
      const double words = (double)tail * k * 128.0 * (double)(M < 128 ? M : 128);
      const double work = 0.58 * S / k * rounds;
      const double read = (double)tail * (double)tn / (double)t128 * 128 * 128 * S / 5.2e6;   // B once
      const double cost = whole + (work > read ? work : read) + 7.0 * rounds + 5e-6 * words + (store ? 4.0 : 0.0);
      if (cost < best) {
        best = cost;
        plan = GemmPlan{FORM_128, tail, k};
      }
    }
  }
  if (t64 <= cus) return 0.45 * S + 3.0 < best ? GemmPlan{FORM_64K, 0, 1} : plan;
  const int64_t turns = (t64 + cus - 1) / cus;           // tiles of 64 rows per unit, rounded up
  const double power = 0.55 * (double)t64 / (double)cus * S;
  const double reach = (turns == 2 && stages >= 100 ? 0.43 : 0.38) * (double)turns * S;
  const bool left_over = turns > 2 && t64 % cus != 0 && 10 * (t64 % cus) <= cus;
  const double c64 = (power > reach ? power : reach) + 8.0 + (left_over ? 0.15 * S : 0.0);
  if (c64 < best && full < 8) plan = GemmPlan{FORM_64, 0, 1};
  return plan;
}

// ---------------------------------------------------------------------------
// Gathers with sparse matrices (sparse_terms.hip, sparse.hip)

constexpr int COLS_LDS = 80 * 1024;       // LDS for staged rows of d: two workgroups per compute unit
// Rows of P from which a workgroup of gather_cols_terms_kernel takes 64 of them
// and not 32, which halves the staging of d (8 rows of d, 2 x 14336 rows of P
// with 80 entries: 11.9 against 13.0 us); with fewer rows 32 keep twice as many
// workgroups (one row of d, 4096 rows of P: 4.3 against 5.1 us).
constexpr int64_t COLS_MANY_ROWS = 8192;

// Rows of d (M x cols, cols of the widest of nterms matrices) that a workgroup
// of gather_cols_terms_kernel stages for an N-row P: 1, 2, 4 or 8; 0: the
// matrices one after the other by gather_cols_kernel, which reads d from memory.
//
// More staged rows read the entries of P fewer times but take longer to stage
// (cols = 1536: 3.6 us for a whole call with one row, 5.8 with eight), so below
// COLS_MANY_ROWS only as many as let all workgroups run at once, two per compute
// unit (8 x 4096 with 24 entries per row: 4.4 us with two, 5.8 with eight, 6.5 with
// one, 4.8 from memory).
//
// From memory: where no row fits; a single narrow matrix, whose rows are short
// (8 x 28672 at 256 columns: 7.5 / 9.0 us); and wide ones, whose staging is paid
// by every workgroup, unless the outputs are many (from memory / staged, 4096
// columns of 64 to 80 entries 1 x 8192 4.2 / 5.6, 16 x 8192 13.9 / 13.0, 8 x 14336 15 /
// 8.3; 8192 columns of 32 to 128 16 x 8192 17 / 28, 64 x 28672 154 / 144 and 234 / 159).
inline int gather_cols_rows(int nterms, int64_t M, int64_t N, int64_t cols, int64_t cus) {
  const bool many = N > COLS_MANY_ROWS;
  if (4 * cols > COLS_LDS || (nterms == 1 && cols <= 512)) return 0;
  if (cols > 8192 || (cols > 4096 && !(many && N >= 768 * 1024 / M)) || (cols > 2048 && N < 128 * 1024 / M)) return 0;
  int mb = 1;
  while (mb < 8 && mb < M && 4 * cols * 2 * mb <= COLS_LDS && (many || (M + mb - 1) / mb * ((N + 31) / 32) > 2 * cus))
    mb *= 2;
  return mb;
}

// The same choice where the entries are known too (the binding holds the arrays;
// the call over several matrices sees device pointers alone): true for the
// matrices one after the other. `entries`: per row, of all n matrices; cols: the
// sum of theirs. Gathered from memory an output costs its entries, staged a part
// of the copy of d's rows and a fixed part besides: from memory / staged, 1536
// columns of 4 entries 64 x 8192 9.3 / 21.9 us, of 8 16 x 28672 8.6 / 18.5, of 12 39 /
// 58 for 64 x 28672, of 24 72 / 62; 1024 columns of 16 12.3 / 17.6 for 16 x 28672.
// Several matrices cost a launch each, 2.5 us (24 and 16 entries, 16 x 14336: 20.1 /
// 16.4; twice 8, 10.4 / 16.6).
inline bool gather_cols_sparse(int n, int64_t M, int64_t N, int64_t cols, int64_t entries) {
  if (cols > 2048 * (int64_t)n || (n > 1 && M * N <= 64 * 1024)) return false;
  return entries < 12 * n + cols / 200;
}

// Row gathers whose rows are drawn inside the call (rows x ncols outputs, n
// matrices, `entries` in a row of all of them, `weight`: the first is a WEIGHT
// stream): true for the matrices one after the other by gather_rows_kernel, one
// word per lane, false for all at once by gather_stream_terms_kernel, four. A
// single matrix with few outputs, or with few entries to share between the
// waves, has nothing to gain from the second, whose fixed cost is 0.3-0.8 us
// higher. Single / all at once: WEIGHT rows of 80 entries 1 x 8192 6.7 / 7.1 us, 8 x
// 5000 8.9 / 9.0, 16 x 5000 13.9 / 10.6; of 256 entries 1 x 8192 18.1 / 17.4; SPARSE rows
// of 24 8 x 8192 7.3 / 6.3, 200 x 8192 32.6 / 36.4; of 4 64 x 8192 7.2 / 10.2, of 16
// 5.1 / 5.7 for 8 x 8192. Two matrices save a launch (24 entries each, 8 x 8192: 12.2 /
// 8.9) unless the launch is long (200 x 18432: 106 / 121).
inline bool gather_rows_single(int n, bool weight, int64_t entries, int64_t rows, int64_t ncols, int64_t cus) {
  const int64_t blocks = rows * ((ncols + 255) / 256);
  if (n > 1) return entries < 32 * n && blocks > 24 * cus;
  if (entries < 20 || (!weight && blocks < cus)) return true;
  if (entries < 32) return blocks < cus || blocks > 6 * cus;
  return weight && entries <= 128 && 2 * rows * ((ncols + 63) / 64) <= 5 * cus;
}

}  // namespace mosaic
