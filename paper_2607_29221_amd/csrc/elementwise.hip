// Elementwise passes of the MOSAIC path: the mask pass (x + u + e -> ring
// elements and/or digit layout), sampling (the same pass with only e), the
// rotation's sign vector, and unmasking without a product term.
//
// Contiguous rows take mask_quad_kernel, transposed plaintext and samples
// mask_turn_kernel, anything else (many short ragged rows, plaintext with two
// strides, one of plaintext and noise transposed) the general mask_kernel; see
// mask_route.
#include "internal.h"

namespace mosaic {
namespace {

__device__ __forceinline__ uint32_t load_x(const void* x, int32_t dt, int64_t off) {
  switch (dt) {
    case 0: return (uint32_t)(int32_t)((const int8_t*)x)[off];
    case 1: return (uint32_t)(int32_t)((const int16_t*)x)[off];
    case 2: return (uint32_t)((const int32_t*)x)[off];
    default: return ((const uint32_t*)x)[off];
  }
}

// General form. One thread owns one 16-column digit group of one row: it reads
// 16 plaintext values, 16 ring words of u, draws 16 noise values (four Philox
// blocks when the group starts on a block boundary), and writes the four
// 16-byte digit planes of the group.
__global__ __launch_bounds__(256) void mask_kernel(MaskLaunch a, int64_t groups) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t i = gid / groups;
  const int64_t g = gid - i * groups;
  if (i >= a.rows) return;
  const int64_t j0 = 16 * g;
  const bool full = (j0 + 16 <= a.cols);
  uint32_t v[16];

  // plaintext
  if (a.x != nullptr) {
    if (full && a.x_dtype == 0 && a.x_cs == 1 &&
        ((((uintptr_t)a.x) + i * a.x_rs + j0) & 15) == 0) {
      const uint4 w = *(const uint4*)((const int8_t*)a.x + i * a.x_rs + j0);
      const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int b = 0; b < 4; ++b) v[4 * q + b] = (uint32_t)(int32_t)(int8_t)(ww[q] >> (8 * b));
    } else {
#pragma unroll
      for (int b = 0; b < 16; ++b) {
        const int64_t j = j0 + b;
        v[b] = (j < a.cols) ? load_x(a.x, a.x_dtype, i * a.x_rs + j * a.x_cs) : 0u;
      }
    }
  } else {
#pragma unroll
    for (int b = 0; b < 16; ++b) v[b] = 0u;
  }

  // precomputed ring mask
  if (a.u != nullptr) {
    const uint32_t* up = a.u + i * a.ldu + j0;
    if (full && ((((uintptr_t)up) & 15) == 0)) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint4 w = ((const uint4*)up)[q];
        v[4 * q + 0] += w.x; v[4 * q + 1] += w.y; v[4 * q + 2] += w.z; v[4 * q + 3] += w.w;
      }
    } else {
#pragma unroll
      for (int b = 0; b < 16; ++b)
        if (j0 + b < a.cols) v[b] += up[b];
    }
  }

  // noise drawn in the pass
  if (a.has_noise) {
    const RngArgs& r = a.noise;
    if (!r.transposed) {
      const uint64_t e0 = (uint64_t)i * (uint64_t)a.cols + (uint64_t)j0;
      if (full && (e0 & 3) == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          uint32_t e4[4];
          sample4_aligned(r, e0 + 4 * q, e4);
          v[4 * q + 0] += e4[0]; v[4 * q + 1] += e4[1]; v[4 * q + 2] += e4[2]; v[4 * q + 3] += e4[3];
        }
      } else {
        for (int b = 0; b < 16; ++b)
          if (j0 + b < a.cols) v[b] += sample_elem(r, e0 + b);
      }
    } else {
      // logical matrix is cols x rows; output (i, j) is its element (j, i)
      for (int b = 0; b < 16; ++b) {
        const int64_t j = j0 + b;
        if (j < a.cols) v[b] += sample_elem(r, (uint64_t)j * (uint64_t)a.rows + (uint64_t)i);
      }
    }
  }

  // padding columns of a digit group are zero
  if (!full) {
#pragma unroll
    for (int b = 0; b < 16; ++b)
      if (j0 + b >= a.cols) v[b] = 0u;
  }

  if (a.out != nullptr) {
    uint32_t* op = a.out + i * a.ldo + j0;
    if (full && ((((uintptr_t)op) & 15) == 0)) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        ((uint4*)op)[q] = make_uint4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    } else {
      for (int b = 0; b < 16; ++b)
        if (j0 + b < a.cols) op[b] = v[b];
    }
  }

  if (a.dig != nullptr) {
    uint32_t planes[4][4];  // [digit t][word q]: digit t of elements 4q .. 4q+3
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t w[4] = {digit_word(v[4 * q]), digit_word(v[4 * q + 1]),
                             digit_word(v[4 * q + 2]), digit_word(v[4 * q + 3])};
      uint32_t t4[4];
      digit_transpose4(w, t4);
#pragma unroll
      for (int t = 0; t < 4; ++t) planes[t][q] = t4[t];
    }
    uint4* dp = (uint4*)(a.dig + i * a.pitch + 64 * g);
#pragma unroll
    for (int t = 0; t < 4; ++t) dp[t] = make_uint4(planes[t][0], planes[t][1], planes[t][2], planes[t][3]);
  }
}

// The mask pass over contiguous rows: four consecutive lanes share one
// 16-column digit group, lane q owning columns 4q .. 4q+3. A lane reads 4
// plaintext values, one 16-byte word of u and one Philox block of noise, and
// forms the four digit words of its columns; a transpose across the four
// lanes (quad shuffles) then hands lane q digit plane q of the whole group, so
// each lane stores 16 contiguous bytes and a wave stores 1 KiB contiguous per
// instruction. Every input is read once and every output written once, so
// all accesses are non-temporal (they do not displace cached data).
// XT: 0 none, 1 int8, 2 int32 or ring words, 3 int16. F: which of u, noise,
// out and digits are present (MQ_* bits). Presence is a compile-time choice:
// with run-time tests the loads of x and u were issued one round trip apart.
//
// RAGGED: rows of any length at any element address (a row length, pitch or
// base that is not a multiple of 4 elements), and int16. The loads and stores
// keep their width at element alignment; only the row's last, partial lane
// goes element by element. A row's first noise element then sits at word
// s = (row cols) % 4 of a Philox block, the same s for the whole workgroup
// (one row each): every lane draws one block and takes its neighbour's through
// LDS, and only the last wave draws one more, so the draws grow by a quarter
// where two blocks a lane would double them. The general kernel above, one
// thread per 16 columns with 4-byte accesses 64 bytes apart and one Philox
// block per element, took 39 us for 1000 x 5003 codes with u and noise (60 MB)
// against 15 us here.
enum { MQ_U = 1, MQ_NOISE = 2, MQ_OUT = 4, MQ_DIG = 8 };
// Workgroup b covers 1024-column slice b % slices of row b / slices, so
// consecutive workgroups stream consecutive memory (79% of the HBM peak
// measured for the int8 mask pass, against 67% with rows varying fastest).
template <int XT, int F, bool RAGGED>
__global__ __launch_bounds__(256) void mask_quad_kernel(MaskLaunch a, int64_t lanes_per_row, uint32_t slices) {
  static_assert(XT != 3 || RAGGED, "int16 rows take the ragged form");
  const uint32_t b = blockIdx.x;
  const int64_t i = b / slices;                     // row
  const int64_t l = (int64_t)(b - (uint32_t)i * slices) * 256 + threadIdx.x;   // lane: columns 4 l .. 4 l + 3
  const int64_t j0 = 4 * l;
  uint32_t v[4] = {0u, 0u, 0u, 0u};
  if constexpr (!RAGGED) {
    if (l >= lanes_per_row) return;                 // whole quads leave together (lanes_per_row % 4 == 0)
    const bool valid = j0 < a.cols;                 // cols % 4 == 0: all four columns valid or all padding
    if (valid) {
      u32x4 xw = {0u, 0u, 0u, 0u}, uw = {0u, 0u, 0u, 0u};
      if (XT == 1) {
        const uint32_t w = __builtin_nontemporal_load((const uint32_t*)((const int8_t*)a.x + i * a.x_rs + j0));
#pragma unroll
        for (int b = 0; b < 4; ++b) xw[b] = (uint32_t)(int32_t)(int8_t)(w >> (8 * b));
      } else if (XT == 2) {
        xw = __builtin_nontemporal_load((const u32x4*)((const uint32_t*)a.x + i * a.x_rs + j0));
      }
      if (F & MQ_U) uw = __builtin_nontemporal_load((const u32x4*)(a.u + i * a.ldu + j0));
#pragma unroll
      for (int b = 0; b < 4; ++b) v[b] = xw[b] + uw[b];
      if (F & MQ_NOISE) {
        uint32_t e[4];
        sample4_aligned(a.noise, (uint64_t)i * (uint64_t)a.cols + (uint64_t)j0, e);
        v[0] += e[0]; v[1] += e[1]; v[2] += e[2]; v[3] += e[3];
      }
      if (F & MQ_OUT) {
        const u32x4 ov = {v[0], v[1], v[2], v[3]};
        __builtin_nontemporal_store(ov, (u32x4*)(a.out + i * a.ldo + j0));
      }
    }
  } else {
    const int64_t left = a.cols - j0;               // columns present: min(left, 4), none if <= 0
    if (left >= 4) {
      u32x4 xw = {0u, 0u, 0u, 0u}, uw = {0u, 0u, 0u, 0u};
      if (XT == 1) {
        const uint32_t w = __builtin_nontemporal_load((const u32_any*)((const int8_t*)a.x + i * a.x_rs + j0));
#pragma unroll
        for (int b = 0; b < 4; ++b) xw[b] = (uint32_t)(int32_t)(int8_t)(w >> (8 * b));
      } else if (XT == 2) {
        xw = __builtin_nontemporal_load((const u32x4_any*)((const uint32_t*)a.x + i * a.x_rs + j0));
      } else if (XT == 3) {
        const auto w = __builtin_nontemporal_load((const u32x2_any*)((const int16_t*)a.x + i * a.x_rs + j0));
        xw = u32x4{(uint32_t)(int32_t)(int16_t)w[0], (uint32_t)((int32_t)w[0] >> 16),
                   (uint32_t)(int32_t)(int16_t)w[1], (uint32_t)((int32_t)w[1] >> 16)};
      }
      if (F & MQ_U) uw = __builtin_nontemporal_load((const u32x4_any*)(a.u + i * a.ldu + j0));
#pragma unroll
      for (int b = 0; b < 4; ++b) v[b] = xw[b] + uw[b];
    } else {
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        if (b >= left) continue;
        if (XT == 1) v[b] = (uint32_t)(int32_t)((const int8_t*)a.x)[i * a.x_rs + j0 + b];
        else if (XT == 2) v[b] = ((const uint32_t*)a.x)[i * a.x_rs + j0 + b];
        else if (XT == 3) v[b] = (uint32_t)(int32_t)((const int16_t*)a.x)[i * a.x_rs + j0 + b];
        if (F & MQ_U) v[b] += a.u[i * a.ldu + j0 + b];
      }
    }
    if (F & MQ_NOISE) {
      const RngArgs& r = a.noise;
      const uint64_t row0 = (uint64_t)i * (uint64_t)a.cols;     // element of the row's first column
      uint32_t e[4];
      if (r.dist == 3) {
        sparse4_any(r, row0 + (uint64_t)j0, e);
      } else {
        const int s = (int)(row0 & 3);
        const uint64_t blk = (row0 >> 2) + (uint64_t)l;
        const uint4 p = philox_block(r, blk);
        e[0] = p.x; e[1] = p.y; e[2] = p.z; e[3] = p.w;
        if (s != 0) {                                 // uniform: one row per workgroup
          __shared__ uint4 blocks[257];
          blocks[threadIdx.x] = p;
          if (threadIdx.x == 255) blocks[256] = philox_block(r, blk + 1);
          __syncthreads();
          const uint4 q = blocks[threadIdx.x + 1];
          const uint32_t w[8] = {p.x, p.y, p.z, p.w, q.x, q.y, q.z, q.w};
#pragma unroll
          for (int b = 0; b < 4; ++b) e[b] = s == 1 ? w[b + 1] : s == 2 ? w[b + 2] : w[b + 3];
        }
        if (r.dist == 2) dgauss4(r, e);
      }
#pragma unroll
      for (int b = 0; b < 4; ++b) v[b] += e[b];
    }
    if (l >= lanes_per_row) return;                 // whole quads leave together
    if (left >= 4) {
      if (F & MQ_OUT) {
        const u32x4 ov = {v[0], v[1], v[2], v[3]};
        __builtin_nontemporal_store(ov, (u32x4_any*)(a.out + i * a.ldo + j0));
      }
    } else {
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        if (b >= left) v[b] = 0u;                   // padding columns of a digit group are zero
        else if (F & MQ_OUT) a.out[i * a.ldo + j0 + b] = v[b];
      }
    }
  }
  if (F & MQ_DIG) {
    uint32_t o[4];
    quad_digit_planes(v, (int)(l & 3), o);
    const u32x4 ov = {o[0], o[1], o[2], o[3]};
    __builtin_nontemporal_store(ov, (u32x4*)(a.dig + i * a.pitch + 16 * l));
  }
}

template <int XT, int F, bool RAGGED>
void launch_mask_quad(uint32_t slices, const MaskLaunch& a, int64_t lanes_per_row, hipStream_t s) {
  hipLaunchKernelGGL((mask_quad_kernel<XT, F, RAGGED>), dim3((unsigned)(a.rows * slices)), dim3(256), 0, s, a,
                     lanes_per_row, slices);
}

typedef void (*MaskQuadLaunch)(uint32_t, const MaskLaunch&, int64_t, hipStream_t);

// At least one output is present: F is 4 to 15.
template <int XT, bool RG>
MaskQuadLaunch mask_quad_for(int f) {
  static const MaskQuadLaunch table[12] = {
      launch_mask_quad<XT, 4, RG>,  launch_mask_quad<XT, 5, RG>,  launch_mask_quad<XT, 6, RG>,
      launch_mask_quad<XT, 7, RG>,  launch_mask_quad<XT, 8, RG>,  launch_mask_quad<XT, 9, RG>,
      launch_mask_quad<XT, 10, RG>, launch_mask_quad<XT, 11, RG>, launch_mask_quad<XT, 12, RG>,
      launch_mask_quad<XT, 13, RG>, launch_mask_quad<XT, 14, RG>, launch_mask_quad<XT, 15, RG>};
  return table[(f & 15) - 4];
}

// Mask pass whose plaintext lies transposed in memory (consecutive rows i of
// the result are consecutive elements, x_rs = 1) and whose noise, if any, is
// that of the transposed matrix: element (i, j) of the result is x[i + j x_cs]
// plus element e = j rows + i of the stream. A workgroup owns a 64 x 64 tile
// of the result: it reads (or draws) four consecutive i of one j per lane,
// 256 contiguous bytes of words per j, turns the tile through LDS, and then
// adds u and writes words and digits as the kernel above does, four columns
// per lane, 256 contiguous bytes per row. The pitch of 65 words makes both
// sides of the exchange free of bank conflicts: the writes of a wave fall in
// banks 4 a + j + b, its reads in banks i + 4 q + b. Bound by HBM; the general
// kernel, whose lanes read x at a row pitch from each other and drew a Philox
// block per element, took 126 us for 4096 x 4096 words to digits (128 MiB,
// 1.1 TB/s) against 28 us here, and 22 us for a transposed 4096 x 1536
// uniform sample against 10.
template <int XT, bool NOISE>
__global__ __launch_bounds__(256) void mask_turn_kernel(MaskLaunch a, uint32_t tiles_j) {
  constexpr int LD = 65;
  __shared__ uint32_t t[64 * LD];
  const int64_t ti = blockIdx.x / tiles_j;
  const int64_t i0 = 64 * ti, j0 = 64 * (int64_t)(blockIdx.x - (uint32_t)ti * tiles_j);
  const int lane4 = 4 * (threadIdx.x & 15);            // first of this lane's four elements of a tile line
  const int line = threadIdx.x >> 4;                   // tile line within a pass of 16
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int jj = 16 * p + line;
    const int64_t j = j0 + jj, i = i0 + lane4;
    const int64_t left = j < a.cols ? a.rows - i : 0;  // elements present: min(left, 4)
    uint32_t v[4] = {0u, 0u, 0u, 0u};
    if (XT != 0) {
      const int64_t off = i + j * a.x_cs;
      if (left >= 4) {
        if (XT == 1) {
          const uint32_t w = __builtin_nontemporal_load((const u32_any*)((const int8_t*)a.x + off));
#pragma unroll
          for (int b = 0; b < 4; ++b) v[b] = (uint32_t)(int32_t)(int8_t)(w >> (8 * b));
        } else if (XT == 2) {
          const u32x4 w = __builtin_nontemporal_load((const u32x4_any*)((const uint32_t*)a.x + off));
#pragma unroll
          for (int b = 0; b < 4; ++b) v[b] = w[b];
        } else {
          const auto w = __builtin_nontemporal_load((const u32x2_any*)((const int16_t*)a.x + off));
          v[0] = (uint32_t)(int32_t)(int16_t)w[0]; v[1] = (uint32_t)((int32_t)w[0] >> 16);
          v[2] = (uint32_t)(int32_t)(int16_t)w[1]; v[3] = (uint32_t)((int32_t)w[1] >> 16);
        }
      } else {
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          if (b >= left) continue;
          if (XT == 1) v[b] = (uint32_t)(int32_t)((const int8_t*)a.x)[off + b];
          else if (XT == 2) v[b] = ((const uint32_t*)a.x)[off + b];
          else v[b] = (uint32_t)(int32_t)((const int16_t*)a.x)[off + b];
        }
      }
    }
    if (NOISE && left > 0) {
      uint32_t e[4];
      sample4_any(a.noise, (uint64_t)j * (uint64_t)a.rows + (uint64_t)i, e);
#pragma unroll
      for (int b = 0; b < 4; ++b) v[b] += e[b];
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) t[(lane4 + b) * LD + jj] = v[b];
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int ii = 16 * p + line;
    const int64_t i = i0 + ii, j = j0 + lane4;
    if (i >= a.rows) break;                            // the 16 lanes of a row leave together
    const int64_t left = a.cols - j;
    uint32_t v[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) v[b] = b < left ? t[ii * LD + lane4 + b] : 0u;
    if (a.u != nullptr) {
      const uint32_t* up = a.u + i * a.ldu + j;
      if (left >= 4) {
        const u32x4 w = __builtin_nontemporal_load((const u32x4_any*)up);
#pragma unroll
        for (int b = 0; b < 4; ++b) v[b] += w[b];
      } else {
#pragma unroll
        for (int b = 0; b < 4; ++b)
          if (b < left) v[b] += up[b];
      }
    }
    if (a.out != nullptr) {
      uint32_t* op = a.out + i * a.ldo + j;
      if (left >= 4) {
        const u32x4 ov = {v[0], v[1], v[2], v[3]};
        __builtin_nontemporal_store(ov, (u32x4_any*)op);
      } else {
#pragma unroll
        for (int b = 0; b < 4; ++b)
          if (b < left) op[b] = v[b];
      }
    }
    if (a.dig != nullptr) {                            // the row's padding columns lie in its last tile
      uint32_t o[4];
      quad_digit_planes(v, threadIdx.x & 3, o);
      const u32x4 ov = {o[0], o[1], o[2], o[3]};
      __builtin_nontemporal_store(ov, (u32x4*)(a.dig + i * a.pitch + 4 * j));
    }
  }
}

template <int XT>
void launch_mask_turn(const MaskLaunch& a, uint32_t tiles_i, uint32_t tiles_j, hipStream_t s) {
  const dim3 grid(tiles_i * tiles_j);
  if (a.has_noise) hipLaunchKernelGGL((mask_turn_kernel<XT, true>), grid, dim3(256), 0, s, a, tiles_j);
  else hipLaunchKernelGGL((mask_turn_kernel<XT, false>), grid, dim3(256), 0, s, a, tiles_j);
}

__global__ __launch_bounds__(256) void signs_kernel(RngArgs r, int64_t n, int8_t* out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t e0 = 4 * i;
  if (e0 >= n) return;
  const uint4 w = philox_block(r, (uint64_t)i);
  const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (e0 + q < n) out[e0 + q] = (ww[q] >> 31) ? (int8_t)-1 : (int8_t)1;
}

// count = 0, ahead of the workgroups that add their partial counts.
__global__ void zero_count_kernel(int64_t* count) { *count = 0; }

// Differing entries of two rows x cols matrices (b null: nonzero entries
// of a): each thread compares
// 4-column groups (grid-stride), a wave and then the workgroup sum their
// counts, and one atomic per workgroup adds the sum to count.
__global__ __launch_bounds__(256) void count_mismatches_kernel(const uint32_t* a, int64_t lda, const uint32_t* b,
                                                               int64_t ldb, int64_t rows, int64_t cols,
                                                               int64_t* count) {
  __shared__ unsigned part[4];
  unsigned n = 0;
  const int64_t per_row = (cols + 3) / 4;
  const int64_t groups = rows * per_row;
  for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < groups; q += (int64_t)gridDim.x * 256) {
    const int64_t i = q / per_row;
    const int64_t j = (q - i * per_row) * 4;
    const uint32_t* ar = a + i * lda + j;
    const uint32_t* br = b != nullptr ? b + i * ldb + j : nullptr;
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (j + c < cols) n += ar[c] != (b != nullptr ? br[c] : 0u) ? 1u : 0u;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) n += __shfl_xor(n, off);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = n;
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned t = part[0] + part[1] + part[2] + part[3];
    if (t != 0) atomicAdd((unsigned long long*)count, (unsigned long long)t);
  }
}

// y = ym - kc - c elementwise (kc, c optional). c may share memory with y or
// y_f32 element for element: each thread reads its element of c before it
// writes that element.
__global__ __launch_bounds__(256) void unmask_elementwise_kernel(GemmLaunch g) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t i = gid / g.N;
  const int64_t j = gid - i * g.N;
  if (i >= g.M) return;
  uint32_t v = g.ym[i * g.ldy + j];
  if (g.kc != nullptr) v -= g.kc[i * g.ldk + j];
  if (g.c != nullptr) v -= g.c[i * g.ldc + j];
  if (g.y != nullptr) g.y[i * g.ldo + j] = (int32_t)v;
  if (g.y_f32 != nullptr) {
    const float f = (float)(int32_t)v * g.s_rows[i] * g.s_cols[j];
    g.y_f32[i * g.ldf + j] = g.bias != nullptr ? __fadd_rn(f, g.bias[j]) : f;
  }
}

}  // namespace

hipError_t launch_mask(const MaskLaunch& a, hipStream_t s) {
  if (a.rows <= 0 || a.cols <= 0) return hipSuccess;
  MaskShape m{};
  m.rows = a.rows;
  m.cols = a.cols;
  m.has_x = a.x != nullptr;
  m.x_row = a.x_cs == 1;
  m.x_turned = a.x_rs == 1;
  m.has_noise = a.has_noise != 0;
  m.noise_transposed = a.noise.transposed != 0;
  m.digits = a.dig != nullptr;
  m.aligned = a.cols % 4 == 0 &&
              (a.x == nullptr || (a.x_dtype == 0 && a.x_rs % 4 == 0 && ((uintptr_t)a.x & 3) == 0) ||
               (a.x_dtype >= 2 && a.x_rs % 4 == 0 && ((uintptr_t)a.x & 15) == 0)) &&
              (a.u == nullptr || (a.ldu % 4 == 0 && ((uintptr_t)a.u & 15) == 0)) &&
              (a.out == nullptr || (a.ldo % 4 == 0 && ((uintptr_t)a.out & 15) == 0));
  const MaskRoute route = mask_route(m, compute_units());
  const int xt = a.x == nullptr ? 0 : a.x_dtype == 0 ? 1 : a.x_dtype == 1 ? 3 : 2;
  if (route == MASK_QUAD || route == MASK_QUAD_RAGGED) {
    const int64_t lanes_per_row = m.digits ? 64 * ((a.cols + 63) / 64) / 4 : 4 * ((a.cols + 15) / 16);
    const int f = (a.u != nullptr ? MQ_U : 0) | (a.has_noise ? MQ_NOISE : 0) | (a.out != nullptr ? MQ_OUT : 0) |
                  (a.dig != nullptr ? MQ_DIG : 0);
    MaskQuadLaunch go;
    if (route == MASK_QUAD)
      go = xt == 0 ? mask_quad_for<0, false>(f) : xt == 1 ? mask_quad_for<1, false>(f) : mask_quad_for<2, false>(f);
    else
      go = xt == 0 ? mask_quad_for<0, true>(f) : xt == 1 ? mask_quad_for<1, true>(f)
         : xt == 2 ? mask_quad_for<2, true>(f) : mask_quad_for<3, true>(f);
    go((uint32_t)mask_quad_slices(m), a, lanes_per_row, s);
  } else if (route == MASK_TURN) {
    const uint32_t ti = (uint32_t)((a.rows + 63) / 64), tj = (uint32_t)((a.cols + 63) / 64);
    if (xt == 0) launch_mask_turn<0>(a, ti, tj, s);
    else if (xt == 1) launch_mask_turn<1>(a, ti, tj, s);
    else if (xt == 3) launch_mask_turn<3>(a, ti, tj, s);
    else launch_mask_turn<2>(a, ti, tj, s);
  } else {
    const int64_t groups = m.digits ? (64 * ((a.cols + 63) / 64)) / 16 : (a.cols + 15) / 16;
    const int64_t blocks = (a.rows * groups + 255) / 256;
    hipLaunchKernelGGL(mask_kernel, dim3((unsigned)blocks), dim3(256), 0, s, a, groups);
  }
  return hipGetLastError();
}

hipError_t launch_signs(const RngArgs& r, int64_t n, int8_t* out, hipStream_t s) {
  const int64_t threads = (n + 3) / 4;
  if (threads == 0) return hipSuccess;
  hipLaunchKernelGGL(signs_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, r, n, out);
  return hipGetLastError();
}

hipError_t launch_count_mismatches(const uint32_t* a, int64_t lda, const uint32_t* b, int64_t ldb, int64_t rows,
                                   int64_t cols, int64_t* count, hipStream_t s, bool clear_count) {
  if (clear_count) hipLaunchKernelGGL(zero_count_kernel, dim3(1), dim3(1), 0, s, count);
  const int64_t groups = rows * ((cols + 3) / 4);
  if (groups == 0) return hipGetLastError();
  // about 2 groups per thread, at most 1024 workgroups
  int64_t grid = (groups + 511) / 512;
  if (grid > 1024) grid = 1024;
  hipLaunchKernelGGL(count_mismatches_kernel, dim3((unsigned)grid), dim3(256), 0, s, a, lda, b, ldb, rows, cols,
                     count);
  return hipGetLastError();
}

hipError_t launch_unmask_elementwise(const GemmLaunch& g, hipStream_t s) {
  const int64_t threads = g.M * g.N;
  if (threads == 0) return hipSuccess;
  hipLaunchKernelGGL(unmask_elementwise_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, g);
  return hipGetLastError();
}

}  // namespace mosaic
