// Launch interfaces between the C ABI layer (abi.cpp) and the kernel files.
// Every launcher assumes its arguments were validated by the ABI layer.
#pragma once

#include <atomic>
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "device_common.h"
#include "dispatch.h"

namespace mosaic {

struct MaskLaunch {
  const void* x;
  int32_t x_dtype;        // mosaic_dtype
  int64_t x_rs, x_cs;
  const uint32_t* u;
  int64_t ldu;
  int32_t has_noise;
  RngArgs noise;
  int64_t rows, cols;
  uint32_t* out;
  int64_t ldo;
  int8_t* dig;
  int64_t pitch;
};
hipError_t launch_mask(const MaskLaunch& a, hipStream_t s);

hipError_t launch_signs(const RngArgs& r, int64_t n, int8_t* out, hipStream_t s);

hipError_t launch_sparse_csr_count(const RngArgs& r, int64_t rows, int64_t cols, int64_t* row_ptr, hipStream_t s);
hipError_t launch_sparse_csr_fill(const RngArgs& r, int64_t rows, int64_t cols, const int64_t* row_ptr,
                                  int32_t* col_idx, uint32_t* values, hipStream_t s);
hipError_t launch_sparse_gather_rows(int64_t rows, const int64_t* row_ptr, const int32_t* col_idx,
                                     const uint32_t* values, const uint32_t* d, int64_t ldd, int64_t ncols,
                                     uint32_t* c, int64_t ldc, int subtract, hipStream_t s);
hipError_t launch_sparse_stream_gather_rows(const RngArgs& r, int64_t rows, int64_t rcols, const uint32_t* d,
                                            int64_t ldd, int64_t ncols, uint32_t* c, int64_t ldc, int subtract,
                                            hipStream_t s);
// Dequantised copy of a finished ring result: y[m, n] = (float)(int32)c *
// s_rows[m] * s_cols[n] (+ bias[n]); y null for none.
struct Dequant {
  const float* s_rows;
  const float* s_cols;
  const float* bias;
  float* y;
  int64_t ld;
};
hipError_t launch_sparse_gather_cols(int64_t M, int64_t N, const int64_t* row_ptr, const int32_t* col_idx,
                                     const uint32_t* values, const uint32_t* d, int64_t ldd, uint32_t* c,
                                     int64_t ldc, int subtract, const Dequant& dq, hipStream_t s);

// The gathers over several matrices at once (sparse_terms.hip).
constexpr int MAX_TERMS = 4;
struct StreamTerm {
  RngArgs r;
  int64_t rcols;
  const uint32_t* d;
  int64_t ldd;
};
struct SparseTerm {
  const int64_t* row_ptr;
  const int32_t* col_idx;
  const uint32_t* values;
  const uint32_t* d;
  int64_t ldd, cols;
};
// One matrix, its row's entries staged in chunks: rows of any length.
hipError_t launch_gather_stream_single(const RngArgs& r, int64_t rows, int64_t rcols, const uint32_t* d, int64_t ldd,
                                       int64_t ncols, uint32_t* c, int64_t ldc, int subtract, hipStream_t s);
hipError_t launch_sparse_stream_gather_rows_terms(const StreamTerm* terms, int nterms, int64_t rows, int64_t ncols,
                                                  uint32_t* c, int64_t ldc, int subtract, hipStream_t s);
hipError_t launch_sparse_gather_cols_terms(const SparseTerm* terms, int nterms, int64_t M, int64_t N, uint32_t* c,
                                           int64_t ldc, int subtract, const Dequant& dq, hipStream_t s);

// Fixed-row-weight (WEIGHT) streams: at most WEIGHT_MAX_COLS columns (the
// row's permutation lives in LDS) and, where a row is staged whole in LDS,
// WEIGHT_MAX_T entries.
constexpr int64_t WEIGHT_MAX_COLS = 8192;
constexpr int64_t WEIGHT_MAX_T = 2048;
hipError_t launch_weighted_sample(const RngArgs& r, int64_t rows, int64_t cols, uint32_t* out, int64_t ldo,
                                  int8_t* dig, int64_t pitch, hipStream_t s);
hipError_t launch_weighted_csr_count(int64_t rows, int64_t t, int64_t* row_ptr, hipStream_t s);
hipError_t launch_weighted_csr_fill(const RngArgs& r, int64_t rows, int64_t cols, const int64_t* row_ptr,
                                    int32_t* col_idx, uint32_t* values, hipStream_t s);

hipError_t launch_mfma_probe(int mode, int64_t iters, int32_t* out, int64_t* ops, hipStream_t s);

// count = #{(i, j) : a(i, j) != b(i, j)}, or != 0 when b is null; with
// clear_count false the entries are added to a count some earlier launch on
// the stream has cleared.
hipError_t launch_count_mismatches(const uint32_t* a, int64_t lda, const uint32_t* b, int64_t ldb, int64_t rows,
                                   int64_t cols, int64_t* count, hipStream_t s, bool clear_count = true);

// Ring product C = A B^T with an epilogue.
// EPI_ACCUM adds the product to c (c += A B^T over the ring): long inner
// dimensions are split into chunks that each fit the int32 accumulators.
enum EpilogueKind { EPI_STORE = 0, EPI_UNMASK = 1, EPI_ACCUM = 2 };

// Inner-dimension chunk of one launch: the four-product shift class
// accumulates 4 K 2^14 < 2^31 only for K < 2^15; a multiple of 64.
constexpr int64_t MAX_K_CHUNK = 32704;
struct GemmLaunch {
  const int8_t* a;
  int64_t a_pitch;
  const int8_t* b;
  int64_t b_pitch;
  int64_t M, N, Kp;       // Kp: K padded to 64
  // B given as ring words: bytes of B's last row that may be read from
  // b (its valid words from b on, rounded up to 16 bytes)
  int64_t b_last;
  // A given as ring words (unmask of at most 16 rows): bytes of A's last
  // row that may be read (its K valid words)
  int64_t a_last;
  // decode kernel, EPI_ACCUM: subtract the product from c instead of adding
  bool negate;
  // tiled kernel (set by its launcher): the last split_tiles tiles run as
  // split_k pieces of the inner dimension, added into c atomically
  int64_t split_tiles;
  int32_t split_k;
  // EPI_STORE
  uint32_t* c;
  int64_t ldc;
  // EPI_UNMASK: out = ym - kc - acc (the elementwise unmask subtracts c,
  // when set, as a finished product)
  const uint32_t* ym;
  int64_t ldy;
  const uint32_t* kc;
  int64_t ldk;
  int32_t* y;
  int64_t ldo;
  const float* s_rows;
  const float* s_cols;
  const float* bias;      // optional, N entries, added to y_f32
  float* y_f32;
  int64_t ldf;
};
hipError_t launch_ring_gemm(const GemmLaunch& g, EpilogueKind epi, hipStream_t s);

// Products with at most SKINNY_MAX_M rows of A (decode shapes) run on a
// kernel that streams B once and splits K inside each workgroup.
constexpr int64_t SKINNY_MAX_M = 64;

// Compute units of the current device (cached per device id; host threads
// may call it concurrently).
inline int compute_units() {
  static std::atomic<int> cached[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) dev = 0;
  if (dev >= 0 && dev < 64) {
    const int c = cached[dev].load(std::memory_order_relaxed);
    if (c > 0) return c;
  }
  int v = 0;
  if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) v = 256;
  if (dev >= 0 && dev < 64) cached[dev].store(v, std::memory_order_relaxed);
  return v;
}
hipError_t launch_ring_gemm_skinny(const GemmLaunch& g, EpilogueKind epi, hipStream_t s);
// C = A B^T for A of at most SKINNY_MAX_M rows (digits) and B given as ring
// words (b = first word, b_pitch = row pitch in bytes, a multiple of 16);
// EPI_STORE or EPI_ACCUM.
hipError_t launch_ring_gemm_words_b(const GemmLaunch& g, EpilogueKind epi, hipStream_t s);
// Unmask (EPI_UNMASK) of at most 16 rows with A given as ring words (a,
// a_pitch bytes per row, a_last as above): the rows' digit planes are formed
// in registers as A is loaded.
hipError_t launch_unmask_words_a(const GemmLaunch& g, hipStream_t s);

// The products of A of one or two rows by dot products (ring_gemv.hip): C = A
// B^T where gemv_takes_store says so, and the unmask with A as ring words where
// gemv_takes_unmask does.
hipError_t launch_ring_gemv(const GemmLaunch& g, hipStream_t s);
hipError_t launch_unmask_gemv_words(const GemmLaunch& g, hipStream_t s);
// d = 0 (rows x cols, leading dimension ldd) and *count = 0 in one launch.
hipError_t launch_clear_check(uint32_t* d, int64_t ldd, int64_t rows, int64_t cols, int64_t* count, hipStream_t s);

// Writes one recombined ring value of C = A B^T at (m, n) through the
// epilogue: EPI_STORE stores it; EPI_UNMASK forms y = ym - val - kc and
// stores it as int32 and/or dequantised fp32 (plus the bias, added after the
// two scale products with no fused multiply-add).
template <int EPI>
__device__ __forceinline__ void gemm_epilogue(const GemmLaunch& g, int64_t m, int64_t n, uint32_t val) {
  if (EPI == EPI_STORE) {
    g.c[m * g.ldc + n] = val;
  } else if (EPI == EPI_ACCUM) {
    g.c[m * g.ldc + n] += val;
  } else {
    uint32_t y = g.ym[m * g.ldy + n] - val;
    if (g.kc != nullptr) y -= g.kc[m * g.ldk + n];
    if (g.y != nullptr) g.y[m * g.ldo + n] = (int32_t)y;
    if (g.y_f32 != nullptr) {
      const float v = (float)(int32_t)y * g.s_rows[m] * g.s_cols[n];
      g.y_f32[m * g.ldf + n] = g.bias != nullptr ? __fadd_rn(v, g.bias[n]) : v;
    }
  }
}

// True if every operand of the tile epilogue is aligned for 16-byte accesses:
// N % 4 == 0 (so a 4-column chunk is wholly inside or outside the matrix),
// 16-byte aligned base pointers and row pitches that are multiples of 4.
inline bool gemm_epilogue_aligned(const GemmLaunch& g, EpilogueKind epi) {
  auto ok = [](const void* p, int64_t ld) { return p == nullptr || ((((uintptr_t)p) & 15) == 0 && (ld & 3) == 0); };
  if (g.N % 4 != 0) return false;
  if (epi == EPI_STORE || epi == EPI_ACCUM) return ok(g.c, g.ldc);
  return ok(g.ym, g.ldy) && ok(g.kc, g.ldk) && ok(g.y, g.ldo) && ok(g.y_f32, g.ldf) &&
         (g.y_f32 == nullptr || ((((uintptr_t)g.s_cols) & 15) == 0 && (((uintptr_t)g.bias) & 15) == 0));
}

// Epilogue of a TM x TN output tile held in LDS (row pitch TROW words) by a
// workgroup of NT threads: chunks of 4 consecutive columns, thread t taking
// chunks t, t + NT, ... with 16-byte accesses; the unmask inputs of all of a
// thread's chunks are loaded first, from addresses clamped into the matrix so
// that the loads need no branches (values of chunks outside the matrix are
// discarded). AL (see gemm_epilogue_aligned): the accesses are aligned.
// Otherwise they are 16 bytes wide at word alignment, and the chunk that holds
// the last columns of an N that is not a multiple of 4 goes word by word
// (every chunk did so before, four words per lane and a load's latency per
// word: 59 against 38 us for the unmask of 333 x 5003 at rank 1536).
template <int EPI, bool AL, int TM, int TN, int NT, int TROW>
__device__ __forceinline__ void gemm_tile_epilogue(const GemmLaunch& g, const uint32_t* tile, int64_t m0,
                                                   int64_t n0, int tid) {
  using W4 = std::conditional_t<AL, u32x4, u32x4_any>;
  using F4 = std::conditional_t<AL, f32x4, f32x4_any>;
  constexpr int CPR = TN / 4;                     // chunks per tile row
  constexpr int PER = TM * CPR / NT;              // chunks per thread
  static_assert(TM * CPR % NT == 0, "tile must split evenly");
  // row m and column n of chunk k; whole: all four columns in the matrix
  const auto at = [&](int k, int& r, int64_t& m, int64_t& n) {
    const int c = tid + NT * k;
    r = c / CPR;
    m = m0 + r;
    n = n0 + 4 * (c % CPR);
  };
  // the chunk of the ragged last columns (or a matrix of fewer than 4)
  const auto ragged = [&](int r, int64_t m, int64_t n) {
    if constexpr (!AL) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n + e < g.N) gemm_epilogue<EPI>(g, m, n + e, tile[r * TROW + (int)(n - n0) + e]);
    }
  };
  int r;
  int64_t m, n;
  if (EPI == EPI_STORE) {
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      at(k, r, m, n);
      if (m >= g.M || n >= g.N) continue;
      if (!AL && n + 4 > g.N) ragged(r, m, n);
      else *(W4*)(g.c + m * g.ldc + n) = *(const u32x4*)(tile + r * TROW + (int)(n - n0));
    }
    return;
  }
  const int64_t last = AL || g.N >= 4 ? g.N - 4 : 0;   // clamp of a chunk's first column
  const bool wide = AL || g.N >= 4;                     // clamped chunks lie inside the row
  if (EPI == EPI_ACCUM) {
    u32x4 cv[PER];                                  // every c chunk is read before the first store
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      at(k, r, m, n);
      if (wide) cv[k] = *(const W4*)(g.c + min(m, g.M - 1) * g.ldc + min(n, last));
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      at(k, r, m, n);
      if (m >= g.M || n >= g.N) continue;
      if (!AL && n + 4 > g.N) ragged(r, m, n);
      else *(W4*)(g.c + m * g.ldc + n) = cv[k] + *(const u32x4*)(tile + r * TROW + (int)(n - n0));
    }
    return;
  }
  const bool dq = g.y_f32 != nullptr;
  u32x4 ymv[PER], kcv[PER];
  f32x4 scv[PER], bv[PER];
  float srv[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    at(k, r, m, n);
    m = min(m, g.M - 1);
    n = min(n, last);
    kcv[k] = u32x4{0u, 0u, 0u, 0u};
    if (!wide) continue;
    ymv[k] = *(const W4*)(g.ym + m * g.ldy + n);
    if (g.kc != nullptr) kcv[k] = *(const W4*)(g.kc + m * g.ldk + n);
    if (dq) {
      scv[k] = *(const F4*)(g.s_cols + n);
      srv[k] = g.s_rows[m];
      bv[k] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (g.bias != nullptr) bv[k] = *(const F4*)(g.bias + n);
    }
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    at(k, r, m, n);
    if (m >= g.M || n >= g.N) continue;
    if (!AL && n + 4 > g.N) {
      ragged(r, m, n);
      continue;
    }
    const u32x4 o = ymv[k] - kcv[k] - *(const u32x4*)(tile + r * TROW + (int)(n - n0));
    if (g.y != nullptr) *(W4*)((uint32_t*)g.y + m * g.ldo + n) = o;
    if (dq) {
      f32x4 f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
#pragma clang fp contract(off)
        f[e] = (float)(int32_t)o[e] * srv[k] * scv[k][e];
        if (g.bias != nullptr) f[e] = f[e] + bv[k][e];   // a rounding of its own
      }
      *(F4*)(g.y_f32 + m * g.ldf + n) = f;
    }
  }
}

// Unmask without a product term (R = 0): out = ym - kc.
hipError_t launch_unmask_elementwise(const GemmLaunch& g, hipStream_t s);

hipError_t launch_hadamard(const float* x, int64_t ldx, float* y, int64_t ldy, int64_t rows,
                           int64_t n, int log2_block, const int8_t* signs, int inverse,
                           hipStream_t s);
bool hadamard28_supported(int log2_block);
hipError_t launch_hadamard28(const float* x, int64_t ldx, float* y, int64_t ldy, int64_t rows, int log2_block,
                             const int8_t* signs, int inverse, hipStream_t s);

// Fused rotate + quantise + mask of Pi_Sec-Linear's input (secure_input.hip).
bool rotate_quantize_mask_supported(int log2_block);
hipError_t launch_rotate_quantize_mask(const float* x, int64_t ldx, int64_t rows, int64_t n, int log2_block,
                                       const int8_t* signs, int32_t qmax, const uint32_t* u, int64_t ldu,
                                       const RngArgs* noise, int8_t* out_dig, int64_t pitch, float* scale,
                                       hipStream_t s);

hipError_t launch_quantize_rows(const float* x, int64_t ldx, int64_t rows, int64_t n, int32_t qmax,
                                int32_t* q, int64_t ldq, int8_t* q_dig, int64_t q_pitch,
                                float* scale, hipStream_t s);

}  // namespace mosaic
