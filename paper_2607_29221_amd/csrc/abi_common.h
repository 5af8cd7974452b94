// Helpers of the C ABI layer: the per-thread error message, and validation and
// translation of arguments that several entry points share.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <string>

#include "../../include/mosaic.h"
#include "internal.h"

namespace mosaic {

inline thread_local std::string g_last_error;

inline mosaic_status fail(mosaic_status st, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
inline mosaic_status fail(mosaic_status st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return st;
}

inline mosaic_status hip_status(hipError_t e, const char* what) {
  if (e == hipSuccess) return MOSAIC_OK;
  return fail(MOSAIC_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

inline int64_t padded_k(int64_t k) { return 64 * ((k + 63) / 64); }

// Discrete Gaussian thresholds in extended precision (see mosaic.h).
inline void dgauss_table(double sigma, int bound, uint64_t* out) {
  long double w[2 * kMaxDgaussBound + 1];
  long double z = 0.0L;
  for (int j = -bound; j <= bound; ++j) {
    long double p;
    if (sigma == 0.0)
      p = (j == 0) ? 1.0L : 0.0L;
    else
      p = expl(-((long double)j * (long double)j) / (2.0L * (long double)sigma * (long double)sigma));
    w[j + bound] = p;
    z += p;
  }
  long double acc = 0.0L;
  for (int k = 0; k < 2 * bound; ++k) {
    acc += w[k];
    const long double v = floorl(acc / z * 4294967296.0L + 0.5L);
    out[k] = (uint64_t)v;
  }
}

inline mosaic_status rng_args(const mosaic_rng* r, RngArgs* a) {
  if (r == nullptr) return fail(MOSAIC_ERR_INVALID_ARG, "rng is NULL");
  *a = RngArgs{};
  a->k0 = (uint32_t)(r->seed & 0xFFFFFFFFu);
  a->k1 = (uint32_t)(r->seed >> 32);
  a->stream = r->stream;
  a->instance = r->instance;
  a->dist = r->dist;
  a->transposed = r->transposed != 0;
  a->sparse_shift = 32;
  switch (r->dist) {
    case MOSAIC_DIST_ZERO:
    case MOSAIC_DIST_UNIFORM:
      break;
    case MOSAIC_DIST_DGAUSS:
      if (r->bound < 0 || r->bound > kMaxDgaussBound)
        return fail(MOSAIC_ERR_INVALID_ARG, "dgauss bound %d outside [0, %d]", r->bound, kMaxDgaussBound);
      if (!(r->sigma >= 0.0) || !std::isfinite(r->sigma))
        return fail(MOSAIC_ERR_INVALID_ARG, "dgauss sigma must be finite and >= 0");
      a->bound = r->bound;
      {
        uint64_t t[2 * kMaxDgaussBound];
        dgauss_table(r->sigma, r->bound, t);
        a->dg_base = -r->bound;
        a->dg_count = 0;
        for (int k = 0; k < 2 * r->bound; ++k) {
          if (t[k] == 0) ++a->dg_base;
          else if (t[k] < (1ull << 32)) a->th[a->dg_count++] = (uint32_t)t[k];
        }
      }
      break;
    case MOSAIC_DIST_SPARSE:
      if (r->log2_inv_density < 0 || r->log2_inv_density > 31)
        return fail(MOSAIC_ERR_INVALID_ARG, "sparse log2_inv_density %d outside [0, 31]", r->log2_inv_density);
      a->sparse_shift = 32 - r->log2_inv_density;
      break;
    case MOSAIC_DIST_WEIGHT:
      if (r->row_weight < 0) return fail(MOSAIC_ERR_INVALID_ARG, "row_weight %d is negative", r->row_weight);
      a->row_weight = r->row_weight;
      break;
    default:
      return fail(MOSAIC_ERR_INVALID_ARG, "unknown distribution %d", r->dist);
  }
  return MOSAIC_OK;
}

// Digit-layout operand of rows x cols; a matrix without elements may be NULL.
inline mosaic_status check_digits(const int8_t* p, int64_t pitch, int64_t rows, int64_t cols, const char* name) {
  if (rows == 0 || cols == 0) {
    if (pitch < 0 || pitch % 64 != 0) return fail(MOSAIC_ERR_INVALID_ARG, "%s pitch must be a multiple of 64", name);
    return MOSAIC_OK;
  }
  if (p == nullptr) return fail(MOSAIC_ERR_INVALID_ARG, "%s is NULL", name);
  if (!aligned16(p)) return fail(MOSAIC_ERR_INVALID_ARG, "%s is not 16-byte aligned", name);
  if (pitch % 64 != 0 || pitch < 4 * padded_k(cols))
    return fail(MOSAIC_ERR_INVALID_ARG, "%s pitch %lld must be a multiple of 64 and >= %lld", name,
                (long long)pitch, (long long)(4 * padded_k(cols)));
  return MOSAIC_OK;
}

// A WEIGHT stream matrix of rows x cols that the row kernels can draw.
inline mosaic_status check_weighted(const mosaic_rng* r, int64_t cols) {
  if (r->transposed) return fail(MOSAIC_ERR_UNSUPPORTED, "WEIGHT streams cannot be transposed");
  if (r->row_weight < 0 || r->row_weight > cols)
    return fail(MOSAIC_ERR_INVALID_ARG, "row_weight %d outside [0, cols = %lld]", r->row_weight, (long long)cols);
  if (cols > WEIGHT_MAX_COLS || r->row_weight > WEIGHT_MAX_T)
    return fail(MOSAIC_ERR_UNSUPPORTED, "WEIGHT needs cols <= %lld and row_weight <= %lld",
                (long long)WEIGHT_MAX_COLS, (long long)WEIGHT_MAX_T);
  return MOSAIC_OK;
}

// rng of the compressed-row calls: a non-transposed SPARSE or WEIGHT stream.
inline mosaic_status check_lpn_rng(const mosaic_rng* r, int64_t cols, RngArgs* a) {
  if (r == nullptr || (r->dist != MOSAIC_DIST_SPARSE && r->dist != MOSAIC_DIST_WEIGHT) || r->transposed)
    return fail(MOSAIC_ERR_INVALID_ARG, "rng must be a non-transposed SPARSE or WEIGHT stream");
  if (r->dist == MOSAIC_DIST_WEIGHT) {
    const mosaic_status st = check_weighted(r, cols);
    if (st != MOSAIC_OK) return st;
  }
  return rng_args(r, a);
}

}  // namespace mosaic
