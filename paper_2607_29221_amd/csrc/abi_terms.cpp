// C ABI of the gathers over several sparse matrices at once (declared in
// include/mosaic.h): validation and dispatch.
#include "abi_common.h"

using namespace mosaic;

extern "C" {

mosaic_status mosaic_sparse_stream_gather_rows_terms(const mosaic_stream_term* terms, int32_t nterms, int64_t rows,
                                                     int64_t ncols, uint32_t* c, int64_t ldc, int32_t subtract,
                                                     void* stream) {
  if (rows < 0 || ncols < 0) return fail(MOSAIC_ERR_INVALID_ARG, "negative size");
  if (nterms < 0 || nterms > MAX_TERMS) return fail(MOSAIC_ERR_INVALID_ARG, "%d terms outside [0, %d]", nterms, MAX_TERMS);
  if (rows == 0 || ncols == 0 || nterms == 0) return MOSAIC_OK;
  if (terms == nullptr || c == nullptr) return fail(MOSAIC_ERR_INVALID_ARG, "NULL operand");
  if (ldc < ncols) return fail(MOSAIC_ERR_INVALID_ARG, "leading dimension < ncols");
  if (rows > kMaxGridThreads / 256 || (ncols + 63) / 64 > 65535) return fail(MOSAIC_ERR_UNSUPPORTED, "too large for one launch");
  StreamTerm t[MAX_TERMS];
  for (int l = 0; l < nterms; ++l) {
    if (terms[l].rcols < 0) return fail(MOSAIC_ERR_INVALID_ARG, "negative size");
    if (terms[l].rcols > 0 && terms[l].d == nullptr) return fail(MOSAIC_ERR_INVALID_ARG, "NULL operand");
    if (terms[l].ldd < ncols) return fail(MOSAIC_ERR_INVALID_ARG, "leading dimension < ncols");
    const mosaic_status st = check_lpn_rng(&terms[l].rng, terms[l].rcols, &t[l].r);
    if (st != MOSAIC_OK) return st;
    t[l].rcols = terms[l].rcols;
    t[l].d = terms[l].d;
    t[l].ldd = terms[l].ldd;
  }
  return hip_status(launch_sparse_stream_gather_rows_terms(t, nterms, rows, ncols, c, ldc, subtract != 0,
                                                           (hipStream_t)stream), "sparse gather launch");
}

mosaic_status mosaic_sparse_gather_cols_terms(const mosaic_sparse_term* terms, int32_t nterms, int64_t M, int64_t N,
                                              uint32_t* c, int64_t ldc, int32_t subtract, const float* s_rows,
                                              const float* s_cols, const float* bias, float* y_f32, int64_t ldf,
                                              void* stream) {
  if (M < 0 || N < 0) return fail(MOSAIC_ERR_INVALID_ARG, "negative size");
  if (nterms < 1 || nterms > MAX_TERMS) return fail(MOSAIC_ERR_INVALID_ARG, "%d terms outside [1, %d]", nterms, MAX_TERMS);
  if (M == 0 || N == 0) return MOSAIC_OK;
  if (terms == nullptr || c == nullptr) return fail(MOSAIC_ERR_INVALID_ARG, "NULL operand");
  if (ldc < N) return fail(MOSAIC_ERR_INVALID_ARG, "ldc < N");
  if (y_f32 != nullptr && (ldf < N || s_rows == nullptr || s_cols == nullptr))
    return fail(MOSAIC_ERR_INVALID_ARG, "y_f32 needs ldf >= N and both scale vectors");
  if (bias != nullptr && y_f32 == nullptr) return fail(MOSAIC_ERR_INVALID_ARG, "bias needs y_f32");
  if (M > 0x7FFFFFFF || (N + 31) / 32 > 65535) return fail(MOSAIC_ERR_UNSUPPORTED, "too large for one launch");
  SparseTerm t[MAX_TERMS];
  for (int l = 0; l < nterms; ++l) {
    const mosaic_sparse_term& x = terms[l];
    if (x.row_ptr == nullptr || x.col_idx == nullptr || x.values == nullptr || x.d == nullptr)
      return fail(MOSAIC_ERR_INVALID_ARG, "NULL operand");
    // rows of d may share memory (ldd < cols), as in the single call
    if (x.cols < 0 || x.ldd < 0) return fail(MOSAIC_ERR_INVALID_ARG, "negative cols or ldd");
    t[l] = SparseTerm{x.row_ptr, x.col_idx, x.values, x.d, x.ldd, x.cols};
  }
  hipError_t e = hipSuccess;
  for_each_launch(M, 1, kMaxGridThreads / 512, [&](int64_t r, int64_t rows, int64_t, int64_t) {
    for (int l = 0; l < nterms; ++l) t[l].d = terms[l].d + r * t[l].ldd;
    const Dequant dq{s_rows != nullptr ? s_rows + r : nullptr, s_cols, bias, y_f32 != nullptr ? y_f32 + r * ldf : nullptr,
                     ldf};
    e = launch_sparse_gather_cols_terms(t, nterms, rows, N, c + r * ldc, ldc, subtract != 0, dq, (hipStream_t)stream);
    return e == hipSuccess;
  });
  return hip_status(e, "sparse gather launch");
}

}  // extern "C"
