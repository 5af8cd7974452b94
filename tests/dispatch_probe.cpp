// The dispatch rules (csrc/dispatch.h) behind a C interface, for the tests.
#include "../paper_2607_29221_amd/csrc/dispatch.h"

using namespace mosaic;

extern "C" {

// flags: 1 plaintext, 2 its rows contiguous, 4 its columns, 8 aligned, 16
// noise, 32 noise transposed, 64 digits
int mask_route_of(int64_t rows, int64_t cols, int flags, int64_t cus) {
  MaskShape a{};
  a.rows = rows;
  a.cols = cols;
  a.has_x = (flags & 1) != 0;
  a.x_row = (flags & 2) != 0;
  a.x_turned = (flags & 4) != 0;
  a.aligned = (flags & 8) != 0;
  a.has_noise = (flags & 16) != 0;
  a.noise_transposed = (flags & 32) != 0;
  a.digits = (flags & 64) != 0;
  return mask_route(a, cus);
}

int gemv_takes(int64_t M, int64_t N, int64_t Kp, int unmask) {
  return unmask != 0 ? gemv_takes_unmask(M, N, Kp) : gemv_takes_store(M, N, Kp);
}

int unmask_words_form_of(int64_t M, int64_t N, int64_t Kp, int64_t cus) {
  return unmask_words_form(M, N, Kp, cus);
}

int gather_cols_rows_of(int nterms, int64_t M, int64_t N, int64_t cols, int64_t cus) {
  return gather_cols_rows(nterms, M, N, cols, cus);
}

int gather_cols_sparse_of(int n, int64_t M, int64_t N, int64_t cols, int64_t entries) {
  return gather_cols_sparse(n, M, N, cols, entries);
}

int gather_rows_single_of(int n, int weight, int64_t entries, int64_t rows, int64_t ncols, int64_t cus) {
  return gather_rows_single(n, weight != 0, entries, rows, ncols, cus);
}

// epilogue: 0 store, 1 accumulate, 2 unmask
void gemm_plan_of(int64_t M, int64_t N, int64_t Kp, int epilogue, int64_t cus, int64_t out[3]) {
  const GemmPlan p = choose_plan(M, N, Kp / 32, cus, epilogue == 0, epilogue == 2);
  out[0] = p.form;
  out[1] = p.split_tiles;
  out[2] = p.split_k;
}

void launches_of(int64_t rows, int64_t units, int64_t most, int (*f)(int64_t, int64_t, int64_t, int64_t)) {
  for_each_launch(rows, units, most, [&](int64_t r, int64_t nr, int64_t u, int64_t nu) { return f(r, nr, u, nu) != 0; });
}

}  // extern "C"
