// Gathers over several sparse LPN matrices at once (the levels of a nested
// mask): c receives the sum over the levels in one launch and one pass over c.
//
// gather_stream_terms_kernel: c(i, k) +-= sum_l sum_j T_l(i, j) d_l(j, k) with
// T_l the stream matrix of level l, its row drawn inside the call (U_a and
// K_c). A workgroup owns 256 (or 64) columns k of one row i. The waves draw the
// levels side by side (a WEIGHT row is one wave's work), then each lane takes
// four consecutive columns, so a load instruction reads 1 KiB of a row of d_l,
// and the waves split the drawn entries; ten loads per lane are in flight, so
// a row of 80 entries is two round trips to memory. Bound by the latency of
// the draw and of those round trips for few rows, and by reading t rows of
// every d_l per row of c (8 x 160 rows of 18432 words, 94 MB: 24 us) for more.
// The levels one after the other, four bytes per lane and four loads in flight
// (gather_rows_kernel) took 38 us there.
//
// gather_cols_terms_kernel: c(m, n) +-= sum_l sum_p P_l(n, p) d_l(m, p) with
// P_l in compressed rows (S_{i+1} Q_i of unmasking). A workgroup stages MB
// rows of d_l in LDS, the MB values of a column side by side, so that an
// entry's gather is one LDS read for MB rows; eight lanes share a row of P_l,
// ten entries each in flight. Gathers from the L2 instead, one request per
// entry and row of d, and the levels one after the other took 30 us for 8 rows
// against 2 x 14336 rows of 80 entries; this kernel 12 us.
//
// Where the gathers of one matrix (sparse.hip) are ahead they run instead, one
// matrix after the other: gather_rows_single and gather_cols_rows.
#include "sparse_common.h"

namespace mosaic {
namespace {

constexpr int DRAW_MAX = 2048;   // columns of a SPARSE row drawn in one go
constexpr int INFLIGHT = 10;     // loads (entries) per lane in flight

struct DrawTerm {
  RngArgs r;
  int64_t rcols;
  const uint32_t* d;
  int64_t ldd;
  int32_t off, cap;              // LDS words: columns at off, values at off + cap, then a WEIGHT row's scratch
};
struct DrawTerms {
  int32_t n;
  DrawTerm t[MAX_TERMS];
};

// COLS columns per workgroup: COLS / 4 lanes side by side, and 1024 / COLS such
// groups that split the drawn entries.
template <int COLS>
__global__ __launch_bounds__(256) void gather_stream_terms_kernel(DrawTerms a, int64_t ncols, uint32_t* c,
                                                                  int64_t ldc, int subtract) {
  constexpr int LPG = COLS / 4, G = 256 / LPG;        // lanes per group, groups
  // entries in flight per lane; of the 16 groups at 64 columns a row of 24
  // entries gives each 1 or 2, one of 80 five, in two turns
  constexpr int U = COLS == 256 ? INFLIGHT : 3;
  extern __shared__ uint32_t lds[];
  __shared__ int count[MAX_TERMS];
  __shared__ u32x4 part[G - 1][LPG];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = COLS == 256 ? wave : tid / LPG, gl = tid % LPG;
  const int64_t i = blockIdx.x;
  const int64_t k = (int64_t)blockIdx.y * COLS + 4 * gl;
  const int64_t left = ncols - k;                     // columns of this lane: min(left, 4)
  if (tid < MAX_TERMS) count[tid] = 0;
  __syncthreads();
  for (int l = 0; l < a.n; ++l) {
    const DrawTerm& t = a.t[l];
    int32_t* col = (int32_t*)lds + t.off;
    uint32_t* val = lds + t.off + t.cap;
    if (t.r.dist == 4) {
      if (wave == l) weighted_row(t.r, i, (int)t.rcols, val + t.cap, col, val);
      if (tid == 0) count[l] = t.r.row_weight;
    } else {                                          // rcols <= DRAW_MAX = 8 x 256
      uint32_t v[DRAW_MAX / 256];
      int total = 0;
      uint32_t hits = 0;
#pragma unroll
      for (int s = 0; s < DRAW_MAX / 256; ++s) {
        const int j = 256 * s + tid;
        if (256 * s >= t.rcols) break;
        const bool nz = j < t.rcols && sparse_elem(t.r, (uint64_t)i * t.rcols + j, &v[s]);
        hits |= nz ? 1u << s : 0u;
        total += __popcll(__ballot(nz));
      }
      int base = 0;
      if (lane == 0 && total > 0) base = atomicAdd(&count[l], total);
      base = __shfl(base, 0);
#pragma unroll
      for (int s = 0; s < DRAW_MAX / 256; ++s) {
        if (256 * s >= t.rcols) break;
        const bool nz = ((hits >> s) & 1) != 0;
        const uint64_t mask = __ballot(nz);
        if (nz) {
          const int pos = base + __popcll(mask & ((1ull << lane) - 1ull));
          col[pos] = 256 * s + tid;
          val[pos] = v[s];
        }
        base += __popcll(mask);
      }
    }
  }
  __syncthreads();
  u32x4 acc = {0u, 0u, 0u, 0u};
  for (int l = 0; l < a.n; ++l) {
    const DrawTerm& t = a.t[l];
    const int32_t* col = (const int32_t*)lds + t.off;
    const uint32_t* val = lds + t.off + t.cap;
    const int n = __builtin_amdgcn_readfirstlane(count[l]);
    for (int q0 = grp; q0 < n; q0 += G * U) {
      // entries past the row's end read the first one's row again, times 0
      const uint32_t* dr[U];
      uint32_t s[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = q0 + G * u;
        const int cu = col[q < n ? q : q0];
        dr[u] = t.d + (int64_t)(COLS == 256 ? __builtin_amdgcn_readfirstlane(cu) : cu) * t.ldd + k;
        s[u] = q < n ? val[q] : 0u;
      }
      if (left >= 4) {
        u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = *(const u32x4_any*)dr[u];
#pragma unroll
        for (int u = 0; u < U; ++u) acc += s[u] * v[u];
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int e = 0; e < 3; ++e)
            if (e < left) acc[e] += s[u] * dr[u][e];
      }
    }
  }
  if (grp > 0) part[grp - 1][gl] = acc;
  __syncthreads();
  if (grp > 0 || left <= 0) return;
#pragma unroll
  for (int g = 0; g < G - 1; ++g) acc += part[g][gl];
  uint32_t* out = c + i * ldc + k;
  if (left >= 4) {
    const u32x4 o = *(const u32x4_any*)out;
    *(u32x4_any*)out = subtract ? o - acc : o + acc;
  } else {
#pragma unroll
    for (int e = 0; e < 3; ++e)
      if (e < left) out[e] = subtract ? out[e] - acc[e] : out[e] + acc[e];
  }
}

struct ColsTerms {
  int32_t n;
  SparseTerm t[MAX_TERMS];
};

// Sums acc[0 .. MB-1] over the eight lanes of a group, the group's lane bits
// 4, 2, 1 in turn: while several sums remain each exchange halves them (a lane
// keeps the half that its bit names), then the last one is added up. The
// lane's sum is that of row *row; writes: one lane per row.
template <int MB>
__device__ __forceinline__ uint32_t group_sum(uint32_t (&acc)[MB], int sub, int* row, bool* writes) {
  int m = 0;
  bool w = true;
  int cnt = MB;
#pragma unroll
  for (int bit = 4; bit >= 1; bit >>= 1) {
    const bool up = (sub & bit) != 0;
    if (cnt > 1) {
      cnt /= 2;
#pragma unroll
      for (int h = 0; h < MB / 2; ++h) {
        if (h >= cnt) break;
        const uint32_t mine = up ? acc[h + cnt] : acc[h], other = up ? acc[h] : acc[h + cnt];
        acc[h] = mine + __shfl_xor(other, bit, 8);
      }
      m += up ? cnt : 0;
    } else {
      acc[0] += __shfl_xor(acc[0], bit, 8);
      w = w && !up;
    }
  }
  *row = m;
  *writes = w;
  return acc[0];
}

// Each lane requests its first entries of a level before the workgroup waits
// for the level's rows of d, and every level's row_ptr comes first of all, so
// that the levels cost one chain of round trips and not one each.
template <int MB, int NT>
__global__ __launch_bounds__(NT) void gather_cols_terms_kernel(ColsTerms a, int64_t M, int64_t N, uint32_t* c,
                                                               int64_t ldc, int subtract, Dequant dq) {
  __shared__ __attribute__((aligned(16))) uint32_t lds[COLS_LDS / 4];
  const int tid = threadIdx.x, sub = tid & 7;
  const int64_t m0 = (int64_t)blockIdx.x * MB;
  const int64_t n = (int64_t)blockIdx.y * (NT / 8) + (tid >> 3);
  const int64_t nn = n < N ? n : N - 1;
  int64_t p[MAX_TERMS], p1[MAX_TERMS];
#pragma unroll
  for (int l = 0; l < MAX_TERMS; ++l)
    if (l < a.n) {
      p[l] = a.t[l].row_ptr[nn];
      p1[l] = a.t[l].row_ptr[nn + 1];
    }
  uint32_t acc[MB];
#pragma unroll
  for (int mm = 0; mm < MB; ++mm) acc[mm] = 0;
  int32_t base = 0;                                 // LDS words of the levels staged so far
#pragma unroll
  for (int l = 0; l < MAX_TERMS; ++l) {
    if (l >= a.n) break;
    const SparseTerm& t = a.t[l];
    uint32_t v[INFLIGHT];
    int32_t col[INFLIGHT];
    int64_t q0 = p[l] + sub;
    const int64_t end = n < N ? p1[l] : 0;
    const auto fetch = [&]() {
#pragma unroll
      for (int u = 0; u < INFLIGHT; ++u) {
        const int64_t q = q0 + 8 * u, qq = q < end ? q : end - 1;
        col[u] = t.col_idx[qq];
        v[u] = t.values[qq];
      }
    };
    if (q0 < end) fetch();
    if (base + MB * t.cols > COLS_LDS / 4) {         // start over: the rows staged before are no longer read
      __syncthreads();
      base = 0;
    }
    uint32_t* rows = lds + base;
    for (int64_t j = tid; j < t.cols; j += NT) {
      uint32_t w[MB];
#pragma unroll
      for (int mm = 0; mm < MB; ++mm) w[mm] = m0 + mm < M ? t.d[(m0 + mm) * t.ldd + j] : 0u;
#pragma unroll
      for (int mm = 0; mm < MB; ++mm) rows[j * MB + mm] = w[mm];
    }
    base += MB * (int)t.cols;
    __syncthreads();
    while (q0 < end) {
#pragma unroll
      for (int u = 0; u < INFLIGHT; ++u) {
        const uint32_t s = q0 + 8 * u < end ? v[u] : 0u;
#pragma unroll
        for (int mm = 0; mm < MB; ++mm) acc[mm] += s * rows[col[u] * MB + mm];
      }
      q0 += 8 * INFLIGHT;
      if (q0 < end) fetch();
    }
  }
  int row;
  bool writes;
  const uint32_t sum = group_sum<MB>(acc, sub, &row, &writes);
  const int64_t m = m0 + row;
  if (n >= N || m >= M || !writes) return;
  uint32_t* out = c + m * ldc + n;
  const uint32_t val = subtract ? *out - sum : *out + sum;
  *out = val;
  if (dq.y != nullptr) {
#pragma clang fp contract(off)
    // the same steps and roundings as the unmask epilogue's dequantisation
    const float f = (float)(int32_t)val * dq.s_rows[m] * dq.s_cols[n];
    dq.y[m * dq.ld + n] = dq.bias != nullptr ? f + dq.bias[n] : f;
  }
}

template <int MB>
void launch_cols(const ColsTerms& a, int64_t M, int64_t N, uint32_t* c, int64_t ldc, int subtract, const Dequant& dq,
                 hipStream_t s) {
  const unsigned gx = (unsigned)((M + MB - 1) / MB);
  if (N > COLS_MANY_ROWS)
    hipLaunchKernelGGL((gather_cols_terms_kernel<MB, 512>), dim3(gx, (unsigned)((N + 63) / 64)), dim3(512), 0, s, a,
                       M, N, c, ldc, subtract, dq);
  else
    hipLaunchKernelGGL((gather_cols_terms_kernel<MB, 256>), dim3(gx, (unsigned)((N + 31) / 32)), dim3(256), 0, s, a,
                       M, N, c, ldc, subtract, dq);
}

}  // namespace

hipError_t launch_sparse_stream_gather_rows_terms(const StreamTerm* terms, int nterms, int64_t rows, int64_t ncols,
                                                  uint32_t* c, int64_t ldc, int subtract, hipStream_t s) {
  if (rows == 0 || ncols == 0) return hipSuccess;
  DrawTerms a{};
  size_t words = 0;
  bool fits = true;
  int64_t entries = 0;                                               // a row's, of all levels (expected)
  for (int l = 0; l < nterms; ++l) {
    const StreamTerm& t = terms[l];
    const bool weight = t.r.dist == 4;
    if (t.rcols == 0 || (weight && t.r.row_weight == 0)) continue;   // an empty sum
    DrawTerm& d = a.t[a.n++];
    d.r = t.r;
    d.rcols = t.rcols;
    d.d = t.d;
    d.ldd = t.ldd;
    d.off = (int32_t)words;
    d.cap = weight ? t.r.row_weight : (int32_t)t.rcols;
    entries += weight ? t.r.row_weight : t.rcols >> (32 - t.r.sparse_shift);
    // long WEIGHT rows are drawn step by step, long SPARSE rows in chunks
    fits = fits && (weight ? t.r.row_weight <= WEIGHT_PAR_T : t.rcols <= DRAW_MAX);
    words += 2 * (size_t)(fits ? d.cap : 0) + (weight ? (weighted_scratch_bytes(t.rcols, t.r.row_weight) + 3) / 4 : 0);
  }
  if (a.n == 0) return hipSuccess;
  if (!fits || 4 * words > 48 * 1024 ||
      gather_rows_single(a.n, a.t[0].r.dist == 4, entries, rows, ncols, compute_units())) {
    for (int l = 0; l < nterms; ++l) {
      const hipError_t e = launch_gather_stream_single(terms[l].r, rows, terms[l].rcols, terms[l].d, terms[l].ldd,
                                                       ncols, c, ldc, subtract, s);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  // 64 columns per workgroup while 256 would leave compute units without one
  // (one row of 8192 columns is latency-bound: more groups share its entries)
  if (rows * ((ncols + 255) / 256) < compute_units())
    hipLaunchKernelGGL(gather_stream_terms_kernel<64>, dim3((unsigned)rows, (unsigned)((ncols + 63) / 64)), dim3(256),
                       4 * words, s, a, ncols, c, ldc, subtract);
  else
    hipLaunchKernelGGL(gather_stream_terms_kernel<256>, dim3((unsigned)rows, (unsigned)((ncols + 255) / 256)),
                       dim3(256), 4 * words, s, a, ncols, c, ldc, subtract);
  return hipGetLastError();
}

hipError_t launch_sparse_stream_gather_rows(const RngArgs& r, int64_t rows, int64_t rcols, const uint32_t* d,
                                            int64_t ldd, int64_t ncols, uint32_t* c, int64_t ldc, int subtract,
                                            hipStream_t s) {
  const StreamTerm t{r, rcols, d, ldd};
  return launch_sparse_stream_gather_rows_terms(&t, 1, rows, ncols, c, ldc, subtract, s);
}

hipError_t launch_sparse_gather_cols_terms(const SparseTerm* terms, int nterms, int64_t M, int64_t N, uint32_t* c,
                                           int64_t ldc, int subtract, const Dequant& dq, hipStream_t s) {
  if (M == 0 || N == 0) return hipSuccess;
  ColsTerms a{};
  a.n = nterms;
  int64_t cols = 0;
  for (int l = 0; l < nterms; ++l) {
    a.t[l] = terms[l];
    cols = terms[l].cols > cols ? terms[l].cols : cols;
  }
  const int mb = gather_cols_rows(nterms, M, N, cols, compute_units());
  if (mb == 0) {                                              // gather d from memory, one matrix at a time
    for (int l = 0; l < nterms; ++l) {
      const Dequant last = l + 1 == nterms ? dq : Dequant{};
      const hipError_t e = launch_sparse_gather_cols(M, N, terms[l].row_ptr, terms[l].col_idx, terms[l].values,
                                                     terms[l].d, terms[l].ldd, c, ldc, subtract, last, s);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  switch (mb) {                                               // at most COLS_LDS of staged rows
    case 1: launch_cols<1>(a, M, N, c, ldc, subtract, dq, s); break;
    case 2: launch_cols<2>(a, M, N, c, ldc, subtract, dq, s); break;
    case 4: launch_cols<4>(a, M, N, c, ldc, subtract, dq, s); break;
    default: launch_cols<8>(a, M, N, c, ldc, subtract, dq, s); break;
  }
  return hipGetLastError();
}

}  // namespace mosaic
