// Ring product C = A B^T over Z_{2^32} for A of one or two rows (one-token
// calls), by 4-way integer dot products: the short-A product of
// ring_gemm_skinny.hip without its matrix instructions, whose 16-row A tile is
// mostly padding here.
//
// With so few rows the product is bound by streaming B, and at the sizes of a
// decode step (25-110 MB) by what stands around the stream. A wave owns ROWS
// rows of B over all of K, so its sums need no other wave: C is neither
// cleared nor added into (a launch, 2-3 us, and the atomics go), and no barrier
// stands between the loads. A load instruction reads 1 KiB of one row, that is
// 16 groups of 16 columns, each lane one digit plane of its group; DEPTH of them
// per row are in flight. A lies in LDS in digit layout, every lane reads the
// four planes of its group.
//
// A lane with plane t of B forms dot_p = sum a_p b_t for the planes p = 0 .. 3 of
// A. The sum over p of dot_p 2^(8 (p + t)) needs no test for p + t <= 3: the
// other limb products carry a factor 2^32 and vanish in the shift. A lane's
// dot_p adds up at most 24 steps of 16 products of at most 2^14, below 2^23.
#include "internal.h"

namespace mosaic {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int ROWS = 2;             // rows of B per wave
constexpr int DEPTH = 4;            // loads in flight per row and lane
constexpr int NW = 4;               // waves per workgroup
constexpr int STEP = 1024;          // bytes of a row per load instruction

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* base, int64_t bytes) {
  // out-of-range offsets read as zero
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

__device__ __forceinline__ v4i load16(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
}

// 16-byte chunk c of A's row at `row` in LDS: a digit chunk as it is, or four
// ring words as their bytes of the group's four planes.
template <bool AW>
__device__ __forceinline__ void stage_chunk(char* row, int c, v4i v) {
  if (!AW) {
    *(v4i*)(row + 16 * c) = v;
  } else {
    const uint32_t w[4] = {(uint32_t)v[0], (uint32_t)v[1], (uint32_t)v[2], (uint32_t)v[3]};
    uint32_t p[4];
    digit_planes4(w, p);
    uint32_t* q = (uint32_t*)(row + 64 * (c >> 2) + 4 * (c & 3));
#pragma unroll
    for (int t = 0; t < 4; ++t) q[4 * t] = p[t];
  }
}

// MR rows of A (g.M = MR, 1 or 2). AW: A arrives as ring words (a_pitch bytes per row,
// a_last valid bytes in its last row); words past K within a row are whatever
// follows in memory, B's zero digits there cancel them. K must be non-zero.
template <int EPI, int MR, bool AW>
__global__ __launch_bounds__(64 * NW) void ring_gemv_kernel(GemmLaunch g) {
  constexpr int NV = MR * ROWS;                          // sums of a wave
  constexpr int LOGV = NV == 2 ? 1 : 2;
  static_assert(NV == 1 << LOGV && MR <= 2, "a power of two, for the reduction");
  constexpr int PRE = 4 / MR;                            // chunks of an A row per thread fetched ahead
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row_bytes = 4 * (int)g.Kp, chunks = row_bytes / 16;
  const int steps = (row_bytes + STEP - 1) / STEP, pitch = steps * STEP;
  const int64_t n0 = ((int64_t)blockIdx.x * NW + wave) * ROWS;
  const int64_t rows_b = g.N - n0 < ROWS ? g.N - n0 : ROWS;      // none if <= 0
  const __amdgpu_buffer_rsrc_t rb = rsrc(g.b + n0 * g.b_pitch, rows_b > 0 ? (rows_b - 1) * g.b_pitch + row_bytes : 0);
  const __amdgpu_buffer_rsrc_t ra = rsrc(g.a, (MR - 1) * g.a_pitch + (AW ? g.a_last : row_bytes));
  // chunk c of A's row m; what lies past A's words reads as zero
  const auto load_a = [&](int m, int c) { return load16(ra, c < chunks ? m * (int)g.a_pitch + 16 * c : 0x7FFFFFF0); };

  // the sum that this lane will hold (see the reduction), and what it is
  // subtracted from: in flight while the product is formed
  const int e = lane >> (6 - LOGV), em = e / ROWS;
  const int64_t en = n0 + e % ROWS;
  const bool writes = (lane & ((64 >> LOGV) - 1)) == 0 && en < g.N;
  uint32_t ym = 0, kc = 0;
  if (EPI == EPI_UNMASK && writes) {
    ym = g.ym[em * g.ldy + en];
    if (g.kc != nullptr) kc = g.kc[em * g.ldk + en];
  }

  // A's first chunks, then B's first loads, then A into LDS
  v4i pre[MR][PRE];
#pragma unroll
  for (int m = 0; m < MR; ++m)
#pragma unroll
    for (int q = 0; q < PRE; ++q) pre[m][q] = load_a(m, tid + 64 * NW * q);
  v4i fb[DEPTH][ROWS];
  const auto fetch = [&](v4i(&f)[ROWS], int i) {
    const int o = i * STEP + lane * 16;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) f[r] = load16(rb, o < row_bytes ? r * (int)g.b_pitch + o : 0x7FFFFFF0);
  };
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) fetch(fb[d], d);
#pragma unroll
  for (int m = 0; m < MR; ++m)
#pragma unroll
    for (int q = 0; q < PRE; ++q)
      if (tid + 64 * NW * q < chunks) stage_chunk<AW>(lds + m * pitch, tid + 64 * NW * q, pre[m][q]);
#pragma unroll
  for (int m = 0; m < MR; ++m)
    for (int c = tid + 64 * NW * PRE; c < chunks; c += 64 * NW) stage_chunk<AW>(lds + m * pitch, c, load_a(m, c));
  __syncthreads();

  int acc[MR][ROWS][4];
#pragma unroll
  for (int m = 0; m < MR; ++m)
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
      for (int p = 0; p < 4; ++p) acc[m][r][p] = 0;
  const char* al = lds + 64 * (lane >> 2);               // this lane's column group of the first step
  for (int i = 0; i < steps; i += DEPTH) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      if (i + d >= steps) break;
      // columns past Kp: B reads as zero there, whatever LDS holds
#pragma unroll
      for (int m = 0; m < MR; ++m)
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const v4i a = *(const v4i*)(al + m * pitch + (i + d) * STEP + 16 * p);
#pragma unroll
          for (int r = 0; r < ROWS; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c)
              acc[m][r][p] = __builtin_amdgcn_sdot4(a[c], fb[d][r][c], acc[m][r][p], false);
        }
      fetch(fb[d], i + d + DEPTH);
    }
  }

  // recombine, then add up over the lanes, lane bits 5 .. 0 in turn: while
  // several sums remain each exchange halves them (a lane keeps the half that
  // its bit names), so a lane ends with sum lane >> (6 - LOGV)
  uint32_t v[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int(&s)[4] = acc[k / ROWS][k % ROWS];
    v[k] = ((uint32_t)s[0] + ((uint32_t)s[1] << 8) + ((uint32_t)s[2] << 16) + ((uint32_t)s[3] << 24))
           << (8 * (lane & 3));
  }
#pragma unroll
  for (int b = 5; b >= 0; --b) {
    const int half = NV >> (6 - b);                      // sums kept in this step, 0: one is left
    if (half > 0) {
      const bool up = ((lane >> b) & 1) != 0;
#pragma unroll
      for (int k = 0; k < half; ++k) {
        const uint32_t mine = up ? v[k + half] : v[k], other = up ? v[k] : v[k + half];
        v[k] = mine + (uint32_t)__shfl_xor((int)other, 1 << b);
      }
    } else {
      v[0] += (uint32_t)__shfl_xor((int)v[0], 1 << b);
    }
  }
  if (!writes) return;
  if (EPI == EPI_STORE) {
    g.c[em * g.ldc + en] = v[0];
  } else {
    const int32_t y = (int32_t)(ym - v[0] - kc);
    if (g.y != nullptr) g.y[em * g.ldo + en] = y;
    if (g.y_f32 != nullptr) {
      const float f = (float)y * g.s_rows[em] * g.s_cols[en];
      g.y_f32[em * g.ldf + en] = g.bias != nullptr ? __fadd_rn(f, g.bias[en]) : f;
    }
  }
}

template <int EPI, int MR, bool AW>
hipError_t launch(const GemmLaunch& g, hipStream_t s) {
  const unsigned lds = (unsigned)(MR * STEP * ((4 * g.Kp + STEP - 1) / STEP));
  hipLaunchKernelGGL((ring_gemv_kernel<EPI, MR, AW>), dim3((unsigned)((g.N + NW * ROWS - 1) / (NW * ROWS))),
                     dim3(64 * NW), lds, s, g);
  return hipGetLastError();
}

template <int EPI, bool AW>
hipError_t launch_rows(const GemmLaunch& g, hipStream_t s) {
  return g.M == 1 ? launch<EPI, 1, AW>(g, s) : launch<EPI, 2, AW>(g, s);
}

}  // namespace

hipError_t launch_ring_gemv(const GemmLaunch& g, hipStream_t s) { return launch_rows<EPI_STORE, false>(g, s); }

hipError_t launch_unmask_gemv_words(const GemmLaunch& g, hipStream_t s) {
  return launch_rows<EPI_UNMASK, true>(g, s);
}

}  // namespace mosaic
