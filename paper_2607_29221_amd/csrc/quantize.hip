// Per-row fixed-point quantisation of Pi_Sec-Linear (Section 5 protocol box):
// s = max |row| / qmax (1 for an all-zero row), q = round-half-even(x / s),
// both in fp32 with correctly rounded division. One block per row: a max
// reduction, then the codes are written as int32 and/or in the digit layout
// (sign-extended into the ring, zero padding).
#include "internal.h"

namespace mosaic {
namespace {

// Four consecutive floats of a row of n starting at column 4 c, at 16-byte
// alignment or (RAGGED) at any float; the columns past the end are 0. In a
// ragged row only the last chunk can be partial.
template <bool RAGGED, bool NT>
__device__ __forceinline__ f32x4 load_chunk(const float* __restrict__ xr, int64_t c, int64_t n) {
  if (!RAGGED) return NT ? __builtin_nontemporal_load((const f32x4*)xr + c) : ((const f32x4*)xr)[c];
  const float* p = xr + 4 * c;
  if (4 * c + 4 <= n) return NT ? (f32x4)__builtin_nontemporal_load((const f32x4_any*)p) : (f32x4)*(const f32x4_any*)p;
  f32x4 f = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (4 * c + i < n) f[i] = p[i];
  return f;
}

// Stores codes v of chunk c (columns 4 c .. 4 c + 3) of a row of n.
template <bool RAGGED, bool NT>
__device__ __forceinline__ void store_codes(int32_t* qr, int64_t c, int64_t n, const uint32_t v[4]) {
  const u32x4 ov = {v[0], v[1], v[2], v[3]};
  if (!RAGGED) {
    if (NT) __builtin_nontemporal_store(ov, (u32x4*)(qr + 4 * c));
    else *(u32x4*)(qr + 4 * c) = ov;
  } else if (4 * c + 4 <= n) {
    if (NT) __builtin_nontemporal_store(ov, (u32x4_any*)(qr + 4 * c));
    else *(u32x4_any*)(qr + 4 * c) = ov;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (4 * c + i < n) qr[4 * c + i] = (int32_t)v[i];
  }
}

// Long rows: thread c handles columns 4 c .. 4 c + 3 with one float4 load, so every
// load and store instruction of a wave covers one contiguous KiB. Pass 1
// reduces max |x| over the row (wave shuffles, then one LDS word per wave);
// pass 2 re-reads the row (now in L2), divides by the fp32 scale, rounds half
// to even and stores int32 codes with int4 stores and/or digit planes: the
// four lanes of a quad hold one 16-column group, and a quad shuffle hands
// each lane one 16-byte plane to store. Padding columns up to the next
// multiple of 64 get zero digits.
template <bool RAGGED>
__global__ __launch_bounds__(256) void quantize_rows_vec_kernel(const float* __restrict__ x, int64_t ldx,
                                                                int64_t n, int32_t qmax, int32_t* q, int64_t ldq,
                                                                int8_t* q_dig, int64_t q_pitch, float* scale) {
  __shared__ float red[4];
  const int64_t row = blockIdx.x;
  const float* xr = x + row * ldx;
  const int64_t nv = (n + 3) / 4;
  float m = 0.0f;
  for (int64_t c = threadIdx.x; c < nv; c += 256) {
    const f32x4 f = load_chunk<RAGGED, false>(xr, c, n);
    m = fmaxf(m, fmaxf(fmaxf(fabsf(f[0]), fabsf(f[1])), fmaxf(fabsf(f[2]), fabsf(f[3]))));
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  const float amax = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  const float s = (amax > 0.0f) ? amax / (float)qmax : 1.0f;
  if (threadIdx.x == 0 && scale != nullptr) scale[row] = s;

  const int64_t nchunks = q_dig ? 16 * ((n + 63) / 64) : nv;   // a multiple of 4 with digits
  for (int64_t c = threadIdx.x; c < nchunks; c += 256) {        // quads stay together (256 % 4 == 0)
    uint32_t v[4] = {0u, 0u, 0u, 0u};
    if (c < nv) {
      const f32x4 f = load_chunk<RAGGED, false>(xr, c, n);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = (uint32_t)(int32_t)rintf(f[i] / s);
      if (q != nullptr) store_codes<RAGGED, false>(q + row * ldq, c, n, v);
    }
    if (q_dig != nullptr) {
      uint32_t o[4];
      quad_digit_planes(v, (int)(c & 3), o);
      *(uint4*)(q_dig + row * q_pitch + 16 * c) = make_uint4(o[0], o[1], o[2], o[3]);
    }
  }
}

// Rows of at most 4 NT NV elements: the row is read once, with non-temporal
// loads, and kept in registers (thread t holds columns 4 (t + NT k) .. + 3,
// k < NV) between the max reduction and the code pass; stores are
// non-temporal. Same arithmetic and output layout as the kernel above.
// RAGGED: a row length, pitch or base that is not a multiple of 4 floats; the
// accesses stay 16 bytes wide at float alignment and the last chunk of a row
// goes float by float. (One thread per 16 columns, 4-byte accesses 64 bytes
// apart and a second read of the row, which these rows took before, needed
// 41 us for 1000 x 5003 floats to int32 codes, 40 MB, against 9 us here.)
template <int NT, int NV, bool RAGGED>
__global__ __launch_bounds__(NT) void quantize_rows_reg_kernel(const float* __restrict__ x, int64_t ldx,
                                                               int64_t n, int32_t qmax, int32_t* q, int64_t ldq,
                                                               int8_t* q_dig, int64_t q_pitch, float* scale) {
  constexpr int NW = NT / 64;
  __shared__ float red[NW];
  const int t = threadIdx.x;
  const int64_t row = blockIdx.x;
  const float* xr = x + row * ldx;
  const int64_t nv = (n + 3) / 4;
  f32x4 f[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int64_t c = t + NT * k;
    f[k] = c < nv ? load_chunk<RAGGED, true>(xr, c, n) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  float m = 0.0f;
#pragma unroll
  for (int k = 0; k < NV; ++k)
    m = fmaxf(m, fmaxf(fmaxf(fabsf(f[k][0]), fabsf(f[k][1])), fmaxf(fabsf(f[k][2]), fabsf(f[k][3]))));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  if ((t & 63) == 0) red[t >> 6] = m;
  __syncthreads();
  float amax = red[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) amax = fmaxf(amax, red[w]);
  const float s = (amax > 0.0f) ? amax / (float)qmax : 1.0f;
  if (t == 0 && scale != nullptr) scale[row] = s;

  const int64_t nchunks = q_dig ? 16 * ((n + 63) / 64) : nv;   // <= NT NV; a multiple of 4 with digits
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int64_t c = t + NT * k;
    if (c >= nchunks) break;                                     // uniform per quad (NT % 4 == 0)
    uint32_t v[4] = {0u, 0u, 0u, 0u};
    if (c < nv) {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = (uint32_t)(int32_t)rintf(f[k][i] / s);
      if (q != nullptr) store_codes<RAGGED, true>(q + row * ldq, c, n, v);
    }
    if (q_dig != nullptr) {
      uint32_t o[4];
      quad_digit_planes(v, (int)(c & 3), o);
      const u32x4 ov = {o[0], o[1], o[2], o[3]};
      __builtin_nontemporal_store(ov, (u32x4*)(q_dig + row * q_pitch + 16 * c));
    }
  }
}

struct QuantizeLaunch {
  const float* x;
  int64_t ldx, rows, n;
  int32_t qmax;
  int32_t* q;
  int64_t ldq;
  int8_t* q_dig;
  int64_t q_pitch;
  float* scale;
};

template <int NT, int NV, bool RAGGED>
void launch_quantize_reg(const QuantizeLaunch& a, hipStream_t s) {
  hipLaunchKernelGGL((quantize_rows_reg_kernel<NT, NV, RAGGED>), dim3((unsigned)a.rows), dim3(NT), 0, s, a.x, a.ldx, a.n,
                     a.qmax, a.q, a.ldq, a.q_dig, a.q_pitch, a.scale);
}

// Register-resident rows: 256 threads up to n = 16384, 1024 threads up to
// 65536; longer rows are read twice.
template <bool RAGGED>
void launch_quantize(const QuantizeLaunch& a, hipStream_t s) {
  if (a.n <= 1024) launch_quantize_reg<256, 1, RAGGED>(a, s);
  else if (a.n <= 2048) launch_quantize_reg<256, 2, RAGGED>(a, s);
  else if (a.n <= 4096) launch_quantize_reg<256, 4, RAGGED>(a, s);
  else if (a.n <= 8192) launch_quantize_reg<256, 8, RAGGED>(a, s);
  else if (a.n <= 16384) launch_quantize_reg<256, 16, RAGGED>(a, s);
  else if (a.n <= 32768) launch_quantize_reg<1024, 8, RAGGED>(a, s);
  else if (a.n <= 65536) launch_quantize_reg<1024, 16, RAGGED>(a, s);
  else
    hipLaunchKernelGGL((quantize_rows_vec_kernel<RAGGED>), dim3((unsigned)a.rows), dim3(256), 0, s, a.x, a.ldx, a.n,
                       a.qmax, a.q, a.ldq, a.q_dig, a.q_pitch, a.scale);
}

}  // namespace

hipError_t launch_quantize_rows(const float* x, int64_t ldx, int64_t rows, int64_t n, int32_t qmax, int32_t* q,
                                int64_t ldq, int8_t* q_dig, int64_t q_pitch, float* scale, hipStream_t s) {
  if (rows == 0) return hipSuccess;
  // digits are 16-byte aligned in every row (checked by the caller)
  const bool aligned = n % 4 == 0 && ldx % 4 == 0 && ((uintptr_t)x & 15) == 0 &&
                       (q == nullptr || (ldq % 4 == 0 && ((uintptr_t)q & 15) == 0));
  // a workgroup per row, of 1024 threads at most
  for_each_launch(rows, 1, kMaxGridThreads / 1024, [&](int64_t r, int64_t part, int64_t, int64_t) {
    const QuantizeLaunch p{x + r * ldx, ldx, part, n, qmax, q != nullptr ? q + r * ldq : nullptr, ldq,
                           q_dig != nullptr ? q_dig + r * q_pitch : nullptr, q_pitch, scale != nullptr ? scale + r : nullptr};
    if (aligned) launch_quantize<false>(p, s);
    else launch_quantize<true>(p, s);
    return hipPeekAtLastError() == hipSuccess;
  });
  return hipGetLastError();
}

}  // namespace mosaic
