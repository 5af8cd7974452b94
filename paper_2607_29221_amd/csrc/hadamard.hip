// Random Hadamard rotation (Section 5): per block of b = 2^LOGB consecutive
// elements of a row, forward y = H_b (d * x) / sqrt(b), inverse
// y = d * (H_b x) / sqrt(b), with H_b in Sylvester order. One workgroup per
// block (several blocks to one for b <= 128): the block transform of
// fwht_block.h, then the scale (and, for the inverse, the signs) and coalesced
// 16-byte stores. The whole block stays in
// LDS (b <= 32768 floats = 128 KiB), so HBM sees one read and one write per
// element.
#include "fwht_block.h"

namespace mosaic {
namespace {

// SIGNS: 0 none, 1 applied on load (forward), 2 applied on store (inverse).
// x is read once and y written once, so both use non-temporal accesses.
template <int LOGB, int SIGNS>
__global__ __launch_bounds__((FwhtShape<LOGB, fwht_tmax(LOGB)>::T)) void fwht_kernel(
    const float* __restrict__ x, int64_t ldx, float* y, int64_t ldy, int64_t blocks_per_row,
    const int8_t* __restrict__ signs, float scale) {
  constexpr int TM = fwht_tmax(LOGB);
  using S = FwhtShape<LOGB, TM>;
  constexpr int T = S::T, E = S::E, NV = S::NV, B = S::B;
  __shared__ float sm[S::SM];
  const int t = threadIdx.x;
  const int64_t row = blockIdx.x / blocks_per_row;
  const int64_t blk = blockIdx.x - row * blocks_per_row;
  const float* xr = x + row * ldx + blk * B;
  float* yr = y + row * ldy + blk * B;
  const int8_t* sg = SIGNS ? signs + blk * B : nullptr;

  float v[E];
  fwht_load<LOGB, SIGNS == 1, true, TM>(xr, sg, v);
  const float sc = scale * fwht_transform<LOGB, TM>(sm, v);   // the transform's lane sign folded into the scale
#pragma unroll
  for (int r = 0; r < E; ++r) v[r] *= sc;
  if (SIGNS == 2) apply_signs<LOGB, TM>(sg, v);
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const f32x4 f = {v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]};
    __builtin_nontemporal_store(f, (f32x4*)yr + t + T * k);
  }
}

// Short blocks, b = 2^LOGB <= 128: a block is the work of b / 4 <= 32 lanes and
// never leaves its wave, so 1024 / b of them share a workgroup of 256 threads
// (one block per workgroup left 60 to 32 of a wave's 64 lanes idle and paid a
// launch slot for 64 to 512 bytes: 443 / 224 / 113 / 58 us at b = 16 / 32 / 64 /
// 128 for 2048 x 16384). Thread g of the grid holds columns 4 g .. 4 g + 3 of
// the rows laid end to end; n4 = n / 4 columns of four per row.
template <int LOGB, int SIGNS>
__global__ __launch_bounds__(256) void fwht_short_kernel(const float* __restrict__ x, int64_t ldx, float* y,
                                                         int64_t ldy, int64_t n4, int64_t total,
                                                         const int8_t* __restrict__ signs, float scale) {
  static_assert(FwhtShape<LOGB>::T <= 32 && FwhtShape<LOGB>::E == 4, "a block within half a wave");
  const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (g >= total) return;                             // whole blocks leave together
  const int64_t row = (g >> 32) == 0 && (n4 >> 32) == 0 ? (uint32_t)g / (uint32_t)n4 : g / n4;
  const int64_t c = g - row * n4;
  const f32x4 f = __builtin_nontemporal_load((const f32x4*)(x + row * ldx) + c);
  float v[4] = {f[0], f[1], f[2], f[3]};
  float d[4] = {1.0f, 1.0f, 1.0f, 1.0f};
  if (SIGNS != 0) {
    const char4 s4 = ((const char4*)signs)[c];
    d[0] = (float)s4.x; d[1] = (float)s4.y; d[2] = (float)s4.z; d[3] = (float)s4.w;
  }
  if (SIGNS == 1) {
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] *= d[r];
  }
  const float sc = scale * fwht_in_wave<LOGB>(v, threadIdx.x & 63);   // the lane sign folded into the scale
#pragma unroll
  for (int r = 0; r < 4; ++r) v[r] *= sc;
  if (SIGNS == 2) {
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] *= d[r];
  }
  const f32x4 o = {v[0], v[1], v[2], v[3]};
  __builtin_nontemporal_store(o, (f32x4*)(y + row * ldy) + c);
}

template <int LOGB>
void launch_fwht_short(const float* x, int64_t ldx, float* y, int64_t ldy, int64_t rows, int64_t n,
                       const int8_t* signs, int inverse, hipStream_t s) {
  const int64_t n4 = n / 4, total = rows * n4;
  const dim3 grid((unsigned)((total + 255) / 256));
  const float scale = (float)(1.0 / sqrt((double)(1 << LOGB)));
  if (signs == nullptr)
    hipLaunchKernelGGL((fwht_short_kernel<LOGB, 0>), grid, dim3(256), 0, s, x, ldx, y, ldy, n4, total, signs, scale);
  else if (!inverse)
    hipLaunchKernelGGL((fwht_short_kernel<LOGB, 1>), grid, dim3(256), 0, s, x, ldx, y, ldy, n4, total, signs, scale);
  else
    hipLaunchKernelGGL((fwht_short_kernel<LOGB, 2>), grid, dim3(256), 0, s, x, ldx, y, ldy, n4, total, signs, scale);
}

template <int LOGB>
void launch_fwht(const float* x, int64_t ldx, float* y, int64_t ldy, int64_t rows, int64_t n,
                 const int8_t* signs, int inverse, hipStream_t s) {
  constexpr int B = FwhtShape<LOGB, fwht_tmax(LOGB)>::B;
  constexpr int T = FwhtShape<LOGB, fwht_tmax(LOGB)>::T;
  const int64_t bpr = n / B;
  const int64_t grid = rows * bpr;
  const float scale = (float)(1.0 / sqrt((double)B));
  if (signs == nullptr)
    hipLaunchKernelGGL((fwht_kernel<LOGB, 0>), dim3((unsigned)grid), dim3(T), 0, s, x, ldx, y, ldy, bpr, signs,
                       scale);
  else if (!inverse)
    hipLaunchKernelGGL((fwht_kernel<LOGB, 1>), dim3((unsigned)grid), dim3(T), 0, s, x, ldx, y, ldy, bpr, signs,
                       scale);
  else
    hipLaunchKernelGGL((fwht_kernel<LOGB, 2>), dim3((unsigned)grid), dim3(T), 0, s, x, ldx, y, ldy, bpr, signs,
                       scale);
}

// The rotation in as many launches as its threads need (one up to 2^34 elements).
template <int LOGB>
hipError_t launch_parts(const float* x, int64_t ldx, float* y, int64_t ldy, int64_t rows, int64_t n,
                        const int8_t* signs, int inverse, hipStream_t s) {
  constexpr int64_t B = 1 << LOGB, T = FwhtShape<LOGB, fwht_tmax(LOGB)>::T;   // threads of a block (B / 4 if short)
  for_each_launch(rows, n / B, kMaxGridThreads / T, [&](int64_t r0, int64_t nr, int64_t b0, int64_t nb) {
    const float* xp = x + r0 * ldx + b0 * B;
    float* yp = y + r0 * ldy + b0 * B;
    const int8_t* sp = signs != nullptr ? signs + b0 * B : nullptr;
    if constexpr (LOGB <= 7) launch_fwht_short<LOGB>(xp, ldx, yp, ldy, nr, nb * B, sp, inverse, s);
    else launch_fwht<LOGB>(xp, ldx, yp, ldy, nr, nb * B, sp, inverse, s);
    return hipPeekAtLastError() == hipSuccess;
  });
  return hipGetLastError();
}

}  // namespace

hipError_t launch_hadamard(const float* x, int64_t ldx, float* y, int64_t ldy, int64_t rows, int64_t n,
                           int log2_block, const int8_t* signs, int inverse, hipStream_t s) {
  switch (log2_block) {
    case 4: return launch_parts<4>(x, ldx, y, ldy, rows, n, signs, inverse, s);
    case 5: return launch_parts<5>(x, ldx, y, ldy, rows, n, signs, inverse, s);
    case 6: return launch_parts<6>(x, ldx, y, ldy, rows, n, signs, inverse, s);
    case 7: return launch_parts<7>(x, ldx, y, ldy, rows, n, signs, inverse, s);
    case 8: return launch_parts<8>(x, ldx, y, ldy, rows, n, signs, inverse, s);
    case 9: return launch_parts<9>(x, ldx, y, ldy, rows, n, signs, inverse, s);
    case 10: return launch_parts<10>(x, ldx, y, ldy, rows, n, signs, inverse, s);
    case 11: return launch_parts<11>(x, ldx, y, ldy, rows, n, signs, inverse, s);
    case 12: return launch_parts<12>(x, ldx, y, ldy, rows, n, signs, inverse, s);
    case 13: return launch_parts<13>(x, ldx, y, ldy, rows, n, signs, inverse, s);
    case 14: return launch_parts<14>(x, ldx, y, ldy, rows, n, signs, inverse, s);
    case 15: return launch_parts<15>(x, ldx, y, ldy, rows, n, signs, inverse, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mosaic
