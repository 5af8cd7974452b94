// Draws of the sparse LPN streams shared by the kernels that store them and
// those that gather with them.
#pragma once

#include "internal.h"

namespace mosaic {

// gate and value of element e (words 2e and 2e + 1 share a Philox block)
__device__ __forceinline__ bool sparse_elem(const RngArgs& r, uint64_t e, uint32_t* val) {
  const uint4 blk = philox_block(r, e >> 1);
  const bool hi = (e & 1) != 0;
  const uint32_t gate = hi ? blk.z : blk.x;
  *val = hi ? blk.w : blk.y;
  return (r.sparse_shift >= 32) ? true : ((gate >> r.sparse_shift) == 0u);
}

// Orders the LDS accesses of one wave: they execute in program order, so only
// the compiler has to keep it.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Entries of row ``row`` of a WEIGHT stream matrix, computed by the calling
// wave alone (several waves of a workgroup can draw different rows side by
// side). scratch: weighted_scratch_bytes(cols, t) of LDS, 4-byte aligned; pos
// / val (LDS, t entries) receive the chosen column and the value of each
// step, visible to the wave on return and to others after a workgroup barrier.
//
// Step j of the partial shuffle draws k_j = j + floor(u_j (cols - j) / 2^32)
// and swaps entries j and k_j of a running permutation (the identity at
// first); its column is the entry that lands at j, i.e. entry k_j just
// before the step. Up to WEIGHT_PAR_T steps that entry is found without
// running the swaps one after the other: position p >= j has been touched
// before step j only by the steps i < j with k_i = p (the steps' own
// positions i are all below j), and the latest of them left there the entry
// that position i held just before step i. Position i in turn held i unless
// an earlier step i' < i had k_{i'} = i, in which case it held what position
// i' held before step i', and so on. So the column of step j is k_j if no
// earlier step chose k_j, else E(i) for the latest such i, with E(i) = i if
// no step before i chose position i and E(i) = E(i') for the latest such i'.
// A table over the positions counts each position's choosers (and keeps
// the first one): a step whose position has one chooser takes it; the few
// steps on positions chosen more than once (a handful per row at t = 80 of
// r = 1024) go to a short list, which answers "latest earlier chooser" for
// them and, with the table, the chains of E. Longer rows take the steps one
// by one on a permutation kept in LDS as perm[k] ^ k, so that zero-filled
// memory is the identity.
constexpr int WEIGHT_PAR_T = 256;

inline size_t weighted_scratch_bytes(int64_t cols, int64_t t) {
  return t <= WEIGHT_PAR_T ? (size_t)(4 * cols + 8 * t + 16) : (size_t)(2 * cols + 4 * t + 16);
}

__device__ __forceinline__ void weighted_row(const RngArgs& r, int64_t row, int cols, void* scratch, int32_t* pos,
                                             uint32_t* val) {
  const int t = r.row_weight;
  const int lane = threadIdx.x & 63;
  const uint64_t w0 = 2 * (uint64_t)t * (uint64_t)row;   // even: each (u, value) pair is one half block
  if (t <= WEIGHT_PAR_T) {
    uint32_t* tab = (uint32_t*)scratch;        // per position: (choosers << 16) | first chooser
    uint32_t* kk = tab + cols;                 // per step: its position
    int32_t* shared_steps = (int32_t*)(kk + t); // steps on positions with several choosers
    int* nshared = (int*)(shared_steps + t);
    uint32_t k[4];
    for (int p = lane; p < cols; p += 64) tab[p] = 0;
    if (lane == 0) *nshared = 0;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int j = lane + 64 * s;
      k[s] = 0;
      if (j < t) {
        const uint64_t w = w0 + 2 * (uint64_t)j;
        const uint4 blk = philox_block(r, w >> 2);
        const bool hi = ((w >> 1) & 1) != 0;
        const uint32_t uj = hi ? blk.z : blk.x;
        val[j] = hi ? blk.w : blk.y;
        k[s] = (uint32_t)j + (uint32_t)(((uint64_t)uj * (uint64_t)(uint32_t)(cols - j)) >> 32);
        kk[j] = k[s];
      }
    }
    wave_sync();
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int j = lane + 64 * s;
      if (j < t) {
        // the first chooser's step number goes to the low half; the others
        // only add to the count, so the two updates commute
        const uint32_t old = atomicAdd(&tab[k[s]], 0x10000u);
        if ((old >> 16) == 0) atomicOr(&tab[k[s]], (uint32_t)j);
      }
    }
    wave_sync();
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int j = lane + 64 * s;
      if (j < t && (tab[k[s]] >> 16) >= 2) shared_steps[atomicAdd(nshared, 1)] = j;
    }
    wave_sync();
    {
      const int n = *nshared;
      // latest step before `before` whose position is p, or -1
      auto latest = [&](uint32_t p, int before) -> int {
        const uint32_t e = tab[p];
        const uint32_t choosers = e >> 16;
        if (choosers == 0) return -1;
        if (choosers == 1) return ((int)(e & 0xFFFFu) < before) ? (int)(e & 0xFFFFu) : -1;
        int best = -1;
        for (int q = 0; q < n; ++q) {
          const int i = shared_steps[q];
          if (i < before && i > best && kk[i] == p) best = i;
        }
        return best;
      };
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int j = lane + 64 * s;
        if (j < t) {
          int x = latest(k[s], j);
          uint32_t col = k[s];
          if (x >= 0) {
            for (int y = latest((uint32_t)x, x); y >= 0; y = latest((uint32_t)x, x)) x = y;
            col = (uint32_t)x;
          }
          pos[j] = (int32_t)col;
        }
      }
    }
    wave_sync();
    return;
  }
  uint16_t* perm = (uint16_t*)scratch;
  uint32_t* u = (uint32_t*)scratch + ((cols + 1) >> 1);
  for (int k = lane; k < cols; k += 64) perm[k] = 0;
  for (int j = lane; j < t; j += 64) {
    const uint64_t w = w0 + 2 * (uint64_t)j;
    const uint4 blk = philox_block(r, w >> 2);
    const bool hi = ((w >> 1) & 1) != 0;
    u[j] = hi ? blk.z : blk.x;
    val[j] = hi ? blk.w : blk.y;
  }
  wave_sync();
  if (lane == 0) {
    for (int j = 0; j < t; ++j) {
      const uint32_t k = (uint32_t)j + (uint32_t)(((uint64_t)u[j] * (uint64_t)(uint32_t)(cols - j)) >> 32);
      const uint32_t a = perm[j] ^ (uint32_t)j;     // entries j and k of the running permutation
      const uint32_t b = perm[k] ^ k;
      perm[j] = (uint16_t)(b ^ (uint32_t)j);
      perm[k] = (uint16_t)(a ^ k);
      pos[j] = (int32_t)b;
    }
  }
  wave_sync();
}

}  // namespace mosaic
