// Ring product over Z_{2^32} on 8-bit MFMA (gfx950).
//
// Both operands arrive as balanced base-256 digits (see mosaic.h). With
// x = sum_i a_i 256^i and y = sum_j b_j 256^j,
//     x y = sum_{i+j<=3} a_i b_j 256^(i+j)   (mod 2^32),
// the ten surviving limb products of the paper's emulation (Section 6.1). The
// kernel groups them by shift s = i + j into four int32 accumulators per
// output (1, 2, 3 and 4 products) and recombines acc_0 + 2^8 acc_1 +
// 2^16 acc_2 + 2^24 acc_3 with wrap-around arithmetic in the epilogue. Each
// digit tile read from LDS feeds up to four MFMAs, so one pass over the
// operands does the work of the paper's ten INT8 GEMM launches.
//
// Accumulator range: a digit product is at most 2^14 in magnitude, so the
// four-product class acc_3 stays below 2^31 for K < 2^15; the ABI splits
// longer inner dimensions into chunks whose products are added into C
// (EPI_ACCUM).
//
// Work decomposition. A wave computes 64 rows x 32 columns as two 32 x 32
// tiles of v_mfma_i32_32x32x32_i8, holding 2 tiles x 4 shift classes x 16 =
// 128 accumulator registers; four waves side by side make a row of waves, 64
// x 128 outputs. The kernel comes in three forms (struct Form), chosen by
// choose_plan. FORM_128: two rows of waves, a 128 x 128 output tile, four
// stages in LDS; two waves per SIMD let one wave's MFMAs run while the other
// waits at a barrier or on LDS. FORM_64K: one row of waves twice, a 64 x 128
// tile whose stages the two groups of waves take in turn, three stages of
// each group in LDS; the groups' products meet in LDS at the end. FORM_64:
// one row of waves, three stages in LDS, so that two workgroups share a
// compute unit.
//
// Pipeline. The K dimension is consumed in stages of 32 columns (128 bytes
// per row per operand). NST stages of a group live in LDS at once (FORM_128:
// 4 x 32 KiB) and are filled by direct buffer-to-LDS loads issued NST stages
// ahead: stage s's fragments are read into registers during stage s-1, so
// once the barrier before stage s has passed, its slot is free and the loads
// of stage s+NST go there. Each wave runs a stage as four groups of 5 MFMAs,
// pinned by scheduling barriers: the 12 LDS reads of stage s+1's fragments
// follow the first three groups (four each), so they have completed by the
// time the next barrier needs them, and one of the wave's 4 direct loads
// follows each group (whole bench steps over the three server shapes 1.2-1.6%
// faster than with the 4 loads after the first two groups, 0.3-0.5% faster
// than with one load and three reads after every group, 4% faster than with
// six reads after each of the first two). The fragments are double-buffered in
// registers. One barrier per stage publishes stage s+1 and retires the slot
// of stage s, which the loads of stage s then refill. All stages but the
// last ones run in a loop with no tests (every stage refills and reads). LDS
// holds the A tiles of a group's slots first and then their B tiles, so that
// every fragment read addresses its slot and tile by an immediate offset from
// one of the lane's eight fragment offsets: that loop computes no addresses in
// vector registers (0.8% faster whole bench steps than slots of A and B
// together, whose third and fourth slots lie beyond the 64 KiB offset range).
//
// LDS rows are 128 bytes (8 chunks of 16 bytes); chunk c of row R sits in
// slot c ^ ((R >> 1) & 7). Sixteen lanes reading one chunk of 16 consecutive
// rows then cover all 64 banks once. A direct load writes 64 consecutive
// 16-byte slots (8 rows), so each lane fetches the chunk that belongs to its
// slot. Operand tiles are addressed through buffer descriptors that cover only
// the block's valid rows: rows past M or N read as zero and never fault.
//
// Epilogue. The recombined tile is staged in the (then idle) LDS and written
// in 16-byte chunks along rows (gemm_tile_epilogue): EPI_STORE writes C,
// EPI_ACCUM adds to C, EPI_UNMASK forms Y = Y' - K_c - C and optionally the
// dequantised fp32 result.
#include "internal.h"

namespace mosaic {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int BN = 128;              // block tile rows (B) = output columns
constexpr int BK = 32;               // columns per stage
constexpr int ROWB = BK * 4;         // bytes per row per stage
constexpr uint32_t kRsrcWord3 = 0x00020000u;

// A form of the kernel: a tile of 64 WMR x 128 outputs, WMR rows of four
// waves; KW such groups of waves, group kw taking stages kw, kw + KW, ...; NST
// stages of each group resident in LDS.
template <int WMR_, int KW_, int NST_>
struct Form {
  static constexpr int WMR = WMR_, KW = KW_, NST = NST_;
  static constexpr int BM = 64 * WMR;            // block tile rows (A)
  static constexpr int NW = 4 * WMR;             // waves of a group
  static constexpr int NT = 64 * NW * KW;        // threads
  static constexpr int OPA = BM * ROWB;          // A part of a stage in LDS
  static constexpr int OPB = BN * ROWB;          // B part (16 KiB)
  static constexpr int GRP = NST * (OPA + OPB);  // LDS of a group
  static constexpr int RB = BN / NW;             // B rows that a wave loads (of A always 16)
  static constexpr int NL = 2 + RB / 8;          // direct loads per wave per stage
  static constexpr int UN = NST % 2 ? 2 * NST : NST;   // stages per iteration of the steady loop
  static_assert(KW * GRP <= 160 * 1024 && BM * (BN + 4) * 4 <= KW * GRP, "LDS");
  static_assert(NST >= 2 && NST <= 4, "wait_loads");
};

struct Tile {
  int64_t tm, tn;
};

// Tile order. Workgroups are dispatched to the 8 XCDs round-robin by id, and
// each XCD has its own L2. The id is first remapped so that XCD x owns a
// contiguous chunk of the logical order (ids x, x+8, x+16, ... become
// consecutive), then the logical order is grouped: GROUP_M row tiles sweep
// the column tiles together. The blocks an XCD runs at once thus cover a
// compact patch of the output, whose operand slices are shared in that XCD's
// L2; XCDs that own the same columns for different row groups sweep them at
// the same pace, so B is shared in the last-level cache as well. Both maps
// are bijections of [0, tiles); correctness does not depend on dispatch
// order.
__device__ __forceinline__ int64_t xcd_order(int64_t pid, int64_t tiles) {
  constexpr int64_t NXCD = 8;
  const int64_t xcd = pid % NXCD;
  const int64_t local = pid / NXCD;
  const int64_t q = tiles / NXCD, r = tiles % NXCD;
  return xcd * q + (xcd < r ? xcd : r) + local;
}

__device__ __forceinline__ Tile tile_at(int64_t lin, int64_t tiles_m, int64_t tiles_n) {
  constexpr int64_t GROUP_M = 8;
  const int64_t per_group = GROUP_M * tiles_n;
  const int64_t group = lin / per_group;
  const int64_t first_m = group * GROUP_M;
  const int64_t gm = (tiles_m - first_m) < GROUP_M ? (tiles_m - first_m) : GROUP_M;
  const int64_t in_group = lin - group * per_group;
  Tile t;
  t.tm = first_m + in_group % gm;
  t.tn = in_group / gm;
  return t;
}

// Direct buffer-to-LDS load of 16 bytes per lane: lane l of the wave writes
// LDS bytes [lds_off + 16 l, lds_off + 16 l + 16). Issued as inline assembly
// so that the compiler, which cannot tell these writes from later LDS reads,
// does not drain every outstanding load before each read; completion is
// tracked by hand with s_waitcnt vmcnt before the barrier that publishes a
// stage. M0 (the LDS base) is set inside the same statement; nothing else in
// this kernel uses M0.
__device__ __forceinline__ void dma16(v4i rs, uint32_t lds_off, int voff, int soff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :: "s"(lds_off), "v"(voff), "s"(rs), "s"(soff) : "memory");
}

// Raw buffer descriptor over [base, base + bytes): out-of-range lanes read 0.
__device__ __forceinline__ v4i make_rsrc(const void* base, int64_t bytes) {
  const uint64_t b = (uint64_t)base;
  return v4i{(int)(uint32_t)b, (int)((uint32_t)(b >> 32) & 0xFFFFu), (int)bytes, (int)kRsrcWord3};
}

// s_waitcnt with only the vector-memory counter constrained: vmcnt(N)
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// At most n stages of this wave's NL direct loads each may still be in flight
// (n <= NST - 1 <= 3).
template <int NL>
__device__ __forceinline__ void wait_loads(int n) {
  if (n >= 3) wait_vm<3 * NL>();
  else if (n == 2) wait_vm<2 * NL>();
  else if (n == 1) wait_vm<NL>();
  else wait_vm<0>();
}

__device__ __forceinline__ int imin(int a, int b) { return a < b ? a : b; }

// Adds a TM x TN tile held in LDS (row pitch TROW words) into C with 32-bit
// atomics (wrap-around adds: exact over the ring), consecutive lanes on
// consecutive words: an atomic instruction then covers whole 128-byte lines,
// where four words per lane spread it over four times as many.
template <int TM, int TN, int NT, int TROW>
__device__ __forceinline__ void gemm_tile_atomic_add(const GemmLaunch& g, const uint32_t* tile, int64_t m0,
                                                     int64_t n0, int tid) {
  static_assert(NT % TN == 0 && TM * TN % NT == 0, "whole rows per pass");
  const int c = tid % TN;
  const int64_t n = n0 + c;
  if (n >= g.N) return;
#pragma unroll 4
  for (int r = tid / TN; r < TM; r += NT / TN) {
    const int64_t m = m0 + r;
    if (m < g.M) atomicAdd(g.c + m * g.ldc + n, tile[r * TROW + c]);
  }
}

// Workgroup b < tiles - split_tiles computes a whole tile, in the XCD-aware
// order over those tiles. The last split_tiles tiles of the logical order
// run as split_k pieces each (workgroup full + p: piece p / split_tiles of
// tile full + p % split_tiles), each piece a contiguous range of stage
// pairs, added into C atomically; C is cleared for those tiles first when the
// result is stored (launch_ring_gemm).
// SPLIT: compiled in only for launches with split tiles, so that the
// whole-tile kernel keeps a compile-time stage origin of 0.
template <class F, int EPI, bool AL, bool SPLIT>
__global__ __launch_bounds__(F::NT, 2) void ring_gemm_kernel(GemmLaunch g) {
  constexpr int BM = F::BM, NST = F::NST, OPA = F::OPA, OPB = F::OPB, NL = F::NL, UN = F::UN, KW = F::KW;
  constexpr int SB = KW * ROWB;                     // a group's bytes of a row from stage to stage
  __shared__ __attribute__((aligned(1024))) char lds_all[KW * F::GRP];

  const int64_t tiles_m = (g.M + BM - 1) / BM;
  const int64_t tiles_n = (g.N + BN - 1) / BN;
  const int64_t full = SPLIT ? tiles_m * tiles_n - g.split_tiles : tiles_m * tiles_n;
  const int total = (int)(g.Kp / BK);   // even: Kp is a multiple of 64
  const bool piece = SPLIT && (int64_t)blockIdx.x >= full;
  const int64_t p = (int64_t)blockIdx.x - full;
  const int64_t q = piece ? p / g.split_tiles : 0;
  const int64_t lin = piece ? full + (p - q * g.split_tiles) : xcd_order(blockIdx.x, full);
  const int s0 = piece ? 2 * (int)((int64_t)(total / 2) * q / g.split_k) : 0;
  const int stages_all = piece ? 2 * (int)((int64_t)(total / 2) * (q + 1) / g.split_k) - s0 : total;
  const Tile tile = tile_at(lin, tiles_m, tiles_n);
  const int64_t m0 = tile.tm * BM;
  const int64_t n0 = tile.tn * BN;
  const int64_t rows_a = (g.M - m0) < BM ? (g.M - m0) : BM;
  const int64_t rows_b = (g.N - n0) < BN ? (g.N - n0) : BN;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kw = KW > 1 ? wave_all / F::NW : 0;
  const int wave = wave_all - kw * F::NW;
  const int stages = __builtin_amdgcn_readfirstlane(stages_all / KW);               // this group's: stage s of it is stage s0 + KW s + kw
  // a group's operands start at its first stage; the ranges end where the
  // tile's rows end
  const int64_t first = (int64_t)(s0 + kw) * ROWB;
  const v4i rsa = make_rsrc(g.a + m0 * g.a_pitch + first, rows_a * g.a_pitch - first);
  const v4i rsb = make_rsrc(g.b + n0 * g.b_pitch + first, rows_b * g.b_pitch - first);
  char* const lds = lds_all + kw * F::GRP;
  const int wm = wave >> 2;
  const int wn = wave & 3;

  // direct loads: wave w fills rows 16 w + 8 q .. +8 (q = 0, 1) of A and RB w +
  // 8 q .. +8 (q < RB / 8) of B; load k: A for k = 0 and 2, else B
  int va[2], vb[F::RB / 8];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int R = wave * 16 + q * 8 + (lane >> 3);
    va[q] = R * (int)g.a_pitch + ((lane & 7) ^ ((R >> 1) & 7)) * 16;
  }
#pragma unroll
  for (int q = 0; q < F::RB / 8; ++q) {
    const int R = wave * F::RB + q * 8 + (lane >> 3);
    vb[q] = R * (int)g.b_pitch + ((lane & 7) ^ ((R >> 1) & 7)) * 16;
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  const uint32_t lds_a = lds0 + wave * 16 * ROWB, lds_b = lds0 + NST * OPA + wave * F::RB * ROWB;

  // fragment reads: lane reads row (lane % 32) of a 32-row tile, chunk
  // 4 (lane / 32) + t for digit t
  const int rr = lane & 31;
  const int f = (rr >> 1) & 7;
  int fo[8];     // A digits 0..3, B digits 0..3
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int p = ((lane >> 5) * 4 + t) ^ f;
    fo[t] = (wm * 64 + rr) * ROWB + p * 16;
    fo[4 + t] = NST * OPA + (wn * 32 + rr) * ROWB + p * 16;
  }

  v16i acc[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][s][v] = 0;

  v4i fa[2][2][4], fb[2][4];             // [register set][tile][digit], [register set][digit]

// SO: the stage's byte offset along a row
#define MOSAIC_DMA(SO, SLOT, k)                                                            \
  do {                                                                                     \
    if ((k) == 0 || (k) == 2) dma16(rsa, lds_a + (SLOT) * OPA + ((k) / 2) * 8 * ROWB, va[(k) / 2], SO); \
    else dma16(rsb, lds_b + (SLOT) * OPB + ((k) == 1 ? 0 : (k) - 2) * 8 * ROWB, vb[(k) == 1 ? 0 : (k) - 2],     \
               SO);                                                                        \
  } while (0)

#define MOSAIC_READ(SLOT, SET, idx)                                                        \
  do {                                                                                     \
    if ((idx) < 8) {                                                                       \
      const int i_ = (idx) >> 2, t_ = (idx) & 3;                                           \
      const uint4 v_ = *(const uint4*)(lds + (SLOT) * OPA + i_ * 32 * ROWB + fo[t_]);      \
      fa[SET][i_][t_] = v4i{(int)v_.x, (int)v_.y, (int)v_.z, (int)v_.w};                   \
    } else {                                                                               \
      const int t_ = (idx) - 8;                                                            \
      const uint4 v_ = *(const uint4*)(lds + (SLOT) * OPB + fo[4 + t_]);                   \
      fb[SET][t_] = v4i{(int)v_.x, (int)v_.y, (int)v_.z, (int)v_.w};                       \
    }                                                                                      \
  } while (0)

  // Keeps fragments in VGPRs (the accumulators own the AGPRs) and makes the
  // wave wait for its outstanding LDS reads of that set.
#define MOSAIC_PIN(SET)                                                                    \
  do {                                                                                     \
    _Pragma("unroll") for (int i = 0; i < 2; ++i)                                          \
    _Pragma("unroll") for (int t = 0; t < 4; ++t) asm volatile("" : "+v"(fa[SET][i][t]));  \
    _Pragma("unroll") for (int t = 0; t < 4; ++t) asm volatile("" : "+v"(fb[SET][t]));     \
  } while (0)

  // MFMA n (0..19) of a stage: tile n % 2, limb pair n / 2. The pairs run
  // grouped by the digit of B (b_0 with a_0..a_3, then b_1, b_2, b_3), so
  // consecutive MFMAs share the B fragment in runs of 8, 6, 4 and 2; the
  // matrix cores draw less power when an operand does not change, which on
  // uniform digits gave 1-7% more throughput than orders that switch both
  // operands. The two tiles alternate, so no MFMA reads the accumulator
  // written by the one just before it.
#define MOSAIC_MFMA(SET, n)                                                                \
  do {                                                                                     \
    constexpr int ta_[10] = {0, 1, 2, 3, 0, 1, 2, 0, 1, 0};                                \
    constexpr int tb_[10] = {0, 0, 0, 0, 1, 1, 1, 2, 2, 3};                                \
    const int i_ = (n) % 2, a_ = ta_[(n) / 2], b_ = tb_[(n) / 2];                          \
    acc[i_][a_ + b_] =                                                                     \
        __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[SET][i_][a_], fb[SET][b_], acc[i_][a_ + b_], 0, 0, 0); \
  } while (0)

  // group g of a stage: MFMAs 5g .. 5g+4, then its share of the direct loads
  // of stage S+NST (one load, or 2, 2, 1, 1 of six) and (g < 3) fragment reads
  // 4g .. 4g+3 of stage S+1. SLOT and NSLOT: S and S+1 modulo NST.
#define MOSAIC_STAGE(CUR, NXT, SO, SLOT, NSLOT, REFILL, NEXT)                              \
  do {                                                                                     \
    const bool refill_ = (REFILL);                                                         \
    const bool next_ = (NEXT);                                                             \
    _Pragma("unroll") for (int gq = 0; gq < 4; ++gq) {                                     \
      _Pragma("unroll") for (int u = 0; u < 5; ++u) MOSAIC_MFMA(CUR, gq * 5 + u);          \
      if (refill_) {                                                                       \
        constexpr int k0_[5] = {0, NL / 3, 2 * (NL / 3), NL == 4 ? 3 : 5, NL};             \
        _Pragma("unroll") for (int k = k0_[gq]; k < k0_[gq + 1]; ++k) MOSAIC_DMA((SO) + NST * SB, SLOT, k); \
      }                                                                                    \
      if (gq < 3 && next_) {                                                               \
        _Pragma("unroll") for (int r = 0; r < 4; ++r) MOSAIC_READ(NSLOT, NXT, 4 * gq + r); \
      }                                                                                    \
      __builtin_amdgcn_sched_barrier(0);                                                   \
    }                                                                                      \
  } while (0)

  // prologue: stages 0 .. NST-1 in flight, stage 0 published and read
#pragma unroll
  for (int s = 0; s < NST; ++s)
    if (s < stages) {
#pragma unroll
      for (int k = 0; k < NL; ++k) MOSAIC_DMA(s * SB, s, k);
    }
  if (stages > 0) {
    wait_loads<NL>(imin(NST - 1, stages - 1));
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int k = 0; k < 12; ++k) MOSAIC_READ(0, 0, k);
  }

  // Before stage S: this wave's loads of stage S+1 have landed (loads of up
  // to stage S+NST-1 issued, at most NST-2 later stages in flight) and its
  // reads of stage S have completed (the pin); the barrier then makes stage
  // S+1 visible to every wave and guarantees nobody still reads stage S's
  // slot, which stage S's loads refill with stage S+NST.
  // The steady state, where every stage refills its slot and reads the next
  // one, runs as a loop without conditions: one basic block per UN stages
  // (the slots in turn), which the scheduler interleaves freely within the
  // pinned groups (the server products 1.5-3% faster than with the tests
  // inside every stage). The last NST stages, when just those remain, run as
  // straight-line code with their waits fixed (bench steps 0.4-0.6% faster
  // than through the general loop, mostly from the short Init X and unmask
  // products); other remainders, and short stage counts, take the general
  // loop.
  int s = 0;
  for (; s + UN + NST <= stages; s += UN) {
    int so = s * SB;                    // kept a scalar: it must not merge with the vector offsets
    asm volatile("" : "+s"(so));
#pragma unroll
    for (int h = 0; h < UN; h += 2) {
      wait_vm<NL * (NST - 2)>();
      MOSAIC_PIN(0);
      __builtin_amdgcn_s_barrier();
      MOSAIC_STAGE(0, 1, so + h * SB, h % NST, (h + 1) % NST, true, true);
      wait_vm<NL * (NST - 2)>();
      MOSAIC_PIN(1);
      __builtin_amdgcn_s_barrier();
      MOSAIC_STAGE(1, 0, so + (h + 1) * SB, (h + 1) % NST, (h + 2) % NST, true, true);
    }
  }
  if (NST % 2 == 0 && s > 0 && stages - s == NST) {
    // no refills, the waits shrink as the loads in flight run out
#pragma unroll
    for (int h = 0; h < NST; h += 2) {
      wait_loads<NL>(NST - 2 - h);
      MOSAIC_PIN(0);
      __builtin_amdgcn_s_barrier();
      MOSAIC_STAGE(0, 1, 0, h % NST, (h + 1) % NST, false, true);
      if (h + 2 < NST) {
        wait_loads<NL>(NST - 3 - h);
        MOSAIC_PIN(1);
        __builtin_amdgcn_s_barrier();
        MOSAIC_STAGE(1, 0, 0, (h + 1) % NST, (h + 2) % NST, false, true);
      } else {
        MOSAIC_PIN(1);
        MOSAIC_STAGE(1, 0, 0, (h + 1) % NST, (h + 2) % NST, false, false);
      }
    }
    s = stages;
  }
  for (int slot = 0; s + 1 < stages; s += 2) {      // s is a multiple of NST here: slot 0
    const int slot1 = slot + 1 < NST ? slot + 1 : 0, slot2 = slot1 + 1 < NST ? slot1 + 1 : 0;
    int so = s * SB;
    asm volatile("" : "+s"(so));
    wait_loads<NL>(imin(NST - 2, stages - 2 - s));
    MOSAIC_PIN(0);
    __builtin_amdgcn_s_barrier();
    MOSAIC_STAGE(0, 1, so, slot, slot1, s + NST < stages, true);
    if (s + 2 < stages) wait_loads<NL>(imin(NST - 2, stages - 3 - s));
    MOSAIC_PIN(1);
    if (s + 2 < stages) __builtin_amdgcn_s_barrier();
    MOSAIC_STAGE(1, 0, so + SB, slot1, slot2, s + 1 + NST < stages, s + 2 < stages);
    slot = slot2;
  }
  if (KW > 1 && s < stages) {           // an odd count: a group's share of an even one
    MOSAIC_PIN(0);
    MOSAIC_STAGE(0, 1, 0, 0, 0, false, false);
  }
  wait_vm<0>();                         // no direct load outlives the loop
#undef MOSAIC_DMA
#undef MOSAIC_READ
#undef MOSAIC_PIN
#undef MOSAIC_MFMA
#undef MOSAIC_STAGE

  // epilogue: recombine the shift classes and write. Output layout of the
  // 32 x 32 MFMA: register v of lane l holds row 8 (v / 4) + 4 (l / 32) + v % 4,
  // column l % 32.
  // Recombine the shift classes and stage the BM x 128 tile in LDS (rows
  // padded to 132 words so the two rows a wave writes per instruction fall in
  // different banks; with two groups of waves the second adds to what the
  // first stored), then write it out in 16-byte chunks along rows: thread t
  // takes chunks t + NT k (row c / 32, columns 4 (c % 32) .. + 3), so each wave
  // instruction covers two whole 512-byte tile rows. A piece of a split tile
  // is added word by word instead (gemm_tile_atomic_add). All loads of the
  // unmask epilogue (Y', K_c, scales) are issued before its first store.
  __builtin_amdgcn_s_barrier();                 // every wave is done reading stage data
  uint32_t* ctile = (uint32_t*)lds_all;
  constexpr int TROW = BN + 4;
#pragma unroll
  for (int k = KW - 1; k >= 0; --k) {           // the last group stores its part, the others add theirs
    if (kw == k) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int r = wm * 64 + i * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
          const int c = wn * 32 + (lane & 31);
          const uint32_t val = (uint32_t)acc[i][0][v] + ((uint32_t)acc[i][1][v] << 8) +
                               ((uint32_t)acc[i][2][v] << 16) + ((uint32_t)acc[i][3][v] << 24);
          if (k == KW - 1) ctile[r * TROW + c] = val;
          else ctile[r * TROW + c] += val;
        }
      }
    }
    __syncthreads();
  }
  if (EPI != EPI_UNMASK && piece) gemm_tile_atomic_add<BM, BN, F::NT, TROW>(g, ctile, m0, n0, tid);
  else gemm_tile_epilogue<EPI, AL, BM, BN, F::NT, TROW>(g, ctile, m0, n0, tid);
}

// C = 0 over the last split_tiles tiles of the logical order (one workgroup
// per tile).
template <int BM>
__global__ __launch_bounds__(256) void clear_split_tiles_kernel(GemmLaunch g) {
  const int64_t tiles_m = (g.M + BM - 1) / BM;
  const int64_t tiles_n = (g.N + BN - 1) / BN;
  const Tile tile = tile_at(tiles_m * tiles_n - g.split_tiles + blockIdx.x, tiles_m, tiles_n);
  const int64_t m0 = tile.tm * BM, n0 = tile.tn * BN;
  for (int e = threadIdx.x; e < BM * BN; e += 256) {
    const int64_t m = m0 + e / BN, n = n0 + e % BN;
    if (m < g.M && n < g.N) g.c[m * g.ldc + n] = 0u;
  }
}

template <class F, int EPI, bool SPLIT>
void launch_form_epi(const GemmLaunch& g, dim3 grid, bool aligned, hipStream_t s) {
  if (aligned) hipLaunchKernelGGL((ring_gemm_kernel<F, EPI, true, SPLIT>), grid, dim3(F::NT), 0, s, g);
  else hipLaunchKernelGGL((ring_gemm_kernel<F, EPI, false, SPLIT>), grid, dim3(F::NT), 0, s, g);
}

// g.split_tiles and g.split_k are set.
template <class F>
hipError_t launch_form(const GemmLaunch& g, EpilogueKind epi, hipStream_t s) {
  const int64_t tiles = ((g.M + F::BM - 1) / F::BM) * ((g.N + BN - 1) / BN);
  const dim3 grid((unsigned)(tiles + g.split_tiles * (g.split_k - 1)));
  const bool aligned = gemm_epilogue_aligned(g, epi);
  if constexpr (F::BM == 128) {          // the form that splits
    if (g.split_tiles > 0) {
      if (epi == EPI_STORE) {
        hipLaunchKernelGGL(clear_split_tiles_kernel<F::BM>, dim3((unsigned)g.split_tiles), dim3(256), 0, s, g);
        launch_form_epi<F, EPI_STORE, true>(g, grid, aligned, s);
      } else {
        launch_form_epi<F, EPI_ACCUM, true>(g, grid, aligned, s);
      }
      return hipGetLastError();
    }
  }
  if (epi == EPI_STORE) launch_form_epi<F, EPI_STORE, false>(g, grid, aligned, s);
  else if (epi == EPI_ACCUM) launch_form_epi<F, EPI_ACCUM, false>(g, grid, aligned, s);
  else launch_form_epi<F, EPI_UNMASK, false>(g, grid, aligned, s);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_ring_gemm(const GemmLaunch& g, EpilogueKind epi, hipStream_t s) {
  if (g.M <= SKINNY_MAX_M) return launch_ring_gemm_skinny(g, epi, s);
  if (g.N <= 0) return hipSuccess;
  const GemmPlan p = choose_plan(g.M, g.N, g.Kp / BK, compute_units(), epi == EPI_STORE, epi == EPI_UNMASK);
  GemmLaunch gs = g;
  gs.split_tiles = p.split_tiles;
  gs.split_k = p.split_k;
  switch (p.form) {
    case FORM_64K: return launch_form<Form<1, 2, 3>>(gs, epi, s);
    case FORM_64: return launch_form<Form<1, 1, 3>>(gs, epi, s);
    default: return launch_form<Form<2, 1, 4>>(gs, epi, s);
  }
}

}  // namespace mosaic
