// Building blocks of the kernels fed by LDS DMA (conv_dma.hip):
// pipeline shapes, the LDS tile layouts and their MFMA operand reads, DMA
// slots, the stage ring and its main loop.
#pragma once
#include <type_traits>

#include "common.h"
#include "internal.h"

namespace fg {
namespace dma {

constexpr unsigned kOOB = 0x80000000u;   // beyond any tensor: loads zero

// Pipeline shape: TM x TN output tile, BK-deep reduction stages, NS of them in
// the LDS ring, WGM x WGN waves each owning (TM/WGM) x (TN/WGN).
template <int BK_, int NS_, int WGM_, int WGN_, int TM_, int TN_>
struct Pipe {
  static constexpr int BK = BK_, NS = NS_, WGM = WGM_, WGN = WGN_, TM = TM_, TN = TN_;
  static constexpr int NW = WGM * WGN, NT = 64 * NW;
  static constexpr int WM = TM / WGM, WN = TN / WGN;
  static constexpr int FM = WM / 32, FN = WN / 32;
  static constexpr int KS = BK / 16;                 // MFMA steps per stage
  static constexpr int A_BYTES = TM * BK * 2, B_BYTES = TN * BK * 2;  // per stage
  static constexpr int PA = A_BYTES / 1024 / NW;     // DMA instrs per wave
  static constexpr int PB = B_BYTES / 1024 / NW;
  static constexpr int CPR = BK / 8;                 // 16-byte chunks per row
  static constexpr int RBA = 2 * TM, RBB = 2 * TN;   // mn-major row bytes
  // waves per SIMD: those of the workgroups whose rings fit the 160 KiB of LDS
  static constexpr int WPE = 160 * 1024 / (NS * (A_BYTES + B_BYTES)) * NW / 4;
  static_assert(A_BYTES == 1024 * NW * PA && B_BYTES == 1024 * NW * PB,
                "DMA instructions must divide among waves");
};
// Square tiles of the large kernels.
template <int BK_, int NS_, int WGM_, int WGN_, int T_ = 256>
struct K : Pipe<BK_, NS_, WGM_, WGN_, T_, T_> {
  using Base = Pipe<BK_, NS_, WGM_, WGN_, T_, T_>;
  static constexpr int T = T_;
  static constexpr int TILE_BYTES = Base::A_BYTES;   // per operand per stage
  static constexpr int PW = Base::PA;                // DMA instrs per operand
  static constexpr int RB = 2 * T;                   // mn-major row bytes
};
constexpr int kRsrcFlags = 0x00020000;   // raw buffer, 32-bit data format

typedef short v4s __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4s lds_v4s;
typedef __attribute__((address_space(3))) void lds_void;

// k-major: 16-byte chunk c of tile row `row` (bytes). 64-byte rows (BK 32)
// permute the 4 chunks by g(row); 128-byte rows (BK 64) the 8 chunks.
// mn-major: byte xor of reduction row k, below 256 so that rows of 256 bytes
// take it too. MX = 1: 64-byte blocks permuted by k & 3 (conflict-free
// transposing reads; rows of 128 bytes, two to a turn of the 64 banks, by bit 1
// of k); MX = 0: 32-byte blocks permuted by (k & 3) | bit 3 of k
// (two-way conflicts), kept for the halo kernel's weights, whose register
// allocation spills into its main loop with the other permutation.
template <int BK>
__device__ __forceinline__ int kmaj_swz(int row) {
  return BK == 32 ? ((row >> 2) & 3) : ((row ^ (row >> 3)) & 7);
}
template <int BK>
__device__ __forceinline__ int kmaj_off(int row, int c) {
  return row * (2 * BK) + ((c ^ kmaj_swz<BK>(row)) << 4);
}
template <int RB, int MX>
__device__ __forceinline__ int mn_xor(int k) {
  if (RB == 128) return ((k >> 1) & 1) << 6;
  return MX ? (k & 3) << 6 : ((k & 3) | (((k >> 3) & 1) << 2)) << 5;
}
template <int RB, int MX = 1>
__device__ __forceinline__ int mnmaj_off(int k, int n) {  // bytes, n % 4 == 0
  return k * RB + ((2 * n) ^ mn_xor<RB, MX>(k));
}

// Workgroup barrier without a memory fence. __syncthreads() would add a
// release fence, which waits for every outstanding LDS-DMA load (vmcnt(0))
// and so drains the ring; ordering is established instead by each wave's
// explicit vmcnt wait on its own loads before it arrives here. The empty asm
// statements keep the compiler from moving LDS accesses across the barrier.
__device__ __forceinline__ void barrier_nofence() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// s_waitcnt with only vmcnt constrained (gfx9 encoding).
template <int N>
__device__ __forceinline__ void wait_vm() {
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | (((N >> 4) & 3) << 14));
}

__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t rs, uint8_t *lds,
                                      unsigned voff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void *)lds, 16, voff, 0, 0, 0);
}

// Tile order across the chip. Workgroups are handed to the 8 XCDs (each with
// its own L2) round-robin by launch index L; tile v = (L % 8) * per + L / 8
// gives each XCD a contiguous run of the tile sequence, in which neighbours
// share operands (the output channels of one column tile, the halo rows of
// adjacent column tiles, one reduction chunk), so they are fetched into that
// XCD's L2 once. The grid is 8 * per one-dimensional; indices past the tile
// count exit.
// `order` (data convolutions): the phases and splits of a tile come fastest
// (kOutputMajor), or the position tiles do, so that an XCD keeps a share of the
// weights rather than of the input (kWeightMajor); kCostly is kWeightMajor with
// tile v = L, for launches whose tiles differ in cost and are listed costliest
// first.
enum { kOutputMajor = 0, kWeightMajor = 1, kCostly = 2 };
struct TileMap {
  int32_t n0, n1, n2;  // tile counts, fastest first
  int32_t per;         // ceil(n0 * n1 * n2 / 8)
  int32_t order;
  __device__ __forceinline__ bool decode(int L, int &i0, int &i1, int &i2) const {
    const int v = order == kCostly ? L : (L & 7) * per + (L >> 3);
    if (v >= n0 * n1 * n2) return false;
    i0 = v % n0;
    const int r = v / n0;
    i1 = r % n1;
    i2 = r / n1;
    return true;
  }
};

// Unsigned division by a divisor fixed per launch, as a multiply-high and two
// shifts (Granlund and Montgomery, "Division by invariant integers using
// multiplication", 1994): exact for every 32-bit dividend.
struct FastDiv {
  uint32_t magic;
  int32_t s1, s2;
  __device__ __forceinline__ unsigned div(unsigned n) const {
    const unsigned t = __umulhi(magic, n);
    return (t + ((n - t) >> s1)) >> s2;
  }
};
inline FastDiv make_fastdiv(uint32_t d) {
  int l = 0;
  while ((1ull << l) < d) ++l;
  const uint64_t m = ((1ull << 32) * ((1ull << l) - d)) / d + 1;
  return {(uint32_t)m, l ? 1 : 0, l ? l - 1 : 0};
}
struct WgradDiv {
  FastDiv pq, q;  // by p * q and by q
};

// MFMA operand of a 32-row block starting at `base` for reduction step ks.
template <int BK, bool KMAJOR, int RB = 512, int MX = 1>
__device__ __forceinline__ u32x4 frag(const uint8_t *tile, int base, int ks,
                                      int lane) {
  if (KMAJOR) {
    return *reinterpret_cast<const u32x4 *>(
        tile + kmaj_off<BK>(base + (lane & 31), 2 * ks + (lane >> 5)));
  } else {
    const int g = lane >> 4, m = lane & 15;
    const int k = 8 * (g >> 1) + (m >> 2) + 16 * ks;
    const int n = base + 16 * (g & 1) + 4 * (m & 3);
    v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_v4s *)(tile + mnmaj_off<RB, MX>(k, n)));
    v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_v4s *)(tile + mnmaj_off<RB, MX>(k + 4, n)));
    u32x2 a = __builtin_bit_cast(u32x2, lo), b = __builtin_bit_cast(u32x2, hi);
    return u32x4{a[0], a[1], b[0], b[1]};
  }
}

// Fragments of one 16-deep reduction step for this wave.
template <class C>
struct Frags {
  u32x4 a[C::FM], b[C::FN];
};

template <class C, bool AK, bool BKM>
__device__ __forceinline__ void load_frags(Frags<C> &f, const uint8_t *ta,
                                           const uint8_t *tb, int ks, int wm0,
                                           int wn0, int lane) {
#pragma unroll
  for (int i = 0; i < C::FM; ++i)
    f.a[i] = frag<C::BK, AK, C::RBA>(ta, wm0 + 32 * i, ks, lane);
#pragma unroll
  for (int j = 0; j < C::FN; ++j)
    f.b[j] = frag<C::BK, BKM, C::RBB>(tb, wn0 + 32 * j, ks, lane);
}

template <class C>
__device__ __forceinline__ void mma(f32x16 (&acc)[C::FM][C::FN],
                                    const Frags<C> &f) {
#pragma unroll
  for (int i = 0; i < C::FM; ++i)
#pragma unroll
    for (int j = 0; j < C::FN; ++j) acc[i][j] = mfma32(f.a[i], f.b[j], acc[i][j]);
}

// s_waitcnt with only lgkmcnt (LDS) constrained to 0.
__device__ __forceinline__ void wait_lds() {
  __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));
}

// Position of this lane's DMA slots (one per wave instruction jj) in a
// k-major tile (row, reduction offset of the chunk) and in an mn-major tile
// (reduction row within the stage, tile column). Each instruction fills 1 KiB
// of LDS: 512/BK k-major rows or 1024/RB mn-major rows. P instructions per
// wave, RB bytes per mn-major row.
template <int P>
struct KmSlot {
  int row[P], coff[P];
};
template <int P>
struct MnSlot {
  int krow[P], ncol[P];
};

template <int BK, int P>
__device__ __forceinline__ KmSlot<P> km_slots(int wave, int lane) {
  KmSlot<P> s;
#pragma unroll
  for (int jj = 0; jj < P; ++jj) {
    int row = (512 / BK) * (P * wave + jj) + lane / (BK / 8);
    int pc = lane % (BK / 8);
    s.row[jj] = row;
    s.coff[jj] = 8 * (pc ^ kmaj_swz<BK>(row));
  }
  return s;
}

template <int RB, int P, int MX = 1>
__device__ __forceinline__ MnSlot<P> mn_slots(int wave, int lane) {
  MnSlot<P> s;
#pragma unroll
  for (int jj = 0; jj < P; ++jj) {
    constexpr int CPM = RB / 16;  // 16-byte chunks per mn-major row
    int k = (1024 / RB) * (P * wave + jj) + lane / CPM;
    int p = lane % CPM;
    s.krow[jj] = k;
    s.ncol[jj] = ((16 * p) ^ mn_xor<RB, MX>(k)) / 2;
  }
  return s;
}

// LDS destination (bytes, wave-uniform) of wave instruction jj of a stage.
template <int P>
__device__ __forceinline__ int dma_dst(int wave, int jj) {
  return 1024 * (P * wave + jj);
}

__device__ __forceinline__ u32x2 to_h4(float a, float b, float c, float d) {
  u32x2 o;
  o[0] = (uint32_t)f32_to_h(a) | ((uint32_t)f32_to_h(b) << 16);
  o[1] = (uint32_t)f32_to_h(c) | ((uint32_t)f32_to_h(d) << 16);
  return o;
}

// Apply the epilogue to 4 consecutive channels; gate and out point at them
// (out is read for FG_EPI_ACC only).
__device__ __forceinline__ void epilogue4(float v[4], int epi, const uint16_t *gate,
                                          const uint16_t *out) {
  if (epi == FG_EPI_RELU) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
  } else if (epi == FG_EPI_GATE) {
    u32x2 gw = *reinterpret_cast<const u32x2 *>(gate);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint16_t gb = (uint16_t)(gw[e >> 1] >> (16 * (e & 1)));
      v[e] = h_to_f32(gb) > 0.f ? v[e] : 0.f;
    }
  } else if (epi == FG_EPI_ACC) {
    u32x2 ow = *reinterpret_cast<const u32x2 *>(out);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      v[e] += h_to_f32((uint16_t)(ow[e >> 1] >> (16 * (e & 1))));
  }
}

// fp16(a + b) for 8 packed pairs (fp32 sum of two fp16 values, one rounding
// to fp16; the sum of two fp16 values is exact in fp32 unless it is far
// below the larger's last bit, where the rounding is the same)
__device__ __forceinline__ u32x4 add_h8(const u32x4 &a, const u32x4 &b) {
  u32x4 o;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float lo = h_to_f32((uint16_t)(a[w] & 0xFFFFu)) + h_to_f32((uint16_t)(b[w] & 0xFFFFu));
    const float hi = h_to_f32((uint16_t)(a[w] >> 16)) + h_to_f32((uint16_t)(b[w] >> 16));
    o[w] = (uint32_t)f32_to_h(lo) | ((uint32_t)f32_to_h(hi) << 16);
  }
  return o;
}

// The ring: stage s of operand X lives in its own LDS array so that the
// compiler can tell the stages apart when it places waits. Unused slots of a
// ring shorter than five stages are token-sized.
struct Ring {
  uint8_t *a[5];
  uint8_t *b[5];
};
#define FG_DMA_RING(C, R)                                                     \
  constexpr int A_ = C::A_BYTES, B_ = C::B_BYTES, S2_ = C::NS > 2,            \
                S3_ = C::NS > 3, S4_ = C::NS > 4;                             \
  __shared__ __attribute__((aligned(1024))) uint8_t sA0[A_], sA1[A_],         \
      sA2[S2_ ? A_ : 16], sA3[S3_ ? A_ : 16], sA4[S4_ ? A_ : 16];             \
  __shared__ __attribute__((aligned(1024))) uint8_t sB0[B_], sB1[B_],         \
      sB2[S2_ ? B_ : 16], sB3[S3_ ? B_ : 16], sB4[S4_ ? B_ : 16];             \
  Ring R;                                                                     \
  R.a[0] = sA0, R.a[1] = sA1, R.a[2] = sA2, R.a[3] = sA3, R.a[4] = sA4;        \
  R.b[0] = sB0, R.b[1] = sB1, R.b[2] = sB2, R.b[3] = sB3, R.b[4] = sB4

// Wait until at most n stages of this wave's DMA loads remain outstanding
// (n <= 3; each stage is PA + PB load instructions).
template <class C>
__device__ __forceinline__ void wait_stages(int n) {
  constexpr int PS = C::PA + C::PB;
  static_assert(3 * PS < 64, "vmcnt range");
  if (n >= 3) wait_vm<3 * PS>();
  else if (n == 2) wait_vm<2 * PS>();
  else if (n == 1) wait_vm<PS>();
  else wait_vm<0>();
}

// Instruction-scheduling hints (LLVM AMDGPU IGroupLP): within the current
// scheduling region, place the MFMAs one by one and put `per` LDS reads
// after each of the first ones, so the reads of the next step issue among
// the MFMAs of this one instead of in a block.
template <int NMF, int NRD>
__device__ __forceinline__ void sched_mfma_reads() {
  constexpr int per = (NRD + NMF - 1) / NMF;
#pragma unroll
  for (int i = 0; i < NMF; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
    if (i * per < NRD) __builtin_amdgcn_sched_group_barrier(0x100, per, 0);  // DS read
  }
}
// After the barrier: reads first (they gate the next step), then the DMA
// loads of the refilled slot with their address arithmetic.
template <int NMF, int NRD, int NVM>
__device__ __forceinline__ void sched_mfma_reads_dma() {
  constexpr int per = (NRD + NMF / 2 - 1) / (NMF / 2);
#pragma unroll
  for (int i = 0; i < NMF / 2; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if (i * per < NRD) __builtin_amdgcn_sched_group_barrier(0x100, per, 0);
  }
  constexpr int pv = (NVM + NMF / 2 - 1) / (NMF / 2);
#pragma unroll
  for (int i = 0; i < NMF / 2; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if (i * pv < NVM) {
      __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);  // VALU
      __builtin_amdgcn_sched_group_barrier(0x020, pv, 0);  // VMEM read
    }
  }
}

// One stage (ring slot U) of the main loop. With `next`, the stage has a
// successor: the barrier that publishes it is crossed before the last step
// and the successor's first fragments are read into f[0]. `full` asserts
// that NS - 2 stages after the successor have been issued and that stage
// it + NS exists.
// `fold` is called after every 32 deep of the reduction (no-op by default).
struct NoFold {
  __device__ __forceinline__ void operator()() const {}
};
template <class C, bool AK, bool BKM, int U, class Issue, class Fold>
__device__ __forceinline__ void stage(f32x16 (&acc)[C::FM][C::FN],
                                      Frags<C> (&f)[2], const Ring &R, int it,
                                      int nst, bool next, bool full, int wm0,
                                      int wn0, int lane, Issue &issue, Fold &fold) {
  constexpr int NS = C::NS, KS = C::KS;
  constexpr int NMF = C::FM * C::FN;
  constexpr int NRD = C::FM * (AK ? 1 : 2) + C::FN * (BKM ? 1 : 2);
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    if (ks + 1 < KS)
      load_frags<C, AK, BKM>(f[(ks + 1) & 1], R.a[U], R.b[U], ks + 1, wm0, wn0,
                             lane);
    mma<C>(acc, f[ks & 1]);
    if (ks + 1 < KS) sched_mfma_reads<NMF, NRD>();
    __builtin_amdgcn_s_setprio(0);
    if (ks % 2 == 1 && ks + 1 < KS) fold();
    if (ks == KS - 2 && next) {
      // own DMA of stage it+1 done: later stages may remain in flight
      wait_stages<C>(full ? NS - 2 : min(NS - 2, nst - 2 - it));
      wait_lds();  // this wave's reads of slot U are complete
      barrier_nofence();
      // Past the barrier a wave has memory work to start (the refill DMA,
      // the next stage's first fragments) before its next MFMAs: raise its
      // issue priority over the other wave on its SIMD until those MFMAs
      // are issued, so the loads go out early. The priority drops back to 0
      // after every MFMA block. (Measured: 1-4% per layer.)
      __builtin_amdgcn_s_setprio(2);
      if (full || it + NS < nst) issue(it + NS, U);
      load_frags<C, AK, BKM>(f[0], R.a[(U + 1) % NS], R.b[(U + 1) % NS], 0, wm0,
                             wn0, lane);
    }
  }
  if constexpr (NMF > 1) {
    if (next) sched_mfma_reads_dma<NMF, NRD, C::PA + C::PB>();
  }
  fold();
}

template <class C, bool AK, bool BKM, int U, class Issue, class Fold>
__device__ __forceinline__ void group(f32x16 (&acc)[C::FM][C::FN],
                                      Frags<C> (&f)[2], const Ring &R, int it0,
                                      int nst, bool tail, int wm0, int wn0,
                                      int lane, Issue &issue, Fold &fold) {
  if constexpr (U < C::NS) {
    const int it = it0 + U;
    if (!tail) {
      stage<C, AK, BKM, U>(acc, f, R, it, nst, true, true, wm0, wn0, lane, issue,
                           fold);
    } else if (it < nst) {
      stage<C, AK, BKM, U>(acc, f, R, it, nst, it + 1 < nst, false, wm0, wn0,
                           lane, issue, fold);
    }
    group<C, AK, BKM, U + 1>(acc, f, R, it0, nst, tail, wm0, wn0, lane, issue, fold);
  }
}

// Runs the pipelined main loop over stages [0, nst): issue(st, slot) issues
// this wave's DMA loads of stage st into ring slot `slot`; stages are issued
// strictly in order. Full groups of NS stages run in a loop whose body has no
// data-dependent control flow around the MFMAs (so the compiler's own LDS
// waits stay exact and its scheduling regions span whole steps); the last
// groups run with per-stage checks.
template <class C, bool AK, bool BKM, class Issue, class Fold = NoFold>
__device__ __forceinline__ void pipeline(f32x16 (&acc)[C::FM][C::FN],
                                         const Ring &R, int nst, int wm0,
                                         int wn0, int lane, Issue &&issue,
                                         Fold &&fold = Fold{}) {
  constexpr int NS = C::NS, KS = C::KS;
  static_assert(NS >= 2 && NS <= 5 && KS >= 2 && KS % 2 == 0, "pipeline shape");
  if (nst <= 0) return;
#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < nst) issue(s, s);
  wait_stages<C>(min(NS - 2, nst - 1));  // publish stage 0
  barrier_nofence();
  if (NS - 1 < nst) issue(NS - 1, NS - 1);
  Frags<C> f[2];
  load_frags<C, AK, BKM>(f[0], R.a[0], R.b[0], 0, wm0, wn0, lane);
  // In a full group every stage has a successor, NS - 2 stages issued after
  // it, and a stage NS ahead to issue, so its waits and issues need no
  // checks: it0 + 2 NS - 1 < nst.
  int it0 = 0;
  for (; it0 + 2 * NS - 1 < nst; it0 += NS)
    group<C, AK, BKM, 0>(acc, f, R, it0, nst, false, wm0, wn0, lane, issue, fold);
  for (; it0 < nst; it0 += NS)
    group<C, AK, BKM, 0>(acc, f, R, it0, nst, true, wm0, wn0, lane, issue, fold);
}

template <class C>
__device__ __forceinline__ void zero(f32x16 (&acc)[C::FM][C::FN]) {
#pragma unroll
  for (int i = 0; i < C::FM; ++i)
#pragma unroll
    for (int j = 0; j < C::FN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
}

}  // namespace dma
}  // namespace fg
