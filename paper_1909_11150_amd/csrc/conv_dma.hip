// Implicit-GEMM convolutions fed by LDS DMA (gfx950 buffer_load ... lds): the
// data convolutions, then the kernel gradients.
//
// Same GEMM formulation as the register-staged kernels in conv_igemm.hip
// (rows = output channels, columns = output positions of one phase), on
// tiles from 64 x 64 to 256 x 256. Operands go from global memory straight
// into LDS: no register staging and no LDS store instructions. A ring of NS
// reduction stages, each BK deep, is kept in LDS, so a stage's loads are
// issued NS - 1 stages before they are consumed. Padding and ragged tails
// cost nothing: an out-of-range buffer offset returns zeros. The tile is
// split among WGM x WGN waves; stage depth, ring length and wave grid are
// template parameters (the configurations in use are named below).
//
// Two LDS tile layouts:
//   k-major  (row = GEMM row/column, BK reduction halves per row; 16-byte
//            chunk c stored at c ^ g(row)); MFMA operands are single 16-byte
//            reads of 32 consecutive rows.
//   mn-major (row = reduction index, 256 halves = 512 bytes per row; 64-byte
//            block b stored at b ^ (row & 3), or for the halo kernel's
//            weights 32-byte blocks as described at mn_xor); MFMA operands
//            are two transposing 8-byte reads (ds_read_b64_tr_b16).
// The permutations are chosen by measurement on gfx950, whose LDS has 64
// banks of 4 bytes: g(row) = (row >> 2) & 3 reads 32 consecutive 64-byte rows
// at full rate from any starting row (the previous ((row >> 1) ^ (row >> 3))
// & 3 ran at half rate), and the mn-major xor of (row & 3) * 64 bytes serves
// each half-wave of a transposing read without conflicts (xor of 32-byte
// blocks: two-way conflicts).
// The mn-major layout lets operands whose reduction index is strided in
// memory (input-gradient and transposed-conv weights, both kernel-gradient
// operands) be copied row by row as they lie in memory.
#include <algorithm>

#include "dma_pipe.h"

namespace fg {
namespace dma {

constexpr int TM = 256, TN = 256;       // output tile of the large kernels
// The configuration the library runs, chosen by timing the network's layers:
// 32-deep stages in a 5-stage ring (160 KiB) with 8 waves of 128 x 64.
#ifndef FG_DMA_DATA_CFG
#define FG_DMA_DATA_CFG 32, 5, 2, 4
#endif
using DataRun = K<FG_DMA_DATA_CFG>;
#ifndef FG_DMA_HALO_NS
#define FG_DMA_HALO_NS 3
#endif
using HaloRun = K<32, FG_DMA_HALO_NS, 2, 4>;  // weights ring; the rest is patches

// ---------------------------------------------------------------------------
// Output tile store of the data convolutions. The accumulator layout gives
// each lane 4 consecutive channels of one output position per register
// group, so storing it directly would scatter 8-byte pieces over 32
// positions per instruction. Instead each wave stages its 128-channel x
// 64-position block in LDS (the ring is free once the last stage is read),
// position-major with 16-byte chunks permuted by the position, and reads it
// back so that 16 lanes cover one position's 256 contiguous bytes: stores
// (and, for the gate epilogue, the gate loads) are whole 128-byte lines.
// fp32 partials (SPLIT) go in two passes of 64 channels.
// `buf` is this wave's 16 KiB of staging LDS and `pos` its 64-entry table;
// the caller guarantees that no wave still reads, and no DMA still writes,
// the LDS they alias (the store begins with a workgroup barrier).
template <class C, bool SPLIT>
__device__ __forceinline__ void store_tile(f32x16 (&acc)[C::FM][C::FN],
                                           uint8_t *buf, int32_t *pos,
                                           const DataConvArgs &a,
                                           const Phase &P, int npix, int n0,
                                           int m0, int wm0, int wn0, int lane,
                                           int split) {
  static_assert(C::WM == 128 && C::WN == 64, "store_tile expects 128 x 64 waves");
  __syncthreads();
  if (lane < 32) {
#pragma unroll
    for (int j = 0; j < C::FN; ++j) {
      const int col = n0 + wn0 + j * 32 + lane;
      int32_t ob = -1;
      if (col < npix) {
        const int b = col % P.mw, t = col / P.mw;
        const int aa = t % P.mh, nn = t / P.mh;
        // split partials are dense; the output has its own pixel stride
        ob = ((nn * a.ho + aa * a.ostr + P.ooh) * a.wo + b * a.ostr + P.oow) *
             (SPLIT ? a.co : a.ldo);
      }
      pos[j * 32 + lane] = ob;
    }
  }
  const size_t out_total = (size_t)a.n * a.ho * a.wo * a.co;
  const int cw = m0 + wm0;  // first channel of this wave's block
  constexpr int PASSES = SPLIT ? 2 : 1;
#pragma unroll
  for (int pass = 0; pass < PASSES; ++pass) {
    // acc -> LDS: position p = j*32 + lane%32, 4 channels per register group
#pragma unroll
    for (int j = 0; j < C::FN; ++j) {
      const int p = j * 32 + (lane & 31);
      uint8_t *row = buf + p * 256;
#pragma unroll
      for (int ii = 0; ii < C::FM / PASSES; ++ii) {
        const int i = pass * (C::FM / PASSES) + ii;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = acc[i][j][4 * g + e];
          if (SPLIT) {
            const int chunk = 8 * ii + 2 * g + (lane >> 5);
            *reinterpret_cast<f32x4 *>(row + ((chunk ^ (p & 15)) << 4)) =
                f32x4{v[0], v[1], v[2], v[3]};
          } else {
            if (a.epi == FG_EPI_RELU) {
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
            }
            const int chunk = 4 * i + g;
            *reinterpret_cast<u32x2 *>(row + ((chunk ^ (p & 15)) << 4) +
                                       8 * (lane >> 5)) =
                to_h4(v[0], v[1], v[2], v[3]);
          }
        }
      }
    }
    wait_lds();
    __builtin_amdgcn_wave_barrier();
    // LDS -> global: 16 lanes per position, 16-byte chunk q of its row.
    // All reads (and gate loads) are issued before any use, so their
    // latencies overlap; gate loads of absent positions read element 0.
    const int q = lane & 15;
    const int ch = SPLIT ? pass * 64 + 4 * q : 8 * q;  // channel within block
    const bool chok = cw + ch < a.co;
    u32x4 d[16];
    int32_t ob[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int p = 4 * k + (lane >> 4);
      d[k] = *reinterpret_cast<const u32x4 *>(buf + p * 256 + ((q ^ (p & 15)) << 4));
      ob[k] = chok ? pos[p] : -1;
    }
    if (!SPLIT && a.epi == FG_EPI_GATE) {
      u32x4 gw[16];
#pragma unroll
      for (int k = 0; k < 16; ++k)
        gw[k] = *reinterpret_cast<const u32x4 *>(a.gate + (ob[k] < 0 ? 0 : ob[k] + cw + ch));
#pragma unroll
      for (int k = 0; k < 16; ++k)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const uint32_t lo = h_to_f32((uint16_t)(gw[k][w] & 0xFFFFu)) > 0.f
                                  ? 0x0000FFFFu : 0u;
          const uint32_t hi = h_to_f32((uint16_t)(gw[k][w] >> 16)) > 0.f
                                  ? 0xFFFF0000u : 0u;
          d[k][w] &= lo | hi;
        }
    }
    if (!SPLIT && a.epi == FG_EPI_ACC) {  // add what the output holds
      u32x4 ow[16];
#pragma unroll
      for (int k = 0; k < 16; ++k)
        ow[k] = *reinterpret_cast<const u32x4 *>(a.out + (ob[k] < 0 ? 0 : ob[k] + cw + ch));
#pragma unroll
      for (int k = 0; k < 16; ++k) d[k] = add_h8(d[k], ow[k]);
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      if (ob[k] < 0) continue;
      if (SPLIT)
        *reinterpret_cast<u32x4 *>(a.part + (size_t)split * out_total + ob[k] + cw +
                                   ch) = d[k];
      else
        *reinterpret_cast<u32x4 *>(a.out + ob[k] + cw + ch) = d[k];
    }
    if (pass + 1 < PASSES) {
      wait_lds();
      __builtin_amdgcn_wave_barrier();
    }
  }
}

// ---------------------------------------------------------------------------
// Data convolution (forward / input gradient / transposed forward).
// Requires reduction channels cr % BK == 0 (a stage lies in one tap).
template <class C, bool WK, bool SPLIT>
__global__ __launch_bounds__(C::NT, C::WPE) void data_conv_dma_kernel(DataConvArgs a,
                                                              TileMap tm) {
  FG_DMA_RING(C, R);
  constexpr int PW = C::PW;

  int tz, ty, tx;  // phase x split, output-channel tile, position tile
  if (tm.order ? !tm.decode(blockIdx.x, tx, ty, tz)
                : !tm.decode(blockIdx.x, tz, ty, tx))
    return;
  const int phase = tz / a.nsplit, split = tz % a.nsplit;
  const Phase P = a.ph[phase];
  const int npix = a.n * P.mh * P.mw;
  const int n0 = tx * C::T;
  const int m0 = ty * C::T;
  if (n0 >= npix) return;
  const int ktot = P.nr * P.ns * a.cr;
  const int nk = ktot / C::BK;
  const int kchunk = (nk + a.nsplit - 1) / a.nsplit;
  const int kbeg = min(nk, split * kchunk), kend = min(nk, kbeg + kchunk);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave / C::WGN) * C::WM, wn0 = (wave % C::WGN) * C::WN;

  const __amdgpu_buffer_rsrc_t rs_act = __builtin_amdgcn_make_buffer_rsrc(
      (void *)a.act, 0, (int)act_span_bytes(a), kRsrcFlags);
  const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc(
      (void *)a.wgt, 0, a.wbytes, kRsrcFlags);

  // B: this lane's output positions (image row/column of tap (0, 0) of the
  // phase) and element offsets
  const KmSlot<PW> bs = km_slots<C::BK, PW>(wave, lane);
  int bh[PW], bw[PW], bbase[PW];
#pragma unroll
  for (int jj = 0; jj < PW; ++jj) {
    int col = n0 + bs.row[jj];
    if (col < npix) {
      int b = col % P.mw, t = col / P.mw;
      int aa = t % P.mh, nn = t / P.mh;
      bh[jj] = aa * a.istr;
      bw[jj] = b * a.istr;
      bbase[jj] = ((nn * a.hi + bh[jj]) * a.wi + bw[jj]) * a.ldi + bs.coff[jj];
    } else {
      bh[jj] = -(1 << 29);  // never inside the image
      bw[jj] = 0;
      bbase[jj] = 0;
    }
  }
  // A: this lane's weight offsets without the stage part, and whether its
  // output channel exists
  int wbase[PW];
  bool wok[PW];
#pragma unroll
  for (int jj = 0; jj < PW; ++jj) {
    if (WK) {
      const KmSlot<PW> as = km_slots<C::BK, PW>(wave, lane);
      const int co = m0 + as.row[jj];
      wok[jj] = co < a.co;
      wbase[jj] = co * a.ldw + as.coff[jj];
    } else {
      const MnSlot<PW> as = mn_slots<C::RB, PW>(wave, lane);
      const int co = m0 + as.ncol[jj];
      wok[jj] = co < a.co;
      wbase[jj] = as.krow[jj] * a.w_red + co;
    }
  }

  // Stage decode (uniform), advanced by one stage per issue() call: the
  // pipeline issues stages strictly in order. Stage st covers reduction
  // offsets [k0, k0 + BK) of tap t = k0 / cr, t = ti * ns + tj.
  int cr0, ti, tj;
  {
    const int k0 = kbeg * C::BK, t = k0 / a.cr;
    cr0 = k0 - t * a.cr;
    ti = t / P.ns;
    tj = t - ti * P.ns;
  }
  auto issue = [&](int, int slot) __attribute__((always_inline)) {
    const int dh = P.dh0 + P.dstep * ti, dw = P.dw0 + P.dstep * tj;
    const int woff = (P.r0 + P.rstep * ti) * a.s + (P.s0 + P.rstep * tj);
    const int delta = (dh * a.wi + dw) * a.ldi + cr0;
    const int wst = WK ? woff * a.cr + cr0 : cr0 * a.w_red + woff * a.w_tap;
    uint8_t *ta = R.a[slot], *tb = R.b[slot];
#pragma unroll
    for (int jj = 0; jj < PW; ++jj) {
      const bool v = (unsigned)(bh[jj] + dh) < (unsigned)a.hi &&
                     (unsigned)(bw[jj] + dw) < (unsigned)a.wi;
      const unsigned o = (unsigned)(bbase[jj] + delta) * 2u;
      dma16(rs_act, tb + dma_dst<PW>(wave, jj), v ? o : kOOB);
    }
#pragma unroll
    for (int jj = 0; jj < PW; ++jj) {
      const unsigned o = (unsigned)(wbase[jj] + wst) * 2u;
      dma16(rs_w, ta + dma_dst<PW>(wave, jj), wok[jj] ? o : kOOB);
    }
    // next stage, without branches (keeps the scheduling region whole)
    cr0 += C::BK;
    const bool wrap = cr0 == a.cr;
    cr0 = wrap ? 0 : cr0;
    tj += wrap;
    const bool wrap2 = tj == P.ns;
    tj = wrap2 ? 0 : tj;
    ti += wrap2;
  };

  f32x16 acc[C::FM][C::FN];
  zero<C>(acc);
  pipeline<C, WK, true>(acc, R, kend - kbeg, wm0, wn0, lane, issue);

  // staging: ring array `wave` (a-side arrays first, constant indices only) and
  // the position tables in the next one
  static_assert(2 * C::NS >= C::NW + 1 && C::TILE_BYTES >= 16384,
                "the store needs one 16 KiB ring array per wave plus one");
  uint8_t *sbuf = R.a[0];
#pragma unroll
  for (int k = 1; k < C::NW; ++k)
    if (wave == k) sbuf = k < C::NS ? R.a[k] : R.b[k - C::NS];
  int32_t *spos = reinterpret_cast<int32_t *>(R.b[C::NW - C::NS]) + 64 * wave;
  store_tile<C, SPLIT>(acc, sbuf, spos, a, P, npix, n0, m0, wm0, wn0, lane, split);
}

// ---------------------------------------------------------------------------
// Data convolution with input reuse ("halo" tiles): stride-1 3x3 convolutions
// (forward, and input gradient, which is one phase whose taps walk the input
// backward) whose 256-position
// tile is a block of whole output rows of one image. Instead of gathering the
// activation operand once per tap (9 times), the tile's input window, with a
// one-pixel halo, is loaded into LDS once per 32-channel chunk as a "patch"
// of (rows + 2) x (width + 2) positions; the 9 taps read shifted views of it.
// The reduction runs channel chunk by chunk, taps inside: stage s = 9 c + t.
// Weights take a 3-stage ring of 32-deep stages; the patch two slots, the
// next chunk's patch being loaded during the current chunk. Every stage
// issues the same number of loads (stages and patches past the end load
// nothing, through the out-of-range offset), so all waits are constants. The
// next chunk's patch is loaded a block per stage, spread over the chunk.
constexpr int kHaloTaps = 9;

// f(integral_constant<int, U>) for U = B .. E-1, unrolled at compile time.
template <int B, int E, class F>
__device__ __forceinline__ void unroll(F &f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    unroll<B + 1, E>(f);
  }
}
constexpr int kPatchRows = 768;                  // capacity, rows of 64 bytes
constexpr int kPatchBytes = kPatchRows * 64;

template <class C>
__device__ __forceinline__ u32x4 frag_row(const uint8_t *tile, int row, int ks,
                                          int lane) {
  return *reinterpret_cast<const u32x4 *>(
      tile + kmaj_off<32>(row, 2 * ks + (lane >> 5)));
}

// Loads in flight after stage s+1's loads, at the barrier inside stage s
// (position u of the unrolled group). The barrier of stage b issues weight
// stage b + NS and then, when its tap t(b) < NPW, this wave's patch block
// t(b) of the next chunk; stage s+1's weights were issued at the barrier of
// stage s+1-NS. (Stages before the first have taps 9-NS+1 .. 8 >= NPW, so
// the prologue needs no stand-ins.)
template <class C, int NPW>
__device__ __forceinline__ constexpr int halo_flight(int u) {
  int f = (C::NS - 2) * C::PW;
  for (int b = 1; b <= C::NS - 1; ++b)
    f += ((u - b) % kHaloTaps + kHaloTaps) % kHaloTaps < NPW ? 1 : 0;
  return f;
}

template <class C, bool WK, bool SPLIT>
__global__ __launch_bounds__(C::NT) void data_conv_halo_kernel(DataConvArgs a,
                                                               TileMap tm) {
  static_assert(C::BK == 32 && (C::NS == 3 || C::NS == 4) && C::KS == 2,
                "halo pipeline shape");
  static_assert(C::WM == 128 && C::WN == 64 && C::NW == 8, "halo wave layout");
  constexpr int NS = C::NS, PW = C::PW;
  constexpr int NPW = kPatchRows / 16 / C::NW;  // patch loads per wave
  // stages per unrolled group: whole pairs of chunks (both patch slots) and
  // whole turns of the weight ring
  constexpr int UNR = NS == 3 ? 2 * kHaloTaps : 4 * kHaloTaps;
  constexpr int TA3 = NS > 3 ? C::TILE_BYTES : 16;
  __shared__ __attribute__((aligned(1024))) uint8_t sA0[C::TILE_BYTES],
      sA1[C::TILE_BYTES], sA2[C::TILE_BYTES], sA3[TA3];
  __shared__ __attribute__((aligned(1024))) uint8_t sP0[kPatchBytes],
      sP1[kPatchBytes];
  uint8_t *ringA[4];
  ringA[0] = sA0, ringA[1] = sA1, ringA[2] = sA2, ringA[3] = sA3;
  uint8_t *patch[2];
  patch[0] = sP0, patch[1] = sP1;

  int split, ty, tx;  // reduction split, output-channel tile, position tile
  if (tm.order ? !tm.decode(blockIdx.x, tx, ty, split)
               : !tm.decode(blockIdx.x, split, ty, tx))
    return;
  const Phase P = a.ph[0];
  const int n0 = tx * TN, m0 = ty * TM;
  const int nchunk = a.cr / 32;
  const int cps = (nchunk + a.nsplit - 1) / a.nsplit;
  const int cbeg = min(nchunk, split * cps), cend = min(nchunk, cbeg + cps);
  const int nst = kHaloTaps * (cend - cbeg);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave / C::WGN) * C::WM, wn0 = (wave % C::WGN) * C::WN;

  const __amdgpu_buffer_rsrc_t rs_act = __builtin_amdgcn_make_buffer_rsrc(
      (void *)a.act, 0, (int)act_span_bytes(a), kRsrcFlags);
  const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc(
      (void *)a.wgt, 0, a.wbytes, kRsrcFlags);

  // tile geometry: rows [aa0, aa0 + 256 / mw) of image img
  const int mw = P.mw, pwid = mw + 2;
  const int img = n0 / (P.mh * mw), aa0 = (n0 / mw) % P.mh;
  const int prows = (TN / mw + 2) * pwid;
  // window origin: the taps walk the input forward (dstep 1, forward pass)
  // or backward (dstep -1, input gradient)
  const int dsg = P.dstep, back = dsg < 0 ? 2 : 0;
  const int h0 = aa0 + P.dh0 - back, w0 = P.dw0 - back;
  // patch loads of this lane: row r, 16-byte chunk (lane & 3) ^ g(r); byte
  // offset of channel 0 of its input position, or -1 outside the image
  int pbase[NPW];
#pragma unroll
  for (int jj = 0; jj < NPW; ++jj) {
    const int r = 16 * (NPW * wave + jj) + (lane >> 2);
    const int h = h0 + r / pwid, w = w0 + r % pwid;
    const bool v = r < prows && (unsigned)h < (unsigned)a.hi &&
                   (unsigned)w < (unsigned)a.wi;
    pbase[jj] = v ? (((img * a.hi + h) * a.wi + w) * a.ldi +
                     8 * ((lane & 3) ^ kmaj_swz<32>(r))) * 2
                  : -1;
  }
  // B fragment rows (patch row of tap (0, 0)) of this lane's positions
  int brow[C::FN];
#pragma unroll
  for (int j = 0; j < C::FN; ++j) {
    const int i = wn0 + 32 * j + (lane & 31);
    brow[j] = (i / mw) * pwid + i % mw;
  }
  // A: weight offsets without the stage part
  int wbase[PW];
  bool wok[PW];
#pragma unroll
  for (int jj = 0; jj < PW; ++jj) {
    if (WK) {
      const KmSlot<PW> as = km_slots<C::BK, PW>(wave, lane);
      const int co = m0 + as.row[jj];
      wok[jj] = co < a.co;
      wbase[jj] = co * a.ldw + as.coff[jj];
    } else {
      const MnSlot<PW> as = mn_slots<C::RB, PW, 0>(wave, lane);
      const int co = m0 + as.ncol[jj];
      wok[jj] = co < a.co;
      wbase[jj] = as.krow[jj] * a.w_red + co;
    }
  }
  // weight stage decode, advanced by one stage per issue (in order)
  int ic = cbeg, it_ = 0;
  auto issue_w = [&](int slot) __attribute__((always_inline)) {
    const int ti = it_ / 3, tj = it_ - 3 * ti;
    const int woff = (P.r0 + P.rstep * ti) * a.s + (P.s0 + P.rstep * tj);
    const int cr0 = 32 * ic;
    const int wst = WK ? woff * a.cr + cr0 : cr0 * a.w_red + woff * a.w_tap;
    const bool live = ic < cend;
#pragma unroll
    for (int jj = 0; jj < PW; ++jj) {
      const unsigned o = (unsigned)(wbase[jj] + wst) * 2u;
      dma16(rs_w, ringA[slot] + dma_dst<PW>(wave, jj), live && wok[jj] ? o : kOOB);
    }
    const bool wrap = ++it_ == kHaloTaps;
    it_ = wrap ? 0 : it_;
    ic += wrap;
  };
  // block jj of this wave's share of chunk c's patch
  auto issue_pb = [&](int pslot, int c, int jj) __attribute__((always_inline)) {
    const unsigned o = (unsigned)(pbase[jj] + 64 * c);
    dma16(rs_act, patch[pslot] + 1024 * (NPW * wave + jj),
          c < cend && pbase[jj] >= 0 ? o : kOOB);
  };

  f32x16 acc[C::FM][C::FN];
  zero<C>(acc);
  Frags<C> f[2];
  auto load = [&](Frags<C> &fr, int slot, int pslot, int t, int ks) __attribute__((always_inline)) {
    const int toff = back * (pwid + 1) + dsg * ((t / 3) * pwid + t % 3);
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
      fr.a[i] = frag<32, WK, 512, 0>(ringA[slot], wm0 + 32 * i, ks, lane);
#pragma unroll
    for (int j = 0; j < C::FN; ++j)
      fr.b[j] = frag_row<C>(patch[pslot], brow[j] + toff, ks, lane);
  };
  constexpr int NMF = C::FM * C::FN;
  constexpr int NRD = C::FM * (WK ? 1 : 2) + C::FN;

  // One stage at position U of the unrolled pair of chunks: A slot U % 3,
  // patch slot U / 9, tap U % 9.
  auto stage = [&](auto Uc, int it) __attribute__((always_inline)) {
    constexpr int U = decltype(Uc)::value;
    constexpr int T = U % kHaloTaps, SLOT = U % NS, PS = (U / kHaloTaps) & 1;
    constexpr int U1 = (U + 1) % UNR;
    // The patch row of a fragment depends on the tap; keep the compiler
    // from precomputing all taps' addresses across the unrolled stages.
#pragma unroll
    for (int j = 0; j < C::FN; ++j) asm volatile("" : "+v"(brow[j]));
    load(f[1], SLOT, PS, T, 1);
    mma<C>(acc, f[0]);
    sched_mfma_reads<NMF, NRD>();
    __builtin_amdgcn_s_setprio(0);
    wait_vm<halo_flight<C, NPW>(U)>();
    wait_lds();
    barrier_nofence();
    __builtin_amdgcn_s_setprio(2);  // as in stage(): loads first past the barrier
    issue_w(SLOT);  // stage it + NS
    // the next chunk's patch, one block per stage over its first NPW taps
    // (its slot's previous chunk is done: every wave is past this barrier)
    if (T < NPW) issue_pb(PS ^ 1, cbeg + it / kHaloTaps + 1, T);
    load(f[0], U1 % NS, (U1 / kHaloTaps) & 1, U1 % kHaloTaps, 0);
    mma<C>(acc, f[1]);
    sched_mfma_reads_dma<NMF, NRD, (T < NPW ? PW + 1 : PW)>();
    __builtin_amdgcn_s_setprio(0);
  };

  static_assert(NPW <= kHaloTaps - (NS - 1), "patch blocks fit the taps");
  // prologue: patch of the first chunk, weight stages 0 .. NS-2; publish
  // stage 0; weight stage NS-1
#pragma unroll
  for (int jj = 0; jj < NPW; ++jj) issue_pb(0, cbeg, jj);
#pragma unroll
  for (int st = 0; st < NS - 1; ++st) issue_w(st);
  wait_vm<(NS - 2) * PW>();
  barrier_nofence();
  issue_w(NS - 1);
  load(f[0], 0, 0, 0, 0);
  int it0 = 0;
  auto step = [&](auto Uc) __attribute__((always_inline)) { stage(Uc, it0 + decltype(Uc)::value); };
  for (; it0 + UNR <= nst; it0 += UNR) unroll<0, UNR>(step);
  // the rest, a whole number of chunks, as a prefix of a group
  constexpr int G9 = kHaloTaps;
  if (it0 + G9 <= nst) unroll<0, G9>(step);
  if constexpr (UNR > 2 * G9) {
    if (it0 + 2 * G9 <= nst) unroll<G9, 2 * G9>(step);
    if (it0 + 3 * G9 <= nst) unroll<2 * G9, 3 * G9>(step);
  }
  wait_vm<0>();  // loads issued past the end have landed

  // staging for the store: A slots, then 16 KiB pieces of the patch slots;
  // position tables after them
  uint8_t *sbuf = sA0;
  if (wave == 1) sbuf = sA1;
  if (wave == 2) sbuf = sA2;
  if (wave >= 3 && wave < 6) sbuf = sP0 + 16384 * (wave - 3);  // (sA3 unused)
  if (wave >= 6) sbuf = sP1 + 16384 * (wave - 6);
  int32_t *spos = reinterpret_cast<int32_t *>(sP1 + 32768) + 64 * wave;
  const int npix = a.n * P.mh * P.mw;
  store_tile<C, SPLIT>(acc, sbuf, spos, a, P, npix, n0, m0, wm0, wn0, lane, split);
}

// Where the weights are large and much larger than the input, an XCD should
// fetch its share of the weights and all of the input, not the reverse: 1024 x
// 9216 weights over 1024 positions 37.3 -> 33.6 us (128 x 128 tiles), 1024 x
// 16384 over 1024 52.0 -> 46.1. Below 8 MiB or at 3 times the input the other
// order is the faster one (768 x 3456 over 1152 20.4 -> 21.7 us this way, 1024 x
// 9216 over 4096 95 -> 125 on small tiles).
static bool weight_major(const DataConvArgs &a) {
  return a.wbytes >= (8 << 20) && (size_t)a.wbytes >= 3 * act_span_bytes(a);
}

// Tile order of a launch over the phases of a (reordered here where they differ
// in cost).
static TileMap data_tile_map(DataConvArgs &a, int tm_, int tn_) {
  int maxpix = 0;
  bool uneven = false;
  for (int i = 0; i < a.nphase; ++i) {
    maxpix = std::max(maxpix, a.n * a.ph[i].mh * a.ph[i].mw);
    uneven |= a.ph[i].nr * a.ph[i].ns != a.ph[0].nr * a.ph[0].ns;
  }
  const int tco = (a.co + tm_ - 1) / tm_, tpix = (maxpix + tn_ - 1) / tn_;
  TileMap tm;
  if (uneven) {
    // phases with different tap counts (strided input gradients): costliest
    // phase first, in launch order, so the cheap tiles fill the tail
    std::stable_sort(a.ph, a.ph + a.nphase, [](const Phase &x, const Phase &y) {
      return x.nr * x.ns > y.nr * y.ns;
    });
    tm = TileMap{tpix, tco, a.nphase * a.nsplit, 0, kCostly};
  } else if (weight_major(a)) {
    tm = TileMap{tpix, tco, a.nphase * a.nsplit, 0, kWeightMajor};
  } else {
    // phases and splits fastest, so every XCD gets an even share of each
    // and the phases of one position tile share input
    tm = TileMap{a.nphase * a.nsplit, tco, tpix, 0, kOutputMajor};
  }
  tm.per = (tm.n0 * tm.n1 * tm.n2 + 7) / 8;
  return tm;
}

// ---------------------------------------------------------------------------
// Data convolutions on small tiles, and of any channel count (multiples of 8).
//
// The 256 x 256 kernels above leave most CUs idle where the output is small, and
// waste the tile where it has fewer channels: there the time is the chain of one
// workgroup's stages and what two launches of a split cost. These tiles (64 x
// 64, 64 channels x 128 positions, 128 x 128) have 64-deep stages (whole
// 128-byte lines, half the barriers), two waves per SIMD and workgroup for the
// two larger ones, and a store through LDS in whole rows. Where 64-deep stages
// would straddle taps, 128 x 128 tiles have 4 waves and 32-deep stages (deep32 in
// conv_igemm.hip). Against such tiles on all of these shapes: 128 channels, K 1152
// over 32768 positions 19.9 -> 15.5 us; the strided input gradient of 64
// channels, K 128 to 512 over 131072 28.4 -> 16.5; 64 channels, K 576 over 6240
// 11.7 -> 6.6; the register-staged kernel on 512 channels, K 2376 over 65536
// 330 -> 182 (256 x 256).
//   GEN: reduction channels that are not a multiple of the stage depth. A
//   stage then straddles taps: every lane copies 8 reduction channels, which
//   lie in one tap, and advances its own (tap, channel) by BK per stage.
template <int P, bool GEN>
struct RedPos;  // reduction position of each of P DMA slots
template <int P>
struct RedPos<P, true> {
  int c[P], t[P];  // channel, tap
  __device__ __forceinline__ void init(int jj, int kk, int cr) {
    t[jj] = kk / cr;
    c[jj] = kk - t[jj] * cr;
  }
  __device__ __forceinline__ void advance(int jj, int dt, int dc, int cr) {
    c[jj] += dc;
    const bool w = c[jj] >= cr;
    c[jj] -= w ? cr : 0;
    t[jj] += dt + w;
  }
};
template <int P>
struct RedPos<P, false> {};

// Store of a wave's WM-channel x WN-position block through LDS, position-major
// rows of WM fp16 values in 16-byte chunks, so that whole 64- or 128-byte rows
// are written (and read, for the gate). `buf`: WM * WN * 2 bytes of this wave's
// own, `pos`: WN entries.
template <class P>
__device__ __forceinline__ void store_rows(f32x16 (&acc)[P::FM][P::FN], uint8_t *buf,
                                           const int32_t *pos, const DataConvArgs &a,
                                           int c0, int lane) {
  constexpr int CPW = P::WM / 8, RB = P::WM * 2;  // chunks, bytes per row
  constexpr int SH = CPW == 16 ? 0 : CPW == 8 ? 1 : 2;  // rows per bank turn, log2
#pragma unroll
  for (int j = 0; j < P::FN; ++j) {
    const int p = j * 32 + (lane & 31);
#pragma unroll
    for (int i = 0; i < P::FM; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] = acc[i][j][4 * g + e];
          if (a.epi == FG_EPI_RELU) v[e] = v[e] > 0.f ? v[e] : 0.f;
        }
        *reinterpret_cast<u32x2 *>(buf + p * RB +
                                   (((4 * i + g) ^ ((p >> SH) & (CPW - 1))) << 4) +
                                   8 * (lane >> 5)) = to_h4(v[0], v[1], v[2], v[3]);
      }
  }
  wait_lds();
  __builtin_amdgcn_wave_barrier();
  constexpr int PPI = 64 / CPW, N = P::WN / PPI;  // positions per instruction
  const int q = lane % CPW, ch = c0 + 8 * q;
  u32x4 d[N];
  int32_t ob[N];
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const int p = k * PPI + lane / CPW;
    d[k] = *reinterpret_cast<const u32x4 *>(buf + p * RB +
                                            ((q ^ ((p >> SH) & (CPW - 1))) << 4));
    ob[k] = ch < a.co ? pos[p] : -1;
  }
  if (a.epi == FG_EPI_GATE) {
    u32x4 gw[N];
#pragma unroll
    for (int k = 0; k < N; ++k)  // absent positions read element 0
      gw[k] = *reinterpret_cast<const u32x4 *>(a.gate + (ob[k] < 0 ? 0 : ob[k] + ch));
#pragma unroll
    for (int k = 0; k < N; ++k)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t lo =
            h_to_f32((uint16_t)(gw[k][w] & 0xFFFFu)) > 0.f ? 0x0000FFFFu : 0u;
        const uint32_t hi = h_to_f32((uint16_t)(gw[k][w] >> 16)) > 0.f ? 0xFFFF0000u : 0u;
        d[k][w] &= lo | hi;
      }
  }
#pragma unroll
  for (int k = 0; k < N; ++k)
    if (ob[k] >= 0) *reinterpret_cast<u32x4 *>(a.out + ob[k] + ch) = d[k];
}

// What becomes of a workgroup's sum: stored whole; one part of a split, stored
// as fp32 partials; or whole, but summed in a.nchunk parts from zero, each added
// to the ones before (the order of a split without its second launch and its
// partials: 256 x 2048 over 8192 positions in 2 parts 26.6 -> 17.7 us).
enum class Sum { kWhole, kPart, kFold };

// Division by the width and height of each phase's output grid.
struct PosDiv {
  FastDiv mw[4], mh[4];
};

template <class P, bool WK, Sum SUM, bool GEN>
__device__ __forceinline__ void data_tile(const DataConvArgs &a, const TileMap &tm,
                                          const PosDiv &pd) {
  FG_DMA_RING(P, R);
  constexpr int PA = P::PA, PB = P::PB, BK = P::BK;

  int tz, ty, tx;  // phase x split, output-channel tile, position tile
  if (tm.order ? !tm.decode(blockIdx.x, tx, ty, tz)
                : !tm.decode(blockIdx.x, tz, ty, tx))
    return;
  const int phase = tz / a.nsplit, split = tz % a.nsplit;
  const Phase F = a.ph[phase];
  const FastDiv dmw = pd.mw[phase], dmh = pd.mh[phase];
  const int npix = a.n * F.mh * F.mw;
  const int n0 = tx * P::TN, m0 = ty * P::TM;
  if (n0 >= npix) return;
  constexpr bool SPLIT = SUM == Sum::kPart;
  const int ktot = F.nr * F.ns * a.cr;
  const int plen = part_len(ktot, a.unit, a.nchunk);
  const int kbeg = SPLIT ? min(ktot, split * plen) : 0;
  const int kend = SPLIT ? min(ktot, kbeg + plen) : ktot;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave / P::WGN) * P::WM, wn0 = (wave % P::WGN) * P::WN;

  const __amdgpu_buffer_rsrc_t rs_act = __builtin_amdgcn_make_buffer_rsrc(
      (void *)a.act, 0, (int)act_span_bytes(a), kRsrcFlags);
  const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc(
      (void *)a.wgt, 0, a.wbytes, kRsrcFlags);

  // position col of the phase: image n, row and column of the grid
  auto decode = [&](int col, int &nn, int &aa, int &b) __attribute__((always_inline)) {
    const unsigned t = dmw.div((unsigned)col);
    b = col - (int)t * F.mw;
    nn = (int)dmh.div(t);
    aa = (int)t - nn * F.mh;
  };

  // B: this lane's positions (image row and column of tap (0, 0)) and offsets
  const KmSlot<PB> bs = km_slots<BK, PB>(wave, lane);
  int bh[PB], bw[PB], bbase[PB];
  RedPos<PB, GEN> rb;
#pragma unroll
  for (int jj = 0; jj < PB; ++jj) {
    const int col = n0 + bs.row[jj];
    int nn, aa, b;
    decode(col, nn, aa, b);
    bh[jj] = col < npix ? aa * a.istr + F.dh0 : -(1 << 29);  // or never inside
    bw[jj] = b * a.istr + F.dw0;
    bbase[jj] = ((nn * a.hi + aa * a.istr + F.dh0) * a.wi + bw[jj]) * a.ldi +
                (GEN ? 0 : bs.coff[jj]);
    if constexpr (GEN) rb.init(jj, kbeg + bs.coff[jj], a.cr);
  }
  // A: this lane's weight offsets without the stage part (k-major: forward
  // weights, whose reduction index is linear in memory)
  int wbase[PA], wkk[PA];
  bool wok[PA];
  RedPos<PA, GEN && !WK> ra;
#pragma unroll
  for (int jj = 0; jj < PA; ++jj) {
    if (WK) {
      const KmSlot<PA> as = km_slots<BK, PA>(wave, lane);
      const int co = m0 + as.row[jj];
      wok[jj] = co < a.co;
      wbase[jj] = co * a.ldw + as.coff[jj];
      wkk[jj] = as.coff[jj];
    } else {
      const MnSlot<PA> as = mn_slots<P::RBA, PA>(wave, lane);
      const int co = m0 + as.ncol[jj];
      wok[jj] = co < a.co;
      wbase[jj] = (GEN ? 0 : as.krow[jj] * a.w_red) + co;
      wkk[jj] = as.krow[jj];
      if constexpr (GEN && !WK) ra.init(jj, kbeg + as.krow[jj], a.cr);
    }
  }
  const int dt = BK / a.cr, dc = BK - dt * a.cr;  // GEN: a stage's advance
  // t / ns = t * nsm >> 8 for the taps there are, t < nr * ns <= 16 (not for every
  // t < 64); later ones, past the end of the sum, are masked off by kend
  const int nsm = (255 + F.ns) / max(F.ns, 1);

  // uniform stage decode (whole stages of one tap), as in the kernels above
  int cr0 = 0, ti = 0, tj = 0, kk0 = kbeg;
  if constexpr (!GEN) {
    const int t = kk0 / a.cr;
    cr0 = kk0 - t * a.cr;
    ti = t / F.ns;
    tj = t - ti * F.ns;
  }
  auto issue = [&](int, int slot) __attribute__((always_inline)) {
    uint8_t *ta = R.a[slot], *tb = R.b[slot];
    if constexpr (GEN) {
#pragma unroll
      for (int jj = 0; jj < PB; ++jj) {
        const int i = (rb.t[jj] * nsm) >> 8, j = rb.t[jj] - i * F.ns;
        const int dh = F.dstep * i, dw = F.dstep * j;
        const bool v = bs.coff[jj] < kend - kk0 && (unsigned)(bh[jj] + dh) < (unsigned)a.hi &&
                       (unsigned)(bw[jj] + dw) < (unsigned)a.wi;
        const unsigned o =
            (unsigned)(bbase[jj] + (dh * a.wi + dw) * a.ldi + rb.c[jj]) * 2u;
        dma16(rs_act, tb + dma_dst<PB>(wave, jj), v ? o : kOOB);
        rb.advance(jj, dt, dc, a.cr);
      }
#pragma unroll
      for (int jj = 0; jj < PA; ++jj) {
        unsigned o;
        bool v;
        if constexpr (WK) {
          o = (unsigned)(wbase[jj] + kk0) * 2u;
          v = wok[jj] && wkk[jj] < kend - kk0;
        } else {
          const int i = (ra.t[jj] * nsm) >> 8, j = ra.t[jj] - i * F.ns;
          const int woff = (F.r0 + F.rstep * i) * a.s + F.s0 + F.rstep * j;
          o = (unsigned)(wbase[jj] + ra.c[jj] * a.w_red + woff * a.w_tap) * 2u;
          v = wok[jj] && wkk[jj] < kend - kk0;
          ra.advance(jj, dt, dc, a.cr);
        }
        dma16(rs_w, ta + dma_dst<PA>(wave, jj), v ? o : kOOB);
      }
      kk0 += BK;
    } else {
      const int dh = F.dstep * ti, dw = F.dstep * tj;
      const int woff = (F.r0 + F.rstep * ti) * a.s + (F.s0 + F.rstep * tj);
      const int delta = (dh * a.wi + dw) * a.ldi + cr0;
      const int wst = WK ? woff * a.cr + cr0 : cr0 * a.w_red + woff * a.w_tap;
#pragma unroll
      for (int jj = 0; jj < PB; ++jj) {
        const bool v = (unsigned)(bh[jj] + dh) < (unsigned)a.hi &&
                       (unsigned)(bw[jj] + dw) < (unsigned)a.wi;
        const unsigned o = (unsigned)(bbase[jj] + delta) * 2u;
        dma16(rs_act, tb + dma_dst<PB>(wave, jj), v ? o : kOOB);
      }
#pragma unroll
      for (int jj = 0; jj < PA; ++jj) {
        const unsigned o = (unsigned)(wbase[jj] + wst) * 2u;
        dma16(rs_w, ta + dma_dst<PA>(wave, jj), wok[jj] ? o : kOOB);
      }
      cr0 += BK;
      const bool wrap = cr0 == a.cr;
      cr0 = wrap ? 0 : cr0;
      tj += wrap;
      const bool wrap2 = tj == F.ns;
      tj = wrap2 ? 0 : tj;
      ti += wrap2;
    }
  };

  f32x16 acc[P::FM][P::FN];
  zero<P>(acc);
  const int nst = (kend - kbeg + BK - 1) / BK;
  if constexpr (SUM == Sum::kFold) {
    f32x16 tot[P::FM][P::FN];
    zero<P>(tot);
    int done = 0, next = plen;  // reduction summed so far, end of the part
    bool first = true;
    auto fold = [&]() __attribute__((always_inline)) {
      done += 32;
      if (done == next && done < ktot) {
#pragma unroll
        for (int i = 0; i < P::FM; ++i)
#pragma unroll
          for (int j = 0; j < P::FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
              tot[i][j][v] = first ? acc[i][j][v] : tot[i][j][v] + acc[i][j][v];
              acc[i][j][v] = 0.f;
            }
        next += plen;
        first = false;
      }
    };
    pipeline<P, WK, true>(acc, R, nst, wm0, wn0, lane, issue, fold);
    if (!first) {
#pragma unroll
      for (int i = 0; i < P::FM; ++i)
#pragma unroll
        for (int j = 0; j < P::FN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[i][j][v] = tot[i][j][v] + acc[i][j][v];
    }
  } else {
    pipeline<P, WK, true>(acc, R, nst, wm0, wn0, lane, issue);
  }

  // element offset of a position (-1: absent); split partials are dense
  const int ldo = SPLIT ? a.co : a.ldo;
  auto opos = [&](int col) __attribute__((always_inline)) {
    int nn, aa, b;
    decode(col, nn, aa, b);
    const int o = ((nn * a.ho + aa * a.ostr + F.ooh) * a.wo + b * a.ostr + F.oow) * ldo;
    return col < npix ? o : -1;
  };
  // Staged rows, except where the output is added to: there the sum is rounded
  // once (the staged rows are fp16 already).
  constexpr int WB = P::WM * P::WN * 2, WP = WB + 4 * P::WN;  // rows, and positions
  constexpr bool ONE = P::NW * WB <= P::B_BYTES && P::NW * 4 * P::WN <= P::B_BYTES;
  constexpr int PER = P::B_BYTES / WP;  // waves per array, else
  static_assert(ONE || (P::A_BYTES == P::B_BYTES && PER > 0 && P::NW <= 2 * P::NS * PER) ||
                    (P::A_BYTES == WB && P::B_BYTES == WB && P::NW < 2 * P::NS),
                "the ring has room to stage the tile");
  if (!SPLIT && a.epi != FG_EPI_ACC) {
    __syncthreads();  // every wave is done reading the ring
    uint8_t *buf;
    int32_t *pos;
    if constexpr (ONE) {  // all rows in one array, the positions in the next
      buf = R.b[0] + wave * WB;
      pos = reinterpret_cast<int32_t *>(R.b[1]) + wave * P::WN;
    } else {              // constant array indices only
      constexpr int W = PER > 0 ? PER : 1;
      buf = R.a[0];
#pragma unroll
      for (int k = 1; k < (P::NW + W - 1) / W; ++k)
        if (wave / W == k) buf = k < P::NS ? R.a[k] : R.b[k - P::NS];
      buf += wave % W * WP;
      pos = PER > 0 ? reinterpret_cast<int32_t *>(buf + WB)
                    : reinterpret_cast<int32_t *>(R.b[P::NS - 1]) + wave * P::WN;
    }
    if (lane < P::WN) pos[lane] = opos(n0 + wn0 + lane);
    store_rows<P>(acc, buf, pos, a, m0 + wm0, lane);
    return;
  }
  const size_t out_total = (size_t)a.n * a.ho * a.wo * a.co;
#pragma unroll
  for (int j = 0; j < P::FN; ++j) {
    const int ob = opos(n0 + wn0 + j * 32 + (lane & 31));
    if (ob < 0) continue;
#pragma unroll
    for (int i = 0; i < P::FM; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int co = m0 + wm0 + i * 32 + 8 * g + 4 * (lane >> 5);
        if (co >= a.co) continue;
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[i][j][4 * g + e];
        if (SPLIT) {
          *reinterpret_cast<f32x4 *>(a.part + split * out_total + ob + co) =
              f32x4{v[0], v[1], v[2], v[3]};
        } else {
          epilogue4(v, a.epi, a.gate + ob + co, a.out + ob + co);
          *reinterpret_cast<u32x2 *>(a.out + ob + co) = to_h4(v[0], v[1], v[2], v[3]);
        }
      }
  }
}

using Data64 = Pipe<64, 3, 2, 2, 64, 64>;       // 4 waves of 32 x 32
using Data64x128 = Pipe<64, 3, 2, 4, 64, 128>;  // 8 waves of 32 x 32
using Data128 = Pipe<64, 2, 4, 2, 128, 128>;    // 8 waves of 32 x 64
using Data128d32 = Pipe<32, 5, 2, 2, 128, 128>;  // 4 waves of 64 x 64
using Data256 = Pipe<32, 5, 2, 4, 256, 256>;    // 8 waves of 128 x 64

// The kernels by what a stage and a sum are: whole taps per stage (overloading the
// 256 x 256 tiles' kernel above), stages that straddle taps, and sums folded in
// parts (either kind of stage).
template <class P, bool WK, bool SPLIT>
__global__ __launch_bounds__(P::NT, P::WPE) void data_conv_dma_kernel(DataConvArgs a, TileMap tm,
                                                                      PosDiv pd) {
  data_tile<P, WK, SPLIT ? Sum::kPart : Sum::kWhole, false>(a, tm, pd);
}
template <class P, bool WK, bool SPLIT>
__global__ __launch_bounds__(P::NT, P::WPE) void data_conv_gen_kernel(DataConvArgs a, TileMap tm,
                                                                      PosDiv pd) {
  data_tile<P, WK, SPLIT ? Sum::kPart : Sum::kWhole, true>(a, tm, pd);
}
template <class P, bool WK, bool GEN>
__global__ __launch_bounds__(P::NT, P::WPE) void data_conv_fold_kernel(DataConvArgs a, TileMap tm,
                                                                       PosDiv pd) {
  data_tile<P, WK, Sum::kFold, GEN>(a, tm, pd);
}
using DataTileKernel = void (*)(DataConvArgs, TileMap, PosDiv);

template <class P, bool WK>
static DataTileKernel data_tile_kernel(bool split, bool gen, bool fold) {
  if constexpr (P::TM == 256) {  // whole taps: the kernel above; it cannot fold
    return split ? data_conv_gen_kernel<P, WK, true> : data_conv_gen_kernel<P, WK, false>;
  } else if constexpr (P::BK == 32) {  // whole taps and parts
    if constexpr (!WK) {  // weights read as they lie: only split sums
      if (fold) return data_conv_fold_kernel<P, WK, false>;
      if (!split) return data_conv_dma_kernel<P, WK, false>;
    }
    return data_conv_dma_kernel<P, WK, true>;
  } else {
    if (fold)
      return gen ? data_conv_fold_kernel<P, WK, true> : data_conv_fold_kernel<P, WK, false>;
    if (gen)
      return split ? data_conv_gen_kernel<P, WK, true> : data_conv_gen_kernel<P, WK, false>;
    return split ? static_cast<DataTileKernel>(data_conv_dma_kernel<P, WK, true>)
                 : static_cast<DataTileKernel>(data_conv_dma_kernel<P, WK, false>);
  }
}

template <class P>
static hipError_t launch_data_tile(const DataConvArgs &a0, bool w_kmajor, bool gen, bool fold,
                                   hipStream_t st) {
  DataConvArgs a = a0;
  const bool split = a.nsplit > 1;
  const DataTileKernel k = w_kmajor ? data_tile_kernel<P, true>(split, gen, fold)
                                    : data_tile_kernel<P, false>(split, gen, fold);
  const TileMap tm = data_tile_map(a, P::TM, P::TN);
  PosDiv pd;
  for (int i = 0; i < 4; ++i) {
    pd.mw[i] = make_fastdiv((uint32_t)std::max(a.ph[i].mw, 1));
    pd.mh[i] = make_fastdiv((uint32_t)std::max(a.ph[i].mh, 1));
  }
  hipLaunchKernelGGL(k, dim3(8 * tm.per), dim3(P::NT), 0, st, a, tm, pd);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Kernel gradients fed by LDS DMA, for any channel counts (multiples of 8).
//
// Rows rho = (tap, input channel), columns = output channels, reduction over
// output positions; both operands are copied row by row from memory into
// mn-major LDS tiles and read with transposing LDS reads. A tile may straddle
// taps and run past the last row or column: each lane copies 8 channels, which
// lie in one tap, so the tap is a property of the lane, decoded once; chunks
// past the end get an out-of-range offset and read zeros.
//
// Three square tiles. 256 has the fewest LDS and L2 bytes per multiply and runs
// the layers with enough tiles and positions to fill the CUs; the others are
// bound by the chain of one workgroup's stages (about 0.3 us per 64 rows) and
// by how few workgroups there are, so they take smaller tiles: 256 x 9 x 256
// over 1800 positions 41 us on one 256 tile row of workgroups, 27.9 at its best
// split, 13.4 unsplit on 64 tiles. Against the register-staged kernels that
// these shapes ran before: 128 x 1152 x 32768 39 -> 27 us with its reduction,
// 160 x 864 x 20925 33 -> 24, 320 x 320 x 21756 65 -> 21.

// Tiles. 64-deep stages (whole 128-byte lines of both operands per barrier) for
// the small ones, whose time is the chain of stages.
using Tile256 = Pipe<32, 4, 2, 4, 256, 256>;  // 8 waves of 128 x 64
using Tile128 = Pipe<64, 2, 2, 2, 128, 128>;  // 4 waves of 64 x 64
using Tile64 = Pipe<64, 3, 2, 2, 64, 64>;     // 4 waves of 32 x 32

// Store of a wave's WM x WN block: rows rho (contiguous in memory for a fixed
// output channel k) within rsc, columns k within a.k. Staged in this wave's
// part of the ring k-major, 64 rows of rho at a time (128-byte rows: 64 fp16
// or, per pass, 32 fp32 values; 16-byte chunks permuted by the row), and read
// back so that 8 lanes write one row's contiguous 128 bytes.
template <class P, bool SPLIT>
__device__ __forceinline__ void store_rho(f32x16 (&acc)[P::FM][P::FN], uint8_t *buf,
                                          const WgradArgs &a, int rsc, int rho0, int k0,
                                          int lane, int split) {
  static_assert(P::WM % 64 == 0 && P::WN == 64, "staged blocks are 64 wide");
  constexpr int HM = P::WM / 64, PASSES = SPLIT ? 2 : 1;
  bool bad = false;
#pragma unroll
  for (int h = 0; h < HM; ++h)
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
#pragma unroll
      for (int j = 0; j < P::FN; ++j) {
        const int kr = j * 32 + (lane & 31);
        uint8_t *row = buf + kr * 128;
        const int sw = (kr >> 1) & 7;
#pragma unroll
        for (int ii = 0; ii < 2 / PASSES; ++ii) {
          const int il = pass * (2 / PASSES) + ii;
          const f32x16 &c = acc[2 * h + il][j];
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            if (SPLIT)
              *reinterpret_cast<f32x4 *>(row + (((2 * g + (lane >> 5)) ^ sw) << 4)) =
                  f32x4{c[4 * g], c[4 * g + 1], c[4 * g + 2], c[4 * g + 3]};
            else
              *reinterpret_cast<u32x2 *>(row + (((4 * il + g) ^ sw) << 4) +
                                         8 * (lane >> 5)) =
                  to_h4(c[4 * g], c[4 * g + 1], c[4 * g + 2], c[4 * g + 3]);
          }
        }
      }
      wait_lds();
      __builtin_amdgcn_wave_barrier();
      const int q = lane & 7;  // 16-byte chunk of the row
      const int rho = rho0 + 64 * h + (SPLIT ? pass * 32 + 4 * q : 8 * q);
#pragma unroll
      for (int t = 0; t < P::WN / 8; ++t) {
        const int kr = 8 * t + (lane >> 3), k = k0 + kr;
        const u32x4 d =
            *reinterpret_cast<const u32x4 *>(buf + kr * 128 + ((q ^ ((kr >> 1) & 7)) << 4));
        if (k >= a.k || rho >= rsc) continue;
        if (SPLIT) {
          *reinterpret_cast<u32x4 *>(a.part + ((size_t)split * a.k + k) * rsc + rho) = d;
        } else {
#pragma unroll
          for (int w = 0; w < 4; ++w) bad |= nonfinite_h2(d[w]);
          *reinterpret_cast<u32x4 *>(a.dw + (size_t)k * rsc + rho) = d;
        }
      }
      wait_lds();
      __builtin_amdgcn_wave_barrier();
    }
  if (!SPLIT && a.flag) flag_nonfinite(a.flag, bad);
}

// The same without staging (blocks less than 64 wide): each lane writes 4
// consecutive rho of one output channel.
template <class P, bool SPLIT>
__device__ __forceinline__ void store_rho_direct(f32x16 (&acc)[P::FM][P::FN],
                                                 const WgradArgs &a, int rsc, int rho0,
                                                 int k0, int lane, int split) {
  bool bad = false;
#pragma unroll
  for (int j = 0; j < P::FN; ++j) {
    const int k = k0 + j * 32 + (lane & 31);
    if (k >= a.k) continue;
#pragma unroll
    for (int i = 0; i < P::FM; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int rho = rho0 + i * 32 + 8 * g + 4 * (lane >> 5);
        if (rho >= rsc) continue;
        const f32x16 &c = acc[i][j];
        if (SPLIT) {
          *reinterpret_cast<f32x4 *>(a.part + ((size_t)split * a.k + k) * rsc + rho) =
              f32x4{c[4 * g], c[4 * g + 1], c[4 * g + 2], c[4 * g + 3]};
        } else {
          const u32x2 hv = to_h4(c[4 * g], c[4 * g + 1], c[4 * g + 2], c[4 * g + 3]);
          bad |= nonfinite_h2(hv[0]) || nonfinite_h2(hv[1]);
          *reinterpret_cast<u32x2 *>(a.dw + (size_t)k * rsc + rho) = hv;
        }
      }
  }
  if (!SPLIT && a.flag) flag_nonfinite(a.flag, bad);
}

// Arguments by value: by reference the 256 tile's register allocation loses
// its unrolled addresses (236 registers instead of 251, 3-6% slower).
template <class P, bool SPLIT>
__device__ __forceinline__ void wgrad_tile(const WgradArgs a, const WgradDiv fd,
                                           const TileMap tm) {
  FG_DMA_RING(P, R);
  constexpr int PA = P::PA, PB = P::PB, BK = P::BK;

  const int rsc = a.r * a.s * a.c;
  int tx, ty, split;  // rho tile, k tile, reduction split
  if (!tm.decode(blockIdx.x, tx, ty, split)) return;
  const int m0 = tx * P::TM, n0 = ty * P::TN;
  const int mbeg = split * a.mchunk;
  const int mend = min(a.mtot, mbeg + a.mchunk);
  const int nst = mend > mbeg ? (mend - mbeg + BK - 1) / BK : 0;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave / P::WGN) * P::WM, wn0 = (wave % P::WGN) * P::WN;

  const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc(
      (void *)a.x, 0, (int)x_span_bytes(a), kRsrcFlags);
  const __amdgpu_buffer_rsrc_t rs_dy = __builtin_amdgcn_make_buffer_rsrc(
      (void *)a.dy, 0, (int)((size_t)a.mtot * a.k * 2), kRsrcFlags);

  // A lane's reduction row m = mbeg + BK * st + krow is decoded into (n, p, q)
  // once, with multiply-shift division; each stage then advances it by BK rows
  // with adds and at most one carry into p and one into n (BK = dq + Q * (dp +
  // P * dn) with dq < Q, dp < P). Integer multiplies run at a quarter of the
  // VALU rate: a division per stage costs more VALU time than the MFMAs leave
  // free. The input position (hq, wq) is that of tap (0, 0); the lane's tap
  // offset (h0, w0) enters the bounds check and the byte offset. Slots whose
  // column is the same in every instruction share one tap.
  const MnSlot<PA> sa = mn_slots<P::RBA, PA>(wave, lane);
  const MnSlot<PB> sb = mn_slots<P::RBB, PB>(wave, lane);
  constexpr int NTAP = P::RBA > 256 ? PA : 1;
  const int pixb = a.ldx * 2, rowb = a.w * pixb, imgb = a.h * rowb;
  int h0[NTAP], w0[NTAP], hq[PA], wq[PA], ox[PA], od[PB];
#pragma unroll
  for (int jj = 0; jj < PA; ++jj) {
    const int rho = m0 + sa.ncol[jj];
    const int tap = rho / a.c, tr = tap / a.s;
    const int th = tr - a.ph, tw = tap - tr * a.s - a.pw;
    if (jj < NTAP) {
      h0[jj] = rho < rsc ? th : -(1 << 29);  // never inside the image
      w0[jj] = tw;
    }
    const int m = mbeg + sa.krow[jj];
    const unsigned nn = fd.pq.div((unsigned)m);
    const unsigned rem = (unsigned)m - nn * (unsigned)(a.p * a.q);
    const unsigned pp = fd.q.div(rem);
    hq[jj] = (int)pp * a.sh;
    wq[jj] = (int)(rem - pp * (unsigned)a.q) * a.sw;
    ox[jj] = (int)nn * imgb + (hq[jj] + th) * rowb + (wq[jj] + tw) * pixb +
             (rho - tap * a.c) * 2;
  }
#pragma unroll
  for (int jj = 0; jj < PB; ++jj)
    od[jj] = n0 + sb.ncol[jj] < a.k
                 ? ((mbeg + sb.krow[jj]) * a.k + n0 + sb.ncol[jj]) * 2
                 : -1;
  const int dq = BK % a.q, dpt = BK / a.q, dp = dpt % a.p, dn = dpt / a.p;
  const int inc_w = dq * a.sw, inc_h = dp * a.sh;
  const int inc_o = inc_w * pixb + inc_h * rowb + dn * imgb;
  const int wlim = a.q * a.sw, hlim = a.p * a.sh;
  const int wrap_o = a.sh * rowb - wlim * pixb;  // q wraps into p
  const int hwrap_o = imgb - hlim * rowb;        // p wraps into n
  const int inc_d = BK * a.k * 2;
  const int mleft = mend - mbeg;

  auto issue = [&](int st, int slot) __attribute__((always_inline)) {
    uint8_t *ta = R.a[slot], *tb = R.b[slot];
#pragma unroll
    for (int jj = 0; jj < PA; ++jj) {
      const int jt = NTAP == 1 ? 0 : jj;
      const bool v = sa.krow[jj] < mleft - BK * st &&
                     (unsigned)(hq[jj] + h0[jt]) < (unsigned)a.h &&
                     (unsigned)(wq[jj] + w0[jt]) < (unsigned)a.w;
      dma16(rs_x, ta + dma_dst<PA>(wave, jj), v ? (unsigned)ox[jj] : kOOB);
      wq[jj] += inc_w;
      hq[jj] += inc_h;
      ox[jj] += inc_o;
      if (wq[jj] >= wlim) {
        wq[jj] -= wlim;
        hq[jj] += a.sh;
        ox[jj] += wrap_o;
      }
      if (hq[jj] >= hlim) {
        hq[jj] -= hlim;
        ox[jj] += hwrap_o;
      }
    }
#pragma unroll
    for (int jj = 0; jj < PB; ++jj) {
      const bool v = sb.krow[jj] < mleft - BK * st && od[jj] >= 0;
      dma16(rs_dy, tb + dma_dst<PB>(wave, jj), v ? (unsigned)od[jj] : kOOB);
      od[jj] += od[jj] >= 0 ? inc_d : 0;
    }
  };

  f32x16 acc[P::FM][P::FN];
  zero<P>(acc);
  pipeline<P, false, false>(acc, R, nst, wm0, wn0, lane, issue);
  if constexpr (P::WM % 64 == 0 && P::WN == 64) {
    // 8 KiB of the ring per wave, a-side arrays first (constant indices only)
    constexpr int WPA = P::A_BYTES / 8192;  // waves per array
    static_assert(P::A_BYTES % 8192 == 0 && P::A_BYTES == P::B_BYTES &&
                      (P::NW + WPA - 1) / WPA <= 2 * P::NS,
                  "the store stages 8 KiB per wave in the ring");
    __syncthreads();  // every wave is done reading the ring
    uint8_t *buf = R.a[0];
#pragma unroll
    for (int k = 1; k < (P::NW + WPA - 1) / WPA; ++k)
      if (wave / WPA == k) buf = k < P::NS ? R.a[k] : R.b[k - P::NS];
    buf += (wave % WPA) * 8192;
    store_rho<P, SPLIT>(acc, buf, a, rsc, m0 + wm0, n0 + wn0, lane, split);
  } else {
    store_rho_direct<P, SPLIT>(acc, a, rsc, m0 + wm0, n0 + wn0, lane, split);
  }
}

template <class P, bool SPLIT>
__global__ __launch_bounds__(P::NT, P::WPE) void wgrad_dma_kernel(WgradArgs a, WgradDiv fd,
                                                                  TileMap tm) {
  wgrad_tile<P, SPLIT>(a, fd, tm);
}

template <class P>
static hipError_t launch_tile(const WgradArgs &a, hipStream_t st) {
  const WgradDiv fd{make_fastdiv((uint32_t)(a.p * a.q)), make_fastdiv((uint32_t)a.q)};
  TileMap tm{(a.r * a.s * a.c + P::TM - 1) / P::TM, (a.k + P::TN - 1) / P::TN, a.nsplit, 0,
             kOutputMajor};
  tm.per = (tm.n0 * tm.n1 * tm.n2 + 7) / 8;
  const auto k = a.nsplit > 1 ? wgrad_dma_kernel<P, true> : wgrad_dma_kernel<P, false>;
  hipLaunchKernelGGL(k, dim3(8 * tm.per), dim3(P::NT), 0, st, a, fd, tm);
  return hipGetLastError();
}

}  // namespace dma

// ---------------------------------------------------------------------------
bool data_halo_ok(const DataConvArgs &a) {
  if (a.nphase != 1 || a.istr != 1 || a.cr % 32 != 0) return false;
  const Phase &P = a.ph[0];
  if ((P.dstep != 1 && P.dstep != -1) || P.nr != 3 || P.ns != 3 || P.mw <= 0 ||
      dma::TN % P.mw != 0)
    return false;
  const int rt = dma::TN / P.mw;  // output rows per tile
  if (P.mh % rt != 0 || (rt + 2) * (P.mw + 2) > dma::kPatchRows) return false;
  return act_span_bytes(a) < 0x7FFFFFFFull &&
         (size_t)a.wbytes < 0x7FFFFFFFull;
}

static hipError_t launch_data_conv_halo(const DataConvArgs &a, bool w_kmajor,
                                 hipStream_t st) {
  const int npix = a.n * a.ph[0].mh * a.ph[0].mw;
  const int tco = (a.co + dma::TM - 1) / dma::TM, tpix = (npix + dma::TN - 1) / dma::TN;
  dma::TileMap tm = dma::weight_major(a)
                        ? dma::TileMap{tpix, tco, a.nsplit, 0, dma::kWeightMajor}
                        : dma::TileMap{a.nsplit, tco, tpix, 0, dma::kOutputMajor};
  tm.per = (tm.n0 * tm.n1 * tm.n2 + 7) / 8;
  dim3 grid(8 * tm.per), block(dma::HaloRun::NT);
  const bool split = a.nsplit > 1;
  if (w_kmajor) {
    if (split)
      hipLaunchKernelGGL((dma::data_conv_halo_kernel<dma::HaloRun, true, true>),
                         grid, block, 0, st, a, tm);
    else
      hipLaunchKernelGGL((dma::data_conv_halo_kernel<dma::HaloRun, true, false>),
                         grid, block, 0, st, a, tm);
  } else {
    if (split)
      hipLaunchKernelGGL((dma::data_conv_halo_kernel<dma::HaloRun, false, true>),
                         grid, block, 0, st, a, tm);
    else
      hipLaunchKernelGGL((dma::data_conv_halo_kernel<dma::HaloRun, false, false>),
                         grid, block, 0, st, a, tm);
  }
  return hipGetLastError();
}

static hipError_t launch_data_conv_dma(const DataConvArgs &a0, bool w_kmajor,
                                       hipStream_t st) {
  using C = dma::DataRun;
  DataConvArgs a = a0;
  const dma::TileMap tm = dma::data_tile_map(a, C::T, C::T);
  dim3 grid(8 * tm.per), block(C::NT);
  const bool split = a.nsplit > 1;
  if (w_kmajor) {
    if (split)
      hipLaunchKernelGGL((dma::data_conv_dma_kernel<C, true, true>), grid, block, 0,
                         st, a, tm);
    else
      hipLaunchKernelGGL((dma::data_conv_dma_kernel<C, true, false>), grid, block, 0,
                         st, a, tm);
  } else {
    if (split)
      hipLaunchKernelGGL((dma::data_conv_dma_kernel<C, false, true>), grid, block, 0,
                         st, a, tm);
    else
      hipLaunchKernelGGL((dma::data_conv_dma_kernel<C, false, false>), grid, block,
                         0, st, a, tm);
  }
  return hipGetLastError();
}

bool data_tile_ok(const DataConvArgs &a) {
  return act_span_bytes(a) < 0x7FFFFFFFull && (size_t)a.wbytes < 0x7FFFFFFFull;
}

DataTileMode data_tile_mode(const DataConvArgs &a, DataTile tile) {
  const int bk = tile == DataTile::k256 || tile == DataTile::k128d32 ? 32 : dma::Data64::BK;
  static_assert(dma::Data64::BK == dma::Data64x128::BK && dma::Data64::BK == dma::Data128::BK);
  bool gen = a.cr % bk != 0;
  for (int i = 0; a.nsplit > 1 && i < a.nphase; ++i)  // parts that end within a stage
    gen |= part_len(a.ph[i].nr * a.ph[i].ns * a.cr, a.unit, a.nchunk) % bk != 0;
  return {gen, a.nsplit == 1 && a.nchunk > 1};
}

hipError_t launch_data_conv_tile(const DataConvArgs &a, DataTile tile, bool w_kmajor,
                                 hipStream_t st) {
  const auto [gen, fold] = data_tile_mode(a, tile);
  switch (tile) {
    case DataTile::k64:
      return dma::launch_data_tile<dma::Data64>(a, w_kmajor, gen, fold, st);
    case DataTile::k64x128:
      return dma::launch_data_tile<dma::Data64x128>(a, w_kmajor, gen, fold, st);
    case DataTile::k128:
      return dma::launch_data_tile<dma::Data128>(a, w_kmajor, gen, fold, st);
    case DataTile::k128d32:
      return dma::launch_data_tile<dma::Data128d32>(a, w_kmajor, gen, fold, st);
    case DataTile::k256:
      return data_halo_ok(a) ? launch_data_conv_halo(a, w_kmajor, st)
             : gen           ? dma::launch_data_tile<dma::Data256>(a, w_kmajor, true, false, st)
                             : launch_data_conv_dma(a, w_kmajor, st);
    default: return hipErrorInvalidValue;
  }
}

bool wgrad_tile_ok(const WgradArgs &a) {
  return x_span_bytes(a) < 0x7FFFFFFFull && (size_t)a.mtot * a.k * 2 < 0x7FFFFFFFull;
}

hipError_t launch_wgrad_tile(const WgradArgs &a, WgTile tile, hipStream_t st) {
  return tile == WgTile::k256   ? dma::launch_tile<dma::Tile256>(a, st)
         : tile == WgTile::k128 ? dma::launch_tile<dma::Tile128>(a, st)
                                : dma::launch_tile<dma::Tile64>(a, st);
}

}  // namespace fg
