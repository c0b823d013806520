// Implicit-GEMM fp16 convolutions on fp16 MFMA (fp32 accumulate) for gfx950.
//
// Data convolutions (forward, input gradient, transposed forward) are one
// kernel: GEMM rows are output channels, columns are output positions of one
// phase, and the reduction runs over (tap, input channel). The input image is
// gathered straight from NHWC memory (zero outside the image); nothing is
// materialised. Strided input gradients and transposed convolutions are split
// into output phases so that no multiply touches an inserted zero. Shapes
// that give too few output tiles to fill the GPU split the reduction across
// workgroups; fp32 partials are then summed in split order by a second kernel
// that also applies the epilogue.
//
// The kernel gradient is a second kernel: rows are (tap, input channel),
// columns output channels, reduction over all output positions, split across
// workgroups with fp32 partials summed afterwards in a fixed order.
//
// Both run the tensors that a buffer resource cannot address; the others take
// the LDS-DMA kernels (conv_dma.hip). The planners of all of them, the split
// reductions and the one-channel head are here too.
//
// Both kernels stage 64-deep reduction slices of each operand in LDS (double
// buffered, one barrier per slice). LDS rows are 128 bytes with the eight
// 16-byte chunks of a row permuted by an XOR of row bits, so the 16-byte MFMA
// operand reads of 8 consecutive rows hit distinct banks. Operands whose
// reduction dimension is strided in memory are transposed in registers on
// their way to LDS. Each of the 4 waves owns a (BM/2) x (BN/2) block of the
// tile and issues v_mfma_f32_32x32x16_f16 over it.
#include <algorithm>
#include <cstring>

#include "common.h"
#include "internal.h"

namespace fg {

constexpr int BK = 64;        // reduction slice per LDS stage (halves)

// 256x256 tile, 8 waves (two per SIMD) of 128x64: one wave's MFMAs overlap
// the other's address, load and LDS instructions.
using BigCfg = Cfg<256, 256, 2, 4>;
// 128x128 tile, 4 waves of 64x64; two workgroups fit on a CU.
using SmallCfg = Cfg<128, 128, 2, 2>;

// Offset (in halves) of 16-byte chunk `chunk` (0..7) of LDS row `row`.
__device__ __forceinline__ int lds_idx(int row, int chunk) {
  return row * BK + ((chunk ^ ((row ^ (row >> 3)) & 7)) << 3);
}

// ---------------------------------------------------------------------------
template <class C>
struct Core {
  static constexpr int FM = C::FM, FN = C::FN;
  f32x16 acc[FM][FN];

  __device__ void zero() {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  }

  __device__ void step(const uint16_t *sA, const uint16_t *sB, int wm0,
                       int wn0, int lane) {
    const int r = lane & 31, kh = lane >> 5;
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      u32x4 a[FM], b[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i)
        a[i] = *reinterpret_cast<const u32x4 *>(
            sA + lds_idx(wm0 + i * 32 + r, 2 * ks + kh));
#pragma unroll
      for (int j = 0; j < FN; ++j)
        b[j] = *reinterpret_cast<const u32x4 *>(
            sB + lds_idx(wn0 + j * 32 + r, 2 * ks + kh));
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = mfma32(a[i], b[j], acc[i][j]);
    }
  }
};

// Transpose 4 rows of 8 halves (row = reduction index) into 8 LDS rows
// row0..row0+7 at 4-half unit kq (8 bytes each).
__device__ __forceinline__ void store_t4x8(uint16_t *s, int row0, int kq,
                                           const u32x4 q[4]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    u32x2 lo, hi;
    lo[0] = pack_lo(q[0][e], q[1][e]);
    lo[1] = pack_lo(q[2][e], q[3][e]);
    hi[0] = pack_hi(q[0][e], q[1][e]);
    hi[1] = pack_hi(q[2][e], q[3][e]);
    const int r0 = row0 + 2 * e, r1 = r0 + 1;
    *reinterpret_cast<u32x2 *>(s + lds_idx(r0, kq >> 1) + (kq & 1) * 4) = lo;
    *reinterpret_cast<u32x2 *>(s + lds_idx(r1, kq >> 1) + (kq & 1) * 4) = hi;
  }
}

__device__ __forceinline__ u32x4 ldg16(const uint16_t *p) {
  return *reinterpret_cast<const u32x4 *>(p);
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

// ---------------------------------------------------------------------------
// Data convolution kernel.
//   WK    weights are k-major (forward: reduction contiguous per output
//         channel) or mn-major (input gradient / transposed: output channel
//         contiguous), the latter transposed in registers.
//   FAST  reduction channels are a multiple of BK, so a slice is one tap.
//   SPLIT the reduction is split across workgroups: write fp32 partials
//         (a.nsplit > 1) instead of the fp16 output.
// blockIdx.z = phase * nsplit + split.
template <class C, bool WK, bool FAST, bool SPLIT>
__global__ __launch_bounds__(C::NT) void data_conv_staged_kernel(DataConvArgs a) {
  constexpr int BM = C::BM, BN = C::BN, NT = C::NT;
  __shared__ __attribute__((aligned(16))) uint16_t sA[2][BM * BK];
  __shared__ __attribute__((aligned(16))) uint16_t sB[2][BN * BK];

  const int phase = blockIdx.z / a.nsplit, split = blockIdx.z % a.nsplit;
  const Phase P = a.ph[phase];
  const int npix = a.n * P.mh * P.mw;
  const int n0 = blockIdx.x * BN;
  const int m0 = blockIdx.y * BM;
  if (n0 >= npix) return;
  const int ntap = P.nr * P.ns;
  const int ktot = ntap * a.cr;
  const int nk = (ktot + BK - 1) / BK;
  const int kchunk = (nk + a.nsplit - 1) / a.nsplit;
  const int kbeg = min(nk, split * kchunk), kend = min(nk, kbeg + kchunk);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave / C::WGN) * C::WM, wn0 = (wave % C::WGN) * C::WN;

  // --- B (activation gather) loader state: 8 threads per column (one
  // 16-byte chunk each), NT/8 columns per pass, BCOL passes.
  constexpr int RPP = NT / 8;  // rows per pass
  constexpr int BCOL = BN / RPP;
  const int bc8 = tid & 7;
  int bbase[BCOL], bh[BCOL], bw[BCOL];
#pragma unroll
  for (int i = 0; i < BCOL; ++i) {
    int col = n0 + (tid >> 3) + RPP * i;
    if (col < npix) {
      int b = col % P.mw, t = col / P.mw;
      int aa = t % P.mh, nn = t / P.mh;
      bh[i] = aa * a.istr;
      bw[i] = b * a.istr;
      bbase[i] = ((nn * a.hi + bh[i]) * a.wi + bw[i]) * a.ldi;
    } else {
      bh[i] = -(1 << 29);  // fails every bounds check
      bw[i] = 0;
      bbase[i] = 0;
    }
  }

  constexpr int AROW = BM / RPP;
  constexpr int AUNITS = (BK / 4) * (BM / 8);
  constexpr int AUPT = (AUNITS + NT - 1) / NT;
  u32x4 ra[WK ? AROW : 4 * AUPT];
  u32x4 rb[BCOL];

  // tap t -> input offset (dh, dw) and kernel element offset woff = r*S + s
  auto tap_geom = [&](int t, int &dh, int &dw, int &woff) {
    int i = t / P.ns, j = t - (t / P.ns) * P.ns;
    dh = P.dh0 + P.dstep * i;
    dw = P.dw0 + P.dstep * j;
    woff = (P.r0 + P.rstep * i) * a.s + (P.s0 + P.rstep * j);
  };

  auto load = [&](int kt) {
    const int k0 = kt * BK;
    int ft = 0, fcr = 0, fdh = 0, fdw = 0, fwoff = 0;
    if (FAST) {  // the whole slice lies in one tap
      ft = k0 / a.cr;
      fcr = k0 - ft * a.cr;
      tap_geom(ft, fdh, fdw, fwoff);
    }
    // B: activations
    {
      int kk = k0 + bc8 * 8, dh, dw, woff, cr;
      bool kv = kk < ktot;
      if (FAST) {
        dh = fdh; dw = fdw; cr = fcr + bc8 * 8;
      } else {
        int t = kv ? kk / a.cr : 0;
        cr = kv ? kk - t * a.cr : 0;
        tap_geom(t, dh, dw, woff);
      }
      const int delta = (dh * a.wi + dw) * a.ldi + cr;
#pragma unroll
      for (int i = 0; i < BCOL; ++i) {
        int hh = bh[i] + dh, ww = bw[i] + dw;
        bool v = kv && hh >= 0 && hh < a.hi && ww >= 0 && ww < a.wi;
        rb[i] = v ? ldg16(a.act + (size_t)(bbase[i] + delta)) : u32x4{0, 0, 0, 0};
      }
    }
    // A: weights
    if (WK) {
      int kk = k0 + bc8 * 8, dh, dw, woff, cr;
      bool kv = kk < ktot;
      if (FAST) {
        woff = fwoff; cr = fcr + bc8 * 8;
      } else {
        int t = kv ? kk / a.cr : 0;
        cr = kv ? kk - t * a.cr : 0;
        tap_geom(t, dh, dw, woff);
      }
      const uint16_t *src = a.wgt + (size_t)woff * a.cr + cr;
#pragma unroll
      for (int i = 0; i < AROW; ++i) {
        int row = m0 + (tid >> 3) + RPP * i;
        ra[i] = (kv && row < a.co) ? ldg16(src + (size_t)row * a.ldw)
                                   : u32x4{0, 0, 0, 0};
      }
    } else {
#pragma unroll
      for (int u = 0; u < AUPT; ++u) {
        int unit = tid + u * NT;
        int cg = unit % (BM / 8), kq = unit / (BM / 8);
        int kk = k0 + kq * 4;
        int row = m0 + cg * 8;
        bool v = unit < AUNITS && kk < ktot && row < a.co;
        int dh, dw, woff, cr;
        if (FAST) {
          woff = fwoff; cr = fcr + kq * 4;
        } else {
          int t = v ? kk / a.cr : 0;
          cr = v ? kk - t * a.cr : 0;
          tap_geom(t, dh, dw, woff);
        }
        // 4 consecutive reduction indices stay inside one tap (cr % 8 == 0)
        const uint16_t *src =
            a.wgt + (size_t)cr * a.w_red + (size_t)woff * a.w_tap + row;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          ra[4 * u + e] = v ? ldg16(src + (size_t)e * a.w_red) : u32x4{0, 0, 0, 0};
      }
    }
  };

  auto store = [&](int buf) {
#pragma unroll
    for (int i = 0; i < BCOL; ++i)
      *reinterpret_cast<u32x4 *>(&sB[buf][lds_idx((tid >> 3) + RPP * i, bc8)]) =
          rb[i];
    if (WK) {
#pragma unroll
      for (int i = 0; i < AROW; ++i)
        *reinterpret_cast<u32x4 *>(
            &sA[buf][lds_idx((tid >> 3) + RPP * i, bc8)]) = ra[i];
    } else {
#pragma unroll
      for (int u = 0; u < AUPT; ++u) {
        int unit = tid + u * NT;
        if (unit < AUNITS) {
          int cg = unit % (BM / 8), kq = unit / (BM / 8);
          store_t4x8(sA[buf], cg * 8, kq, &ra[4 * u]);
        }
      }
    }
  };

  Core<C> core;
  core.zero();
  if (kbeg < kend) {
    load(kbeg);
    store(0);
  }
  __syncthreads();
  for (int kt = kbeg; kt < kend; ++kt) {
    const int cur = (kt - kbeg) & 1;
    if (kt + 1 < kend) load(kt + 1);
    core.step(sA[cur], sB[cur], wm0, wn0, lane);
    if (kt + 1 < kend) store(cur ^ 1);
    __syncthreads();
  }

  // --- epilogue: lane holds 4 consecutive output channels of one position.
  constexpr int FM = C::FM, FN = C::FN;
  const size_t out_total = (size_t)a.n * a.ho * a.wo * a.co;
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    int col = n0 + wn0 + j * 32 + (lane & 31);
    if (col >= npix) continue;
    int b = col % P.mw, t = col / P.mw;
    int aa = t % P.mh, nn = t / P.mh;
    // split partials are dense; the output has its own pixel stride
    size_t obase = ((size_t)(nn * a.ho + aa * a.ostr + P.ooh) * a.wo +
                    b * a.ostr + P.oow) *
                   (SPLIT ? a.co : a.ldo);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        int co = m0 + wm0 + i * 32 + 8 * g + 4 * (lane >> 5);
        if (co >= a.co) continue;
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = core.acc[i][j][4 * g + e];
        if (SPLIT) {
          f32x4 o = {v[0], v[1], v[2], v[3]};
          *reinterpret_cast<f32x4 *>(a.part + split * out_total + obase + co) = o;
        } else {
          epilogue4(v, a.epi, a.gate + obase + co, a.out + obase + co);
          *reinterpret_cast<u32x2 *>(a.out + obase + co) =
              to_h4(v[0], v[1], v[2], v[3]);
        }
      }
  }
}

// Elements i4..i4+3 of part[first], part[first + step], ... (first < nsplit)
// summed in that order. A short sum is bound by the latency of its loads, so
// four are issued before their adds; one load a step, as before, waits for
// each in turn. 3x3 kernel gradients, 16 channels (2304 outputs): 4.4 -> 3.2
// us; 128 channels, 5.1 -> 4.3; 1x1 of 768 channels, 12.2 -> 11.1.
__device__ __forceinline__ f32x4 sum_parts(const float *part, int first, int step, int nsplit,
                                           int64_t len, int64_t i4) {
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  int k = first;
  bool any = false;
  auto add = [&](const f32x4 &v) {
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] = any ? s[e] + v[e] : v[e];
    any = true;
  };
  for (; k + 3 * step < nsplit; k += 4 * step) {
    f32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      v[u] = *reinterpret_cast<const f32x4 *>(part + (size_t)(k + u * step) * len + i4);
#pragma unroll
    for (int u = 0; u < 4; ++u) add(v[u]);
  }
  if (k >= nsplit) return s;
  // the last 1 to 3, loaded together too (absent ones repeat the first)
  f32x4 v[3];
#pragma unroll
  for (int u = 0; u < 3; ++u)
    v[u] = *reinterpret_cast<const f32x4 *>(
        part + (size_t)(k + u * step < nsplit ? k + u * step : first) * len + i4);
#pragma unroll
  for (int u = 0; u < 3; ++u)
    if (k + u * step < nsplit) add(v[u]);
  return s;
}

// Sum nsplit fp32 partial arrays of len elements (dense, co channels per
// pixel) in split order, apply the epilogue, round to fp16 into out (and
// read gate) at pixel stride ldo. len and co are multiples of 4.
__global__ __launch_bounds__(256) void split_epilogue_kernel(
    const float *part, int nsplit, int64_t len, int co, int ldo, int epi,
    const uint16_t *gate, uint16_t *out) {
  int64_t i4 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (i4 >= len) return;
  const f32x4 s = sum_parts(part, 0, 1, nsplit, len, i4);
  const int64_t pix = i4 / co;
  const int64_t o = pix * ldo + (i4 - pix * co);
  float v[4] = {s[0], s[1], s[2], s[3]};
  epilogue4(v, epi, gate + o, out + o);
  *reinterpret_cast<u32x2 *>(out + o) = to_h4(v[0], v[1], v[2], v[3]);
}

// ---------------------------------------------------------------------------
// Kernel-gradient kernel: rows rho = (tap, c) of the x patch, columns k.
template <class C, bool SPLIT>
__global__ __launch_bounds__(C::NT) void wgrad_staged_kernel(WgradArgs a) {
  constexpr int BM = C::BM, BN = C::BN, NT = C::NT;
  __shared__ __attribute__((aligned(16))) uint16_t sA[2][BM * BK];
  __shared__ __attribute__((aligned(16))) uint16_t sB[2][BN * BK];

  const int rsc = a.r * a.s * a.c;
  const int m0 = blockIdx.x * BM;  // rho
  const int n0 = blockIdx.y * BN;  // k
  const int split = blockIdx.z;
  const int mbeg = split * a.mchunk;
  const int mend = min(a.mtot, mbeg + a.mchunk);
  const int nk = mend > mbeg ? (mend - mbeg + BK - 1) / BK : 0;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave / C::WGN) * C::WM, wn0 = (wave % C::WGN) * C::WN;
  const int pq = a.p * a.q;

  constexpr int AUNITS = (BK / 4) * (BM / 8);
  constexpr int AUPT = (AUNITS + NT - 1) / NT;
  constexpr int BUNITS = (BK / 4) * (BN / 8);
  constexpr int BUPT = (BUNITS + NT - 1) / NT;
  u32x4 ra[4 * AUPT], rb[4 * BUPT];

  // per A unit: the tap and channel of its 8 rows are fixed for the block
  int ar[AUPT], as_[AUPT], ac[AUPT];
  bool arv[AUPT];
#pragma unroll
  for (int u = 0; u < AUPT; ++u) {
    int unit = tid + u * NT;
    int rho = m0 + (unit % (BM / 8)) * 8;
    arv[u] = unit < AUNITS && rho < rsc;
    int t = rho / a.c;
    ac[u] = rho - t * a.c;
    ar[u] = t / a.s;
    as_[u] = t - ar[u] * a.s;
  }

  auto load = [&](int kt) {
    const int k0 = mbeg + kt * BK;
#pragma unroll
    for (int u = 0; u < AUPT; ++u) {
      int unit = tid + u * NT;
      int mq = unit / (BM / 8);
      int m = k0 + mq * 4;
      int nn = m / pq, rem = m - nn * pq;
      int p = rem / a.q, q = rem - p * a.q;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        int hh = p * a.sh - a.ph + ar[u], ww = q * a.sw - a.pw + as_[u];
        bool v = arv[u] && (m + e) < mend && hh >= 0 && hh < a.h && ww >= 0 &&
                 ww < a.w;
        ra[4 * u + e] =
            v ? ldg16(a.x + ((size_t)((nn * a.h + hh) * a.w + ww)) * a.ldx + ac[u])
              : u32x4{0, 0, 0, 0};
        // next reduction row: advance (n, p, q)
        if (++q == a.q) {
          q = 0;
          if (++p == a.p) {
            p = 0;
            ++nn;
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < BUPT; ++u) {
      int unit = tid + u * NT;
      int kg = unit % (BN / 8), mq = unit / (BN / 8);
      int k = n0 + kg * 8;
      int m = k0 + mq * 4;
      bool uv = unit < BUNITS && k < a.k;
      const uint16_t *src = a.dy + (size_t)m * a.k + k;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        rb[4 * u + e] = (uv && (m + e) < mend) ? ldg16(src + (size_t)e * a.k)
                                               : u32x4{0, 0, 0, 0};
    }
  };

  auto store = [&](int buf) {
#pragma unroll
    for (int u = 0; u < AUPT; ++u) {
      int unit = tid + u * NT;
      if (unit < AUNITS)
        store_t4x8(sA[buf], (unit % (BM / 8)) * 8, unit / (BM / 8), &ra[4 * u]);
    }
#pragma unroll
    for (int u = 0; u < BUPT; ++u) {
      int unit = tid + u * NT;
      if (unit < BUNITS)
        store_t4x8(sB[buf], (unit % (BN / 8)) * 8, unit / (BN / 8), &rb[4 * u]);
    }
  };

  Core<C> core;
  core.zero();
  if (nk > 0) {
    load(0);
    store(0);
  }
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int cur = kt & 1;
    if (kt + 1 < nk) load(kt + 1);
    core.step(sA[cur], sB[cur], wm0, wn0, lane);
    if (kt + 1 < nk) store(cur ^ 1);
    __syncthreads();
  }

  constexpr int FM = C::FM, FN = C::FN;
  bool bad = false;
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    int k = n0 + wn0 + j * 32 + (lane & 31);
    if (k >= a.k) continue;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        int rho = m0 + wm0 + i * 32 + 8 * g + 4 * (lane >> 5);
        if (rho >= rsc) continue;
        const f32x16 &c = core.acc[i][j];
        if (!SPLIT) {
          const u32x2 h = to_h4(c[4 * g], c[4 * g + 1], c[4 * g + 2], c[4 * g + 3]);
          bad |= nonfinite_h2(h[0]) | nonfinite_h2(h[1]);
          *reinterpret_cast<u32x2 *>(a.dw + (size_t)k * rsc + rho) = h;
        } else {
          f32x4 o = {c[4 * g], c[4 * g + 1], c[4 * g + 2], c[4 * g + 3]};
          *reinterpret_cast<f32x4 *>(
              a.part + ((size_t)split * a.k + k) * rsc + rho) = o;
        }
      }
  }
  if (!SPLIT && a.flag) flag_nonfinite(a.flag, bad);
}

// Sum nsplit fp32 partial arrays of len elements in split order, round to
// fp16. len is a multiple of 4. flag (or null): set to 1 if a result is
// +-inf or NaN.
__global__ __launch_bounds__(256) void split_reduce_kernel(const float *part,
                                                           int nsplit,
                                                           int64_t len,
                                                           uint16_t *out,
                                                           int32_t *flag) {
  int64_t i4 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  bool bad = false;
  if (i4 < len) {
    const f32x4 s = sum_parts(part, 0, 1, nsplit, len, i4);
    const u32x2 h = to_h4(s[0], s[1], s[2], s[3]);
    bad = nonfinite_h2(h[0]) | nonfinite_h2(h[1]);
    *reinterpret_cast<u32x2 *>(out + i4) = h;
  }
  if (flag) flag_nonfinite(flag, bad);
}

// Same sum when the partials are many and short (nsplit large, len small):
// one workgroup per 4 outputs; thread t adds splits t, t+256, ... in order,
// then a fixed-shape tree in LDS combines the 256 thread sums.
__global__ __launch_bounds__(256) void split_reduce_wide_kernel(
    const float *part, int nsplit, int64_t len, uint16_t *out, int32_t *flag) {
  __shared__ f32x4 red[256];
  const int64_t i4 = (int64_t)blockIdx.x * 4;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  if ((int)threadIdx.x < nsplit) s = sum_parts(part, threadIdx.x, 256, nsplit, len, i4);
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      f32x4 a = red[threadIdx.x], b = red[threadIdx.x + w];
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] += b[e];
      red[threadIdx.x] = a;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    f32x4 t = red[0];
    const u32x2 h = to_h4(t[0], t[1], t[2], t[3]);
    *reinterpret_cast<u32x2 *>(out + i4) = h;
    if (flag && (nonfinite_h2(h[0]) | nonfinite_h2(h[1]))) *flag = 1;
  }
}

// Same sum for a moderate number of longer partials (more than
// kMaxSerialSplit splits): each workgroup covers 64 outputs as 16 groups of
// 4, with 16 lanes per group; lane j adds splits j, j + 16, ... in order,
// then a fixed-shape tree combines the 16 lane sums. (In the serial sum of
// split_reduce_kernel the loads of a group wait for the group before.)
constexpr int kMaxSerialSplit = 16;
__global__ __launch_bounds__(256) void split_reduce_multi_kernel(
    const float *part, int nsplit, int64_t len, uint16_t *out, int32_t *flag) {
  __shared__ f32x4 red[16][16];  // [lane][group]
  const int grp = threadIdx.x & 15, lane = threadIdx.x >> 4;
  const int64_t i4 = ((int64_t)blockIdx.x * 16 + grp) * 4;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  if (i4 < len) s = sum_parts(part, lane, 16, nsplit, len, i4);  // nsplit > 16 > lane
  red[lane][grp] = s;
  __syncthreads();
  for (int w = 8; w > 0; w >>= 1) {
    if (lane < w) {
      f32x4 a = red[lane][grp], b = red[lane + w][grp];
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] += b[e];
      red[lane][grp] = a;
    }
    __syncthreads();
  }
  bool bad = false;
  if (lane == 0 && i4 < len) {
    const f32x4 t = red[0][grp];
    const u32x2 h = to_h4(t[0], t[1], t[2], t[3]);
    bad = nonfinite_h2(h[0]) | nonfinite_h2(h[1]);
    *reinterpret_cast<u32x2 *>(out + i4) = h;
  }
  if (flag) flag_nonfinite(flag, bad);
}

// ---------------------------------------------------------------------------
// Single-output-channel 1x1 convolution (the network head): bandwidth-bound,
// so no MFMA. L lanes (a power of two) cooperate on one position.
__global__ __launch_bounds__(256) void head_fwd_kernel(
    const uint16_t *x, const uint16_t *w, uint16_t *y, int64_t npix, int c,
    int L, int logL, int epi, const uint16_t *gate) {
  const int lane = threadIdx.x & 63;
  const int sub = lane & (L - 1);
  const int per_wave = 64 / L;
  const int64_t wave_id = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  const int nchunk = c / 8;
  for (int64_t base = wave_id * per_wave; base < npix;
       base += nwaves * per_wave) {
    int64_t pix = base + (lane >> logL);
    float acc = 0.f;
    if (pix < npix) {
      for (int ch = sub; ch < nchunk; ch += L) {
        u32x4 xv = ldg16(x + pix * c + ch * 8);
        u32x4 wv = ldg16(w + ch * 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc += h_to_f32((uint16_t)xv[e]) * h_to_f32((uint16_t)wv[e]);
          acc += h_to_f32((uint16_t)(xv[e] >> 16)) *
                 h_to_f32((uint16_t)(wv[e] >> 16));
        }
      }
    }
    for (int o = 1; o < L; o <<= 1) acc += __shfl_xor(acc, o, 64);
    if (pix < npix && sub == 0) {
      float v = acc;
      if (epi == FG_EPI_RELU) v = v > 0.f ? v : 0.f;
      if (epi == FG_EPI_GATE) v = h_to_f32(gate[pix]) > 0.f ? v : 0.f;
      y[pix] = f32_to_h(v);
    }
  }
}

// dx[m][c] = epi(dy[m] * w[c]); one thread per 8 channels.
__global__ __launch_bounds__(256) void head_bwd_data_kernel(
    const uint16_t *dy, const uint16_t *w, uint16_t *dx, int64_t npix, int c,
    int epi, const uint16_t *gate) {
  const int nchunk = c / 8;
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= npix * nchunk) return;
  int64_t pix = idx / nchunk;
  int ch = (int)(idx - pix * nchunk);
  float d = h_to_f32(dy[pix]);
  u32x4 wv = ldg16(w + ch * 8);
  u32x4 gv = u32x4{0, 0, 0, 0};
  if (epi == FG_EPI_GATE) gv = ldg16(gate + pix * c + ch * 8);
  u32x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float v0 = d * h_to_f32((uint16_t)wv[e]);
    float v1 = d * h_to_f32((uint16_t)(wv[e] >> 16));
    if (epi == FG_EPI_RELU) {
      v0 = v0 > 0.f ? v0 : 0.f;
      v1 = v1 > 0.f ? v1 : 0.f;
    } else if (epi == FG_EPI_GATE) {
      v0 = h_to_f32((uint16_t)gv[e]) > 0.f ? v0 : 0.f;
      v1 = h_to_f32((uint16_t)(gv[e] >> 16)) > 0.f ? v1 : 0.f;
    }
    o[e] = (uint32_t)f32_to_h(v0) | ((uint32_t)f32_to_h(v1) << 16);
  }
  *reinterpret_cast<u32x4 *>(dx + pix * c + ch * 8) = o;
}

// Partial kernel gradient of the head: block b sums positions
// [b*chunk, (b+1)*chunk) for all c channels into part[b][c] (fixed order).
constexpr int kHeadWgradThreads = 256;
__global__ __launch_bounds__(kHeadWgradThreads) void head_wgrad_kernel(
    const uint16_t *x, const uint16_t *dy, int64_t npix, int c, int64_t chunk,
    float *part) {
  __shared__ float red[kHeadWgradThreads * 8];
  const int nchunk = c / 8;
  const int rows = kHeadWgradThreads / nchunk;  // positions in flight
  const int ch = threadIdx.x % nchunk, row = threadIdx.x / nchunk;
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  int64_t beg = (int64_t)blockIdx.x * chunk;
  int64_t end = beg + chunk < npix ? beg + chunk : npix;
  if (row < rows) {
    // four positions per iteration, their loads issued together
    int64_t pix = beg + row;
    for (; pix + 3 * rows < end; pix += 4 * rows) {
      float d[4];
      u32x4 xv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        d[u] = h_to_f32(dy[pix + u * rows]);
        xv[u] = ldg16(x + (pix + u * rows) * c + ch * 8);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc[2 * e] += d[u] * h_to_f32((uint16_t)xv[u][e]);
          acc[2 * e + 1] += d[u] * h_to_f32((uint16_t)(xv[u][e] >> 16));
        }
    }
    for (; pix < end; pix += rows) {
      float d = h_to_f32(dy[pix]);
      u32x4 xv = ldg16(x + pix * c + ch * 8);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[2 * e] += d * h_to_f32((uint16_t)xv[e]);
        acc[2 * e + 1] += d * h_to_f32((uint16_t)(xv[e] >> 16));
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[threadIdx.x * 8 + e] = acc[e];
  __syncthreads();
  if (threadIdx.x < nchunk) {
    float s[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] = 0.f;
    for (int rr = 0; rr < rows; ++rr)
#pragma unroll
      for (int e = 0; e < 8; ++e) s[e] += red[(rr * nchunk + ch) * 8 + e];
#pragma unroll
    for (int e = 0; e < 8; ++e) part[(size_t)blockIdx.x * c + ch * 8 + e] = s[e];
  }
}

// ---------------------------------------------------------------------------
// Host side: tile selection and launchers.
namespace {

int64_t data_tiles(const DataConvArgs &a, int bm, int bn) {
  int64_t t = 0;
  for (int i = 0; i < a.nphase; ++i) {
    int64_t np = (int64_t)a.n * a.ph[i].mh * a.ph[i].mw;
    t += ((np + bn - 1) / bn) * ((a.co + bm - 1) / bm);
  }
  return t;
}

int64_t data_nk_max(const DataConvArgs &a) {
  int64_t nk = 0;
  for (int i = 0; i < a.nphase; ++i) {
    int64_t kt = (int64_t)a.ph[i].nr * a.ph[i].ns * a.cr;
    nk = std::max<int64_t>(nk, (kt + BK - 1) / BK);
  }
  return nk;
}

constexpr int64_t kCUs = 256;

// Work of a data convolution on tm x tn tiles: tiles over all phases, their
// reduction stages of bk in all (each phase has its own taps), the most of one.
struct DataWork {
  int32_t tiles, stages, longest;
};
struct PhaseWork {
  int32_t tiles[4], nk[4], nphase;
  PhaseWork(const DataConvArgs &a, int tm, int tn, int bk) : nphase(a.nphase) {
    const int tco = (a.co + tm - 1) / tm;
    for (int i = 0; i < nphase; ++i) {
      const Phase &P = a.ph[i];
      tiles[i] = (int32_t)(((int64_t)a.n * P.mh * P.mw + tn - 1) / tn) * tco;
      nk[i] = (P.nr * P.ns * a.cr + bk - 1) / bk;
    }
  }
  DataWork split(int ns) const {
    DataWork w{0, 0, 0};
    for (int i = 0; i < nphase; ++i) {
      const int32_t st = ns == 1 ? nk[i] : (nk[i] + ns - 1) / ns;
      w.tiles += tiles[i];
      w.stages += tiles[i] * st * ns;
      if (tiles[i]) w.longest = std::max(w.longest, st);
    }
    return w;
  }
};
DataWork data_work(const DataConvArgs &a, int tm, int tn, int bk) {
  return PhaseWork(a, tm, tn, bk).split(1);
}

// Plans of the last shapes a host thread asked for: a call asks at least twice
// (workspace, launch), a program for the same shapes every step, and working
// one out takes 1 to 2 us of the 5 that a launch costs the host. One place per
// hash: of two shapes that share one, each is worked out anew when its turn comes.
template <class Key, class Plan>
struct PlanMemo {
  static constexpr unsigned N = 64;
  struct Entry {
    Key key;
    Plan plan;
    bool set;
  };
  Entry e[N];  // zero-initialised
  // Keys are compared as bytes (filled over zeros).
  Entry &at(const Key &k) {
    const uint32_t *w = reinterpret_cast<const uint32_t *>(&k);
    uint32_t h = 2166136261u;
    for (size_t i = 0; i < sizeof(Key) / 4; ++i) h = (h ^ w[i]) * 16777619u;
    return e[(h ^ (h >> 15)) % N];
  }
};

}  // namespace

// Number of equal parts a reduction of nk stages is summed in, over 128 x 128 or
// (big) 256 x 256 tiles, by rates of workgroups in flop/s. The rates are those of
// earlier kernels, whose splits these parts were; they are part of what they define
// (the order of a forward pass's sums, the least workspace of a call) and need no
// update.
struct PartRates {
  double big, small, alone;              // alone: a 128 x 128 one with its CU to itself
  double partial_bw, launch_s, round_s;  // a split's partials and launch; per round of tiles
};
struct PartCount {
  bool big;
  int32_t n;
};
static PartCount part_count(int64_t tiles_big, int64_t tiles_small, int64_t nk, int64_t out,
                            bool allow_big, const PartRates &r, int max_n) {
  PartCount best{false, 1};
  double best_t = 1e30;
  for (int big = 0; big < 2; ++big) {
    if (big && !allow_big) continue;
    const int t = big ? 256 : 128;
    const int64_t tiles = big ? tiles_big : tiles_small, slots = big ? kCUs : 2 * kCUs;
    for (int ns = 1; ns <= max_n; ++ns) {
      if (ns > 1 && (nk + ns - 1) / ns < 4) break;
      const double rate = big ? r.big : tiles * ns <= kCUs ? r.alone : r.small;
      const int64_t rounds = (tiles * ns + slots - 1) / slots;
      double tt = rounds * (2.0 * t * t * BK * (double)((nk + ns - 1) / ns) / rate + r.round_s);
      if (ns > 1) tt += ns * (double)out * 8.0 / r.partial_bw + r.launch_s;
      if (tt < best_t * 0.98) {
        best_t = tt;
        best = PartCount{big != 0, ns};
      }
    }
  }
  return best;
}

// Summation order of a forward or transposed-forward pass, and the plan of the
// register-staged kernels: the reduction is summed in n equal parts, each
// from zero, and the parts are added in order. An activation's last bit decides
// ReLU gates downstream (a network's input gradient moves by 3-4% in 2-norm when
// one layer's sums are reordered), so the order of a shape is fixed by this
// function alone, and every kernel that takes the shape keeps it: as parts of a
// split, or by folding its accumulators at the same places (data_tile). big: whole-
// row shapes take channels before taps.
static PartCount sum_order(const DataConvArgs &a) {
  const bool lds = a.cr % 32 == 0 && data_tile_ok(a);
  const PartRates r{3.0e12, lds ? 0.85e12 : 1.3e12, lds ? 2.1e12 : 1.3e12, 6.0e12, 4e-6, 0.0};
  return part_count(data_tiles(a, 256, 256), data_tiles(a, 128, 128), data_nk_max(a),
                    (int64_t)a.n * a.ho * a.wo * a.co, a.co >= 256, r, 16);
}

size_t data_least_ws_bytes(const DataConvArgs &a) {
  const PartCount pc = sum_order(a);
  return pc.n > 1 ? (size_t)pc.n * a.n * a.ho * a.wo * a.co * sizeof(float) : 0;
}

// Tile and split count of a data convolution, by an estimate of its time (as
// for the kernel gradient below):
//   fixed + max(longest chain of stages * alone, L * mean chain * shared)
// + the output's store, or a split's partials and second launch; L the
// workgroups per CU, rounded up. Fitted to 1500 timings of four tiles at 1 to
// 16 splits over 53 passes (0.01 to 160 GFLOP, 16 to 1024 channels, strided and
// transposed ones among them); mean error 9%, the choice within 1.5% of the
// best timing in the mean. What the tiles trade: the chain of one workgroup's
// stages (small tiles: less of it, more workgroups) against LDS bytes per
// multiply. Best unsplit times: 128 channels over 32768 positions, K 1152: 15.5
// us on 128 x 128 tiles (19.9 on the earlier 4-wave ones in 32-deep stages),
// 16.8 on 64 x 128, 21.3 on 64 x 64; 64 over 6240, K 576: 8.3, 7.4, 6.6; 768
// over 65536, K 768: 97, 136, 160 and 97 on 256 x 256.
struct DataTileCost {
  DataTile tile;
  int32_t tm, tn, bk;
  double fixed;          // us: launch, first loads, drain
  double alone, shared;  // us per 64-deep stage
};
constexpr DataTileCost kDataTiles[] = {
    {DataTile::k256, 256, 256, 32, 6.9, 1.10, 1.45},
    {DataTile::k128, 128, 128, 64, 4.4, 0.63, 0.46},
    {DataTile::k64x128, 64, 128, 64, 4.2, 0.38, 0.33},
    {DataTile::k64, 64, 64, 64, 3.9, 0.29, 0.217},
    {DataTile::k128d32, 128, 128, 32, 4.4, 0.70, 0.52}};
constexpr double kHaloShared = 1.33;      // of 256 x 256 tiles whose input is reused
constexpr double kGen256Shared = 1.95;    // of 256 x 256 tiles across taps
constexpr double kGenFactor = 1.2;        // stages across taps, the other tiles
constexpr double kMnFactor = 1.09;        // weights read transposed
constexpr double kFoldFactor = 1.08;      // parts summed in one workgroup
constexpr double kDataStoreBw = 2.66e6;   // bytes/us of the fp16 output
constexpr double kDataReduce = 3.2;       // us: the second launch of a split
constexpr double kDataPartialBw = 5.3e6;  // bytes/us, 8 per partial element
constexpr int kMaxDataSplit = 16;

// Whether 128 x 128 tiles in ns parts take 32-deep stages (4 waves, a ring of five)
// instead of 64-deep ones (8 waves, two): where a 64-deep stage would straddle taps
// or parts and a 32-deep one does not. With weights read transposed always: 96
// channels, K 3096 over 14756 positions 18.7 us, 22.7 in 64-deep stages; 224, K 2016
// over 143260 163 and 183 (436 such passes 0.93 of the time in the geometric mean,
// 6 of them more than 1.03). With weights read as they lie only for a split into
// parts of 20 and more 64-deep stages, one workgroup to a CU at most: 576 channels,
// K 6656 over 1298 positions 40.8 and 47.0 (55 passes 0.90); with more to a CU they
// take 0.95 to 1.07 of the time, shorter, whole and folded sums 0.97 to 1.13, as 128
// channels, K 864 over 22960 14.6 and 13.4.
static bool deep32(const DataConvArgs &a, const PartCount &so, int ns) {
  if (a.cr % 32 != 0) return false;
  bool straddles = a.cr % 64 != 0;
  for (int i = 0; a.fixed_order && ns > 1 && i < a.nphase; ++i)
    straddles |= part_len(a.ph[i].nr * a.ph[i].ns * a.cr, 32, ns) % 64 != 0;
  const bool mn = a.ldw == 0;
  return straddles &&
         (mn || (ns > 1 && part_len(a.ph[0].nr * a.ph[0].ns * a.cr, 32, so.n) >= 20 * 64 &&
                 data_work(a, 128, 128, 64).tiles * ns <= kCUs));
}

// max_ws_bytes bounds the partials of a split whose order is free.
static DataPlan make_data_plan(const DataConvArgs &a, size_t max_ws_bytes) {
  DataPlan pl{DataTile::k64, 1, 1, 64, 0};
  const int64_t out = (int64_t)a.n * a.ho * a.wo * a.co;
  const bool lds = data_tile_ok(a), fixed = a.fixed_order;
  const PartCount so = fixed || !lds ? sum_order(a) : PartCount{false, 0};
  const bool halo = data_halo_ok(a);
  const int unit = a.cr % 32 == 0 ? 32 : 64;  // of the parts
  if (!lds) {
    pl.tile = so.big ? DataTile::kStaged256 : DataTile::kStaged128;
    pl.nsplit = so.n;
  } else if (fixed && so.big && halo) {
    pl.tile = DataTile::k256;
    pl.nsplit = so.n;
  } else {
    const bool mn = a.ldw == 0;
    double best = 1e30;
    for (const DataTileCost &c : kDataTiles) {
      // 256 x 256: whole-row shapes only where their order is free
      if (c.tm == 256 && (a.co < 256 || (fixed && halo))) continue;
      const PhaseWork pw(a, c.tm, c.tn, c.bk);
      for (int ns = 1; ns <= kMaxDataSplit; ++ns) {
        if (fixed && ns != 1 && ns != so.n) continue;
        if (!fixed && ns > 1 && (size_t)ns * out * sizeof(float) > max_ws_bytes) break;
        if (fixed && ns == 1 && so.n > 1 && c.tm == 256) continue;  // cannot fold
        const DataWork w = pw.split(ns);
        if (w.tiles == 0 || (ns > 1 && !fixed && w.longest * c.bk < 128)) break;
        if (ns > 1 && !fixed && w.tiles * (ns - 1) >= 4 * kCUs) break;  // full already
        bool gen = a.cr % c.bk != 0;
        if (fixed && ns > 1)  // a part may end within a stage
          for (int i = 0; i < a.nphase; ++i)
            gen |= part_len(a.ph[i].nr * a.ph[i].ns * a.cr, unit, ns) % c.bk != 0;
        // 32-deep stages: here against the smallest tiles, in no more parts (and so no
        // more workspace) than those take, else see below
        if (c.tile == DataTile::k128d32 && !(pl.tile == DataTile::k64 &&
                                             ns <= pl.nsplit && mn && deep32(a, so, ns)))
          continue;
        double shared = c.shared, f = mn ? kMnFactor : 1.0;
        if (c.tm == 256)
          shared = halo ? kHaloShared : gen ? kGen256Shared : c.shared;
        else if (gen)
          f *= kGenFactor;
        if (fixed && ns == 1 && so.n > 1) f *= kFoldFactor;
        const double d = c.bk / 64.0, wgs = (double)w.tiles * ns;
        const double per_cu = (double)((w.tiles * ns + kCUs - 1) / kCUs);
        double t = c.fixed +
                   f * d * std::max(w.longest * c.alone, per_cu * (w.stages / wgs) * shared);
        t += ns == 1 ? out * 2.0 / kDataStoreBw
                     : kDataReduce + ns * (double)out * 8.0 / kDataPartialBw;
        if (t < best * 0.98) {  // fewer splits and larger tiles on near ties
          best = t;
          pl.tile = c.tile;
          pl.nsplit = ns;
        }
      }
    }
  }
  if (pl.tile == DataTile::k128 && deep32(a, so, pl.nsplit)) pl.tile = DataTile::k128d32;
  pl.nchunk = fixed ? so.n : pl.nsplit;
  // the kernels' own stages where the order is free
  pl.unit = fixed ? unit : pl.tile == DataTile::k256 || pl.tile == DataTile::k128d32 ? 32 : 64;
  pl.ws_bytes = pl.nsplit > 1 ? (size_t)pl.nsplit * out * sizeof(float) : 0;
  return pl;
}

DataPlan plan_data_conv(const DataConvArgs &a, size_t max_ws_bytes) {
  struct Key {
    DataConvArgs a;
    uint64_t cap;
  };
  static thread_local PlanMemo<Key, DataPlan> memo;
  Key key;  // the shape alone
  memset(&key, 0, sizeof(key));
  memcpy(&key.a, &a, sizeof(a));
  key.a.act = key.a.wgt = key.a.gate = nullptr;
  key.a.out = nullptr;
  key.a.part = nullptr;
  key.a.epi = key.a.nsplit = key.a.nchunk = key.a.unit = 0;
  key.cap = max_ws_bytes;
  auto &e = memo.at(key);
  if (!e.set || memcmp(&e.key, &key, sizeof(key)) != 0) {
    e.plan = make_data_plan(a, max_ws_bytes);
    memcpy(&e.key, &key, sizeof(key));
    e.set = true;
  }
  return e.plan;
}

template <class C, bool WK, bool FAST>
static hipError_t launch_dc(const DataConvArgs &a, hipStream_t st) {
  int maxpix = 0;
  for (int i = 0; i < a.nphase; ++i)
    maxpix = std::max(maxpix, a.n * a.ph[i].mh * a.ph[i].mw);
  dim3 grid((maxpix + C::BN - 1) / C::BN, (a.co + C::BM - 1) / C::BM,
            a.nphase * a.nsplit);
  if (a.nsplit > 1)
    hipLaunchKernelGGL((data_conv_staged_kernel<C, WK, FAST, true>), grid, dim3(C::NT),
                       0, st, a);
  else
    hipLaunchKernelGGL((data_conv_staged_kernel<C, WK, FAST, false>), grid,
                       dim3(C::NT), 0, st, a);
  return hipGetLastError();
}

template <class C>
static hipError_t launch_dc_tile(const DataConvArgs &a, bool w_kmajor,
                                 hipStream_t st) {
  const bool fast = (a.cr % BK) == 0;
  if (w_kmajor)
    return fast ? launch_dc<C, true, true>(a, st)
                : launch_dc<C, true, false>(a, st);
  return fast ? launch_dc<C, false, true>(a, st)
              : launch_dc<C, false, false>(a, st);
}

static hipError_t launch_data_conv_plan(const DataConvArgs &a, DataTile tile, bool w_kmajor,
                                        hipStream_t st) {
  hipError_t e = prof_begin(st);
  if (e != hipSuccess) return e;
  e = tile == DataTile::kStaged256   ? launch_dc_tile<BigCfg>(a, w_kmajor, st)
      : tile == DataTile::kStaged128 ? launch_dc_tile<SmallCfg>(a, w_kmajor, st)
                                     : launch_data_conv_tile(a, tile, w_kmajor, st);
  if (e == hipSuccess) e = prof_end(st);
  if (e != hipSuccess || a.nsplit == 1) return e;
  const int64_t len = (int64_t)a.n * a.ho * a.wo * a.co;
  hipLaunchKernelGGL(split_epilogue_kernel,
                     dim3((unsigned)((len / 4 + 255) / 256)), dim3(256), 0, st,
                     a.part, a.nsplit, len, a.co, a.ldo, a.epi, a.gate, a.out);
  return hipGetLastError();
}

// The call's arguments with the plan's split filled in.
static DataConvArgs planned(const DataConvArgs &a0, const DataPlan &pl) {
  DataConvArgs a = a0;
  a.nsplit = pl.nsplit;
  a.nchunk = pl.nchunk;
  a.unit = pl.unit;
  return a;
}

hipError_t launch_data_conv(const DataConvArgs &a, bool w_kmajor, hipStream_t st,
                            size_t max_ws_bytes) {
  const DataPlan pl = plan_data_conv(a, max_ws_bytes);
  return launch_data_conv_plan(planned(a, pl), pl.tile, w_kmajor, st);
}

// Kernel names as a kernel trace prints them, without namespaces, and with a
// pipeline's configuration (Pipe<...>, K<...>) as its tile: nothing for 256 x 256,
// T for a square, TMxTN else, "/32" after a smaller one in 32-deep stages. F2: by two truth values, F3: by three.
#define F2(K, T)                                  \
  {                                               \
    {K "<" T "false, false>", K "<" T "false, true>"}, \
        {K "<" T "true, false>", K "<" T "true, true>"} \
  }
#define F3(K, T) \
  { F2(K, T "false, "), F2(K, T "true, ") }

const char *data_conv_kernel_name(const DataConvArgs &a0, bool w_kmajor) {
  static const char *halo[2][2] = F2("data_conv_halo_kernel", "");  // weights, split
  static const char *dma[5][2][2] = {  // by DataTile, then the same
      F2("data_conv_dma_kernel", ""), F2("data_conv_dma_kernel", "128, "),
      F2("data_conv_dma_kernel", "64x128, "), F2("data_conv_dma_kernel", "64, "),
      F2("data_conv_dma_kernel", "128/32, ")};
  static const char *gen[5][2][2] = {
      F2("data_conv_gen_kernel", ""), F2("data_conv_gen_kernel", "128, "),
      F2("data_conv_gen_kernel", "64x128, "), F2("data_conv_gen_kernel", "64, "),
      F2("data_conv_gen_kernel", "128/32, ")};
  static const char *fold[5][2][2] = {  // weights, stages across taps
      {{"", ""}, {"", ""}}, F2("data_conv_fold_kernel", "128, "),
      F2("data_conv_fold_kernel", "64x128, "), F2("data_conv_fold_kernel", "64, "),
      F2("data_conv_fold_kernel", "128/32, ")};
  static const char *staged[2][2][2][2] = {  // weights, whole taps per slice, split
      F3("data_conv_staged_kernel", "Cfg<128, 128, 2, 2>, "),
      F3("data_conv_staged_kernel", "Cfg<256, 256, 2, 4>, ")};
  const DataPlan pl = plan_data_conv(a0);
  const DataConvArgs a = planned(a0, pl);
  const bool split = pl.nsplit > 1;
  if (pl.tile == DataTile::kStaged128 || pl.tile == DataTile::kStaged256)
    return staged[pl.tile == DataTile::kStaged256][w_kmajor][a.cr % BK == 0][split];
  if (pl.tile == DataTile::k256 && data_halo_ok(a)) return halo[w_kmajor][split];
  const DataTileMode m = data_tile_mode(a, pl.tile);
  return m.fold ? fold[(int)pl.tile][w_kmajor][m.gen]
                : (m.gen ? gen : dma)[(int)pl.tile][w_kmajor][split];
}

const char *wgrad_kernel_name(const fg_conv_desc &d) {
  int32_t p = (d.h + 2 * d.pad_h - d.r) / d.stride_h + 1;
  int32_t q = (d.w + 2 * d.pad_w - d.s) / d.stride_w + 1;
  static const char *names[5][2] = {  // by WgTile, split
      {"wgrad_dma_kernel<false>", "wgrad_dma_kernel<true>"},
      {"wgrad_dma_kernel<128, false>", "wgrad_dma_kernel<128, true>"},
      {"wgrad_dma_kernel<64, false>", "wgrad_dma_kernel<64, true>"},
      {"wgrad_staged_kernel<Cfg<256, 256, 2, 4>, false>",
       "wgrad_staged_kernel<Cfg<256, 256, 2, 4>, true>"},
      {"wgrad_staged_kernel<Cfg<128, 128, 2, 2>, false>",
       "wgrad_staged_kernel<Cfg<128, 128, 2, 2>, true>"}};
  const WgradPlan pl = plan_wgrad(d, p, q);
  return names[(int)pl.tile][pl.nsplit > 1];
}
#undef F2
#undef F3

// Tile and split count of a kernel gradient, by an estimate of its time:
//   kWgradFixed + stages * max(alone, L * shared) (+ a split's reduction),
// stages of 64 rows in the longest split, L the workgroups per CU (rounded up).
// `alone` is the chain of one workgroup's stages (loads, barrier, transposing
// reads, MFMAs), `shared` what the CU needs per workgroup stage when several
// interleave. Fitted to 900 timings of the three tiles at 1 to 256 splits over
// 25 shapes (0.01 to 310 GFLOP, 16 to 1024 channels, 1x1 to 4x4 kernels); mean
// error 7.5%, the choice within 4% of the best timing in the mean. The tiles
// trade LDS traffic for workgroups: 512 x 4608 x 65536 (K x RSC x positions)
// takes 340 us on 256 x 256 tiles, 427 on 128 and 577 on 64; 512 x 2376 x 1024
// 29, 15 and 11 us.
struct WgradTileCost {
  WgTile tile;
  int32_t t;
  double alone, shared;  // us per 64-row stage
};
constexpr WgradTileCost kWgradTiles[] = {{WgTile::k256, 256, 1.08, 1.39},
                                         {WgTile::k128, 128, 0.65, 0.52},
                                         {WgTile::k64, 64, 0.33, 0.22}};
constexpr double kWgradFixed = 4.4;       // us: launch, first loads, tile store
constexpr double kWgradReduce = 2.8;      // us: the reduction's launch
constexpr double kWgradPartialBw = 5.6e6; // bytes/us, 8 per partial element
constexpr int kMaxWgradSplit = 256;

// The register-staged kernels (tensors beyond a buffer resource): their
// 128 x 128 tiles everywhere but where both counts fill a 256 x 256 one.
static WgradPlan plan_staged(int64_t rsc, int64_t k, int64_t mtot, int max_split) {
  const bool big = rsc >= 256 && k >= 256;
  const int64_t t = big ? 256 : 128;
  const int64_t tiles = ((rsc + t - 1) / t) * ((k + t - 1) / t);
  const int64_t want = (kCUs + tiles - 1) / tiles;
  WgradPlan pl;
  pl.tile = big ? WgTile::kStaged256 : WgTile::kStaged128;
  pl.nsplit = (int32_t)std::max<int64_t>(
      1, std::min<int64_t>(std::min<int64_t>(want, max_split), mtot / (4 * BK)));
  return pl;
}

// all_stages: a few tiles may split into as many parts as there are stages.
static WgradPlan make_wgrad_plan(const fg_conv_desc &d, int32_t p, int32_t q,
                                 size_t max_ws_bytes, bool all_stages = true) {
  const int64_t rsc = (int64_t)d.r * d.s * d.c, k = d.k;
  const int64_t mtot = (int64_t)d.n * p * q;
  const size_t cap = max_ws_bytes / ((size_t)k * rsc * sizeof(float));
  const int max_split = cap >= (size_t)kMaxWgradSplit ? kMaxWgradSplit
                                                      : (cap < 2 ? 1 : (int)cap);
  WgradArgs wa;
  wa.n = d.n; wa.h = d.h; wa.w = d.w; wa.c = d.c; wa.k = d.k;
  wa.ldx = d.x_ld ? d.x_ld : d.c;
  wa.mtot = (int32_t)mtot;
  const int64_t nk = (mtot + BK - 1) / BK;  // 64-row stages
  WgradPlan pl;
  if (!wgrad_tile_ok(wa)) {
    pl = plan_staged(rsc, k, mtot, max_split);
  } else {
    double best = 1e30;
    for (const WgradTileCost &c : kWgradTiles) {
      if (c.t == 256 && (rsc < 256 || k < 256)) continue;
      const int64_t tiles = ((rsc + c.t - 1) / c.t) * ((k + c.t - 1) / c.t);
      // no split, a few, and as many as fill the CUs 1 to 6 times; where even once,
      // on the smallest tiles, is more than there are stages, or than a bound on
      // the workspace leaves, as many as those (64 x 64 outputs over 14432
      // positions, 226 stages on one tile: 24.4 us in 4 parts, 8.4 in 226). From 36
      // stages on, where both take 8.2 us: with 20 7.0 and 8.3, with 64 10.7 and 8.0.
      int64_t cand[10] = {1, 2, 3, 4};
      for (int l = 1; l <= 6; ++l) cand[3 + l] = l * kCUs / tiles;
      const int64_t most =
          all_stages && nk >= 36 ? std::min<int64_t>(nk, max_split) : max_split;
      int64_t last = 0;
      for (int64_t ns : cand) {
        if (c.tile == WgTile::k64 && last <= 4) ns = std::min(ns, most);
        if (ns <= last || ns > max_split || ns > nk) continue;
        last = ns;
        const int64_t st = (nk + ns - 1) / ns, wgs = tiles * ((nk + st - 1) / st);
        const int64_t per_cu = (wgs + kCUs - 1) / kCUs;
        double t = kWgradFixed + st * std::max(c.alone, per_cu * c.shared);
        if (ns > 1) t += kWgradReduce + ns * (double)(k * rsc) * 8.0 / kWgradPartialBw;
        if (t < best * 0.98) {  // fewer splits and larger tiles on near ties
          best = t;
          pl.tile = c.tile;
          pl.nsplit = (int32_t)ns;
        }
      }
    }
  }
  int64_t chunk = (mtot + pl.nsplit - 1) / pl.nsplit;
  chunk = (chunk + BK - 1) / BK * BK;
  const int64_t ns = (mtot + chunk - 1) / chunk;
  pl.nsplit = (int32_t)ns;
  pl.mchunk = (int32_t)chunk;
  pl.ws_bytes = ns > 1 ? (size_t)ns * k * rsc * sizeof(float) : 0;
  return pl;
}

// The size below the plan's own that a kernel gradient given `has` bytes keeps to:
// that of the split the earlier kernels took (their rates fitted to the network's
// layers; up to 16 parts, or 256 where the gradient has no 256 x 256 tile), or, if
// the call brings less, that of the plan without splits into all stages where
// that is smaller. The query gave both, so programs may keep either.
size_t wgrad_least_ws_bytes(const fg_conv_desc &d, int32_t p, int32_t q, size_t has) {
  constexpr PartRates kRates{6.35e12, 1.3e12, 1.3e12, 4.05e12, 6.3e-6, 4.2e-6};
  const int64_t rsc = (int64_t)d.r * d.s * d.c, k = d.k, mtot = (int64_t)d.n * p * q;
  const bool big = rsc >= 256 && k >= 256;
  auto tiles = [&](int64_t t) { return ((rsc + t - 1) / t) * ((k + t - 1) / t); };
  const PartCount pc = part_count(tiles(256), tiles(128), (mtot + BK - 1) / BK, k * rsc, big,
                                  kRates, big ? 16 : kMaxWgradSplit);
  const int64_t chunk = ((mtot + pc.n - 1) / pc.n + BK - 1) / BK * BK;
  const int64_t ns = (mtot + chunk - 1) / chunk;
  const size_t earlier = ns > 1 ? (size_t)ns * k * rsc * sizeof(float) : 0;
  return has >= earlier
             ? earlier
             : std::min(earlier, make_wgrad_plan(d, p, q, SIZE_MAX, false).ws_bytes);
}

// max_ws_bytes bounds the fp32 partials of a split (and so the split count);
// a bound that the plan without one keeps does not change the plan.
WgradPlan plan_wgrad(const fg_conv_desc &d, int32_t p, int32_t q,
                     size_t max_ws_bytes) {
  if (max_ws_bytes != SIZE_MAX) {
    const WgradPlan pl = plan_wgrad(d, p, q, SIZE_MAX);
    if (pl.ws_bytes <= max_ws_bytes) return pl;
  }
  struct Key {
    fg_conv_desc d;
    int32_t capped;
    uint64_t cap;
  };
  static thread_local PlanMemo<Key, WgradPlan> memo;
  Key key;
  memset(&key, 0, sizeof(key));
  key.d = d;
  key.capped = max_ws_bytes != SIZE_MAX;
  key.cap = max_ws_bytes;
  auto &e = memo.at(key);
  if (!e.set || memcmp(&e.key, &key, sizeof(key)) != 0) {
    e.plan = make_wgrad_plan(d, p, q, max_ws_bytes);
    memcpy(&e.key, &key, sizeof(key));
    e.set = true;
  }
  return e.plan;
}

template <class C>
static hipError_t launch_staged_wgrad(const WgradArgs &a, hipStream_t st) {
  dim3 grid((a.r * a.s * a.c + C::BM - 1) / C::BM, (a.k + C::BN - 1) / C::BN, a.nsplit);
  if (a.nsplit > 1)
    hipLaunchKernelGGL((wgrad_staged_kernel<C, true>), grid, dim3(C::NT), 0, st, a);
  else
    hipLaunchKernelGGL((wgrad_staged_kernel<C, false>), grid, dim3(C::NT), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_wgrad(const WgradArgs &a, WgTile tile, hipStream_t st) {
  hipError_t e = prof_begin(st);
  if (e != hipSuccess) return e;
  switch (tile) {
    case WgTile::kStaged256: e = launch_staged_wgrad<BigCfg>(a, st); break;
    case WgTile::kStaged128: e = launch_staged_wgrad<SmallCfg>(a, st); break;
    default: e = launch_wgrad_tile(a, tile, st);
  }
  if (e == hipSuccess) e = prof_end(st);
  if (e != hipSuccess || a.nsplit == 1) return e;
  const int64_t len = (int64_t)a.k * a.r * a.s * a.c;
  if (a.nsplit > kMaxSerialSplit) {
    hipLaunchKernelGGL(split_reduce_multi_kernel, dim3((unsigned)((len + 63) / 64)),
                       dim3(256), 0, st, a.part, a.nsplit, len, a.dw, a.flag);
    return hipGetLastError();
  }
  dim3 g2((unsigned)((len / 4 + 255) / 256));
  hipLaunchKernelGGL(split_reduce_kernel, g2, dim3(256), 0, st, a.part,
                     a.nsplit, len, a.dw, a.flag);
  return hipGetLastError();
}

static int pow2_at_least(int v) {
  int p = 1;
  while (p < v) p <<= 1;
  return p;
}

hipError_t launch_head_fwd(const uint16_t *x, const uint16_t *w, uint16_t *y,
                           int64_t npix, int32_t c, int32_t epi,
                           const uint16_t *gate, hipStream_t st) {
  int L = pow2_at_least(c / 8);
  if (L > 64) L = 64;
  int logL = 0;
  while ((1 << logL) < L) ++logL;
  int64_t waves = (npix * L + 63) / 64;
  int64_t blocks = (waves + 3) / 4;
  if (blocks > 4096) blocks = 4096;
  hipError_t e = prof_begin(st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(head_fwd_kernel, dim3((unsigned)blocks), dim3(256), 0, st,
                     x, w, y, npix, c, L, logL, epi, gate);
  e = hipGetLastError();
  return e == hipSuccess ? prof_end(st) : e;
}

hipError_t launch_head_bwd_data(const uint16_t *dy, const uint16_t *w,
                                uint16_t *dx, int64_t npix, int32_t c,
                                int32_t epi, const uint16_t *gate,
                                hipStream_t st) {
  int64_t n = npix * (c / 8);
  hipError_t e = prof_begin(st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(head_bwd_data_kernel, dim3((unsigned)((n + 255) / 256)),
                     dim3(256), 0, st, dy, w, dx, npix, c, epi, gate);
  e = hipGetLastError();
  return e == hipSuccess ? prof_end(st) : e;
}

static int64_t head_wgrad_blocks(int64_t npix) {
  // about 256 positions per workgroup, four workgroups per CU on the
  // full-size head
  int64_t b = (npix + 255) / 256;
  return b < 1 ? 1 : (b > 2048 ? 2048 : b);
}

size_t head_wgrad_ws_bytes(const fg_conv_desc &d) {
  int64_t npix = (int64_t)d.n * d.h * d.w;
  return (size_t)head_wgrad_blocks(npix) * d.c * sizeof(float);
}

hipError_t launch_head_wgrad(const uint16_t *x, const uint16_t *dy,
                             uint16_t *dw, int64_t npix, int32_t c, float *ws,
                             int32_t *flag, hipStream_t st) {
  int64_t nb = head_wgrad_blocks(npix);
  int64_t chunk = (npix + nb - 1) / nb;
  hipError_t e = prof_begin(st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(head_wgrad_kernel, dim3((unsigned)nb),
                     dim3(kHeadWgradThreads), 0, st, x, dy, npix, c, chunk,
                     ws);
  e = hipGetLastError();
  if (e == hipSuccess) e = prof_end(st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(split_reduce_wide_kernel, dim3((unsigned)(c / 4)),
                     dim3(256), 0, st, ws, (int)nb, (int64_t)c, dw, flag);
  return hipGetLastError();
}

}  // namespace fg
