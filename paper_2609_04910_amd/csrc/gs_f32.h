// gs_f32.h -- the fp32-accuracy tier of the forward sum (Eq. 1) for fp32
// points and a single value channel (the single-precision setting of App.
// A.2: C = 1).
//
// Scores.  Each fp32 point set is scaled by an exact power of two 2^e (its
// largest magnitude into [2^14, 2^15)) and split into two fp16 numbers,
// x 2^e = hi + lo with hi = fp16(x 2^e) and lo = fp16(x 2^e - hi) (the
// difference is exact in fp32), so hi + lo carries 22 significant bits and
// no part leaves the fp16 range.  q.k is then three fp16 MFMAs per operand
// chunk, lo.hi + hi.lo + hi.hi (lo.lo, below 2^-22 of the product, is
// dropped), accumulated in fp32 on top of the key bias, in scaled units
// 2^(eq + ek); the exponent fma folds the scale back into tau'.
//
// Values.  As in the fp16 tier, |v_n| enters the exponent (log2 |v_n 2^ev| in
// the key bias, max |v 2^ev| in [0.5, 1)), so exp2 yields Phi |v_n| in fp32
// directly.  Nothing is rounded to fp16 after the exponent: the signed sum
// sum_n sign(v_n) Phi |v_n| is accumulated in fp32 on the vector unit, with
// the signs read as +-1.0f from the step scalars in the row order of the
// score tile, in three levels: the eight terms of a lane in one step, the
// steps of a block of kAccBlock steps, and the blocks, added with Kahan's
// compensation (a flat fp32 sum over N/32 steps would lose about
// 2^-24 sqrt(N/32) / 3 of the sum).  So no row-maximum shift is needed: the
// only values lost are those below the fp32 normal range.
#pragma once

#include "gs_kernels.h"
#include "gs_prep.h"

namespace gs {

// Key steps per block of the blocked, compensated row sum.
constexpr int kAccBlock = 16;

// Queries per wave (16-row tiles) of the fp32-tier forward kernel.
constexpr int f32_qt(int DP) { return DP >= 8 ? 1 : 8 / DP; }

// s_m = sum_n Phi(q_m, k_n) v_n for fp32 points, C = 1 (see the top of this
// file).  qh / ql, kh / kl: split copies (RT layout); nhq: query half norms;
// scal: key_scalars32; slots: [0] max |v|, [2] max |q|, [3] max |k| (the
// key slot is [2] when q and k are the same array: kslot selects it).
// Key steps are split over grid.y as in k_fwd (partials at part_stride);
// problems of a batch on grid.z (strides of bz).
template <int DP>
__global__ __launch_bounds__(kBlockThreads) void k_fwd32(
    const uint4* __restrict__ qh, const uint4* __restrict__ ql, const float* __restrict__ nhq,
    const uint4* __restrict__ kh, const uint4* __restrict__ kl, const float* __restrict__ scal,
    const uint32_t* __restrict__ slots, int kslot, float tau2, int64_t M, int steps_total,
    int steps_per_split, float* __restrict__ out, int64_t part_stride, Bz bz) {
  qh = zoff(qh, bz.ws);
  ql = zoff(ql, bz.ws);
  nhq = zoff(nhq, bz.ws);
  kh = zoff(kh, bz.ws);
  kl = zoff(kl, bz.ws);
  scal = zoff(scal, bz.ws);
  slots = zoff(slots, bz.ws);
  out = zoff(out, bz.out);
  constexpr int QT = f32_qt(DP);
  constexpr int KCH = 2 * DP;    // 1-KiB chunks of one key copy per step
  constexpr int NCH = 2 * KCH;   // hi and lo
  constexpr int STAGE = NCH * 1024 + kScalarFloats * 4;
  constexpr int NS = ring_stages(STAGE, NCH + 1);
  __shared__ __attribute__((aligned(1024))) char lds[NS * STAGE];

  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t dlane = dma_lane_offset(lane);
  const int wave = threadIdx.x / kWave;
  const int j = lane & 15, g = lane >> 4;
  const int64_t q0 = ((int64_t)blockIdx.x * kWavesPerBlock + wave) * (16 * QT);
  const int s_begin = blockIdx.y * steps_per_split;
  const int s_end = min(steps_total, s_begin + steps_per_split);
  out += blockIdx.y * part_stride;

  const bool mine = g == wave;
  const uint32_t nsteps = (uint32_t)max(0, s_end - s_begin);
  const auto rkh = make_rsrc(reinterpret_cast<const char*>(kh) + (int64_t)s_begin * KCH * 1024,
                             nsteps * KCH * 1024);
  const auto rkl = make_rsrc(reinterpret_cast<const char*>(kl) + (int64_t)s_begin * KCH * 1024,
                             nsteps * KCH * 1024);
  const auto rsc = make_rsrc(scal + (int64_t)s_begin * kScalarFloats, nsteps * kScalarFloats * 4);
  const uint32_t lds0 = lds_address(lds);
  auto issue = [&](int s, int stage) {
    if (!mine) return;
    const uint32_t base = lds0 + stage * STAGE;
    const uint32_t ls = (uint32_t)(s - s_begin);
#pragma unroll
    for (int c = 0; c < KCH; ++c) dma_x4(rkh, (ls * KCH + c) * 1024, base + c * 1024, dlane);
#pragma unroll
    for (int c = 0; c < KCH; ++c) dma_x4(rkl, (ls * KCH + c) * 1024, base + (KCH + c) * 1024, dlane);
    dma_x1(rsc, ls * kScalarFloats * 4, base + NCH * 1024, 4 * lane);
  };

  const int es = scale_exponent(slots[2]) + scale_exponent(slots[kslot]) + 2 * kSplitHeadroom;
  const float tau2s = ldexpf(tau2, -es);
  uint4 qhr[QT][DP], qlr[QT][DP];
  float bq[QT], A[QT], Ac[QT], blk[QT];  // sum of blocks, its compensation, current block
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    load_k_tile<DP>(qh, q0 / 16 + qt, j, g, qhr[qt]);
    load_k_tile<DP>(ql, q0 / 16 + qt, j, g, qlr[qt]);
    bq[qt] = tau2 * nhq[q0 + 16 * qt + j];
    A[qt] = Ac[qt] = blk[qt] = 0.0f;
  }
  settle(qhr);
  settle(qlr);
  settle(bq);
  // Kahan: A + Ac carries the sum of the finished blocks
  auto close_block = [&]() {
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
      const float y = blk[qt] - Ac[qt];
      const float t = A[qt] + y;
      Ac[qt] = (t - A[qt]) - y;
      A[qt] = t;
      blk[qt] = 0.0f;
    }
  };
  int in_block = 0;

  auto compute = [&](int stage) {
    const char* base = lds + stage * STAGE;
    const uint4* khb = reinterpret_cast<const uint4*>(base);
    const uint4* klb = reinterpret_cast<const uint4*>(base + KCH * 1024);
    const float* sc = reinterpret_cast<const float*>(base + NCH * 1024);
    float part[QT];
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) part[qt] = 0.0f;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      const floatx4 cin = *reinterpret_cast<const floatx4*>(sc + 16 * kt + 4 * g);
      const floatx4 sg = *reinterpret_cast<const floatx4*>(sc + 32 + 16 * kt + 4 * g);
      uint4 khr[DP], klr[DP];
      load_k_tile_lds<DP>(khb, kt, j, g, khr);
      load_k_tile_lds<DP>(klb, kt, j, g, klr);
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) {
        floatx4 acc = cin;
#pragma unroll
        for (int dc = 0; dc < DP; ++dc) {
          acc = mfma_f16(klr[dc], qhr[qt][dc], acc);
          acc = mfma_f16(khr[dc], qlr[qt][dc], acc);
        }
#pragma unroll
        for (int dc = 0; dc < DP; ++dc) acc = mfma_f16(khr[dc], qhr[qt][dc], acc);
#pragma unroll
        for (int r = 0; r < 4; ++r) part[qt] = fmaf(exp2_clamped(fmaf(acc[r], tau2s, bq[qt])), sg[r], part[qt]);
      }
    }
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) blk[qt] += part[qt];
    if (++in_block == kAccBlock) {
      close_block();
      in_block = 0;
    }
  };
  key_stream<NS, NCH + 1>(s_begin, s_end, issue, compute);
  close_block();

  // the four row groups of the tile hold disjoint key subsets: add them in a
  // fixed order (every lane gets the same value)
  const int ev = scale_exponent(slots[0]) - 1;
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    float x = A[qt] - Ac[qt];
    x += __shfl_xor(x, 16, kWave);
    x += __shfl_xor(x, 32, kWave);
    const int64_t m = q0 + 16 * qt + j;
    if (g == 0 && m < M) out[m] = ldexpf(x, -ev);
  }
}

}  // namespace gs

namespace gs {

// Several value channels (fp32 points, C > 1).  One pass over the wave's keys
// through the LDS ring.  P = 2^(x - off) is evaluated in fp32, split into fp16
// hi + lo 2^-kSplitLow (hi = P rounded, lo = (P - hi) 2^kSplitLow rounded) and
// contracted with the values, split the same way (v 2^ev = vh + vl 2^-kSplitLow):
// vh.Ph into a block accumulator that is added to the running sum with Kahan's
// compensation every kAccBlock steps, vl.Ph + vh.Pl into a second accumulator
// in units of 2^-kSplitLow.
//
// off is a running offset per row: the row's largest exponent, rounded down to
// a whole number, at the last step in which some exponent of the row exceeded
// the offset by more than kPRaise.  So P stays below 2^5; hi and lo together
// resolve 2^-36 of the row maximum or better, as with an exact maximum; the
// exponents that matter are small numbers, which fp32 rounds least; and whole
// offsets make every rescaling of the accumulators exact.  (A first pass over
// all keys for the exact maxima computed every split score, three MFMAs per
// operand pair, a second time: B = 4, M = N = 16384, D = C = 32
// 650 -> 473 us, D = 100, C = 5 657 -> 296 us, M = N = 16384; error against 64
// bits 3.4e-7 -> 1.8e-7, from the smaller exponents.)
constexpr float kPRaise = 4.0f;
// Queries per wave (16-row tiles) of the several-channel kernel.
constexpr int f32c_qt(int DP, int CT) { return (DP >= 4 || CT >= 4) ? 1 : 2; }
// Channels per launch of the several-channel kernel (16 * CT at most).
constexpr int kF32MaxChannels = 64;

// vh / vl: split values in KS layout, already advanced to this launch's first
// channel; vstep: bytes per key step of those arrays (R * 64); cw: channels
// of this launch; C: row stride of out (the problem's channel count); out
// already advanced to the first channel.
template <int DP, int CT>
__global__ __launch_bounds__(kBlockThreads) void k_fwd32c(
    const uint4* __restrict__ qh, const uint4* __restrict__ ql, const float* __restrict__ nhq,
    const uint4* __restrict__ kh, const uint4* __restrict__ kl, const float* __restrict__ scal,
    const uint4* __restrict__ vh, const uint4* __restrict__ vl, int vstep,
    const uint32_t* __restrict__ slots, int kslot, float tau2, int64_t M, int C, int cw, int steps_total,
    int steps_per_split, float* __restrict__ out, int64_t part_stride, Bz bz) {
  qh = zoff(qh, bz.ws);
  ql = zoff(ql, bz.ws);
  nhq = zoff(nhq, bz.ws);
  kh = zoff(kh, bz.ws);
  kl = zoff(kl, bz.ws);
  scal = zoff(scal, bz.ws);
  vh = zoff(vh, bz.ws);
  vl = zoff(vl, bz.ws);
  slots = zoff(slots, bz.ws);
  out = zoff(out, bz.out);
  constexpr int QT = f32c_qt(DP, CT);
  constexpr int KCH = 2 * DP;           // 1-KiB chunks of one key copy per step
  constexpr int NCH = 2 * KCH + 2 * CT; // key hi, lo, value hi, lo
  constexpr int STAGE = NCH * 1024 + kScalarFloats * 4;
  constexpr int NS = ring_stages(STAGE, NCH + 1);
  __shared__ __attribute__((aligned(1024))) char lds[NS * STAGE];

  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t dlane = dma_lane_offset(lane);
  const int wave = threadIdx.x / kWave;
  const int j = lane & 15, g = lane >> 4;
  const int64_t q0 = ((int64_t)blockIdx.x * kWavesPerBlock + wave) * (16 * QT);
  const int s_begin = blockIdx.y * steps_per_split;
  const int s_end = min(steps_total, s_begin + steps_per_split);
  out += blockIdx.y * part_stride;

  const bool mine = g == wave;
  const uint32_t nsteps = (uint32_t)max(0, s_end - s_begin);
  const auto rkh = make_rsrc(reinterpret_cast<const char*>(kh) + (int64_t)s_begin * KCH * 1024,
                             nsteps * KCH * 1024);
  const auto rkl = make_rsrc(reinterpret_cast<const char*>(kl) + (int64_t)s_begin * KCH * 1024,
                             nsteps * KCH * 1024);
  const auto rvh = make_rsrc(reinterpret_cast<const char*>(vh) + (int64_t)s_begin * vstep,
                             nsteps * (uint32_t)vstep);
  const auto rvl = make_rsrc(reinterpret_cast<const char*>(vl) + (int64_t)s_begin * vstep,
                             nsteps * (uint32_t)vstep);
  const auto rsc = make_rsrc(scal + (int64_t)s_begin * kScalarFloats, nsteps * kScalarFloats * 4);
  const uint32_t lds0 = lds_address(lds);
  auto issue = [&](int s, int stage) {
    if (!mine) return;
    const uint32_t base = lds0 + stage * STAGE;
    const uint32_t ls = (uint32_t)(s - s_begin);
#pragma unroll
    for (int c = 0; c < KCH; ++c) dma_x4(rkh, (ls * KCH + c) * 1024, base + c * 1024, dlane);
#pragma unroll
    for (int c = 0; c < KCH; ++c) dma_x4(rkl, (ls * KCH + c) * 1024, base + (KCH + c) * 1024, dlane);
#pragma unroll
    for (int c = 0; c < CT; ++c)
      dma_x4(rvh, ls * (uint32_t)vstep + c * 1024, base + (2 * KCH + c) * 1024, dlane);
#pragma unroll
    for (int c = 0; c < CT; ++c)
      dma_x4(rvl, ls * (uint32_t)vstep + c * 1024, base + (2 * KCH + CT + c) * 1024, dlane);
    dma_x1(rsc, ls * kScalarFloats * 4, base + NCH * 1024, 4 * lane);
  };

  const int es = scale_exponent(slots[2]) + scale_exponent(slots[kslot]) + 2 * kSplitHeadroom;
  const float tau2s = ldexpf(tau2, -es);
  uint4 qhr[QT][DP], qlr[QT][DP];
  float bq[QT];
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    load_k_tile<DP>(qh, q0 / 16 + qt, j, g, qhr[qt]);
    load_k_tile<DP>(ql, q0 / 16 + qt, j, g, qlr[qt]);
    bq[qt] = tau2 * nhq[q0 + 16 * qt + j];
  }
  settle(qhr);
  settle(qlr);
  settle(bq);
  auto score = [&](const uint4 (&khr)[DP], const uint4 (&klr)[DP], int qt, floatx4 cin) {
    floatx4 acc = cin;
#pragma unroll
    for (int dc = 0; dc < DP; ++dc) {
      acc = mfma_f16(klr[dc], qhr[qt][dc], acc);
      acc = mfma_f16(khr[dc], qlr[qt][dc], acc);
    }
#pragma unroll
    for (int dc = 0; dc < DP; ++dc) acc = mfma_f16(khr[dc], qhr[qt][dc], acc);
    return acc;
  };

  // offsets, and the constant term of the exponent relative to them
  float off[QT], be[QT];
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    off[qt] = -__builtin_inff();
    be[qt] = __builtin_inff();
  }
  floatx4 O1[QT][CT], O2[QT][CT], T[QT][CT], Tc[QT][CT];
#pragma unroll
  for (int qt = 0; qt < QT; ++qt)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      O1[qt][ct] = O2[qt][ct] = T[qt][ct] = Tc[qt][ct] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    }
  auto close_block = [&]() {
#pragma unroll
    for (int qt = 0; qt < QT; ++qt)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float y = O1[qt][ct][r] - Tc[qt][ct][r];
          const float t = T[qt][ct][r] + y;
          Tc[qt][ct][r] = (t - T[qt][ct][r]) - y;
          T[qt][ct][r] = t;
          O1[qt][ct][r] = 0.0f;
        }
  };
  int in_block = 0;
  auto compute = [&](int stage) {
    const char* base = lds + stage * STAGE;
    const uint4* khb = reinterpret_cast<const uint4*>(base);
    const uint4* klb = reinterpret_cast<const uint4*>(base + KCH * 1024);
    const uint4* vhb = reinterpret_cast<const uint4*>(base + 2 * KCH * 1024);
    const uint4* vlb = reinterpret_cast<const uint4*>(base + (2 * KCH + CT) * 1024);
    const float* sc = reinterpret_cast<const float*>(base + NCH * 1024);
    uint4 vhr[CT], vlr[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      vhr[ct] = vhb[(16 * ct + j) * 4 + lds_col(j, g)];
      vlr[ct] = vlb[(16 * ct + j) * 4 + lds_col(j, g)];
    }
    floatx4 sc2[QT][2];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      const floatx4 cin = *reinterpret_cast<const floatx4*>(sc + 16 * kt + 4 * g);
      uint4 khr[DP], klr[DP];
      load_k_tile_lds<DP>(khb, kt, j, g, khr);
      load_k_tile_lds<DP>(klb, kt, j, g, klr);
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) sc2[qt][kt] = score(khr, klr, qt, cin);
    }
    float p[QT][2][4];
    float ymax = -__builtin_inff();
    auto exponents = [&](int qt) {
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 4; ++r) p[qt][kt][r] = fmaf(sc2[qt][kt][r], tau2s, be[qt]);
    };
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
      exponents(qt);
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
        ymax = max_into(ymax, floatx4{p[qt][kt][0], p[qt][kt][1], p[qt][kt][2], p[qt][kt][3]});
    }
    if (__any(ymax > kPRaise)) {
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) {
        float raw = -__builtin_inff();
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) raw = max_into(raw, sc2[qt][kt]);
        // (finite also where every exponent so far is -inf)
        const float nw = fmaxf(fmaxf(off[qt], -3.0e38f), floorf(fmaf(wave_max_over_g(raw), tau2s, bq[qt])));
        const float f = nw > off[qt] ? exp2f(off[qt] - nw) : 1.0f;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            O1[qt][ct][r] *= f;
            O2[qt][ct][r] *= f;
            T[qt][ct][r] *= f;
            Tc[qt][ct][r] *= f;
          }
        off[qt] = nw;
        be[qt] = bq[qt] - nw;
        exponents(qt);
      }
    }
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 4; ++r) p[qt][kt][r] = __builtin_amdgcn_exp2f(p[qt][kt][r]);
      const uint4 bh = pack_tile_pair(p[qt]);
      const uint32_t hw[4] = {bh.x, bh.y, bh.z, bh.w};
      float lo[2][4];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const halfx2 h2 = __builtin_bit_cast(halfx2, hw[e >> 1]);
        // (exact: both products are, and the difference)
        lo[e >> 2][e & 3] = fmaf((float)h2[e & 1], -kSplitLowScale, p[qt][e >> 2][e & 3] * kSplitLowScale);
      }
      const uint4 bl = pack_tile_pair(lo);
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        O1[qt][ct] = mfma_f16(vhr[ct], bh, O1[qt][ct]);
        O2[qt][ct] = mfma_f16(vlr[ct], bh, O2[qt][ct]);
        O2[qt][ct] = mfma_f16(vhr[ct], bl, O2[qt][ct]);
      }
    }
    if (++in_block == kAccBlock) {
      close_block();
      in_block = 0;
    }
  };
  key_stream<NS, NCH + 1>(s_begin, s_end, issue, compute);
  close_block();

  const int ev = scale_exponent(slots[0]);
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    const int64_t m = q0 + 16 * qt + j;
    if (m >= M) continue;
    // 2^(off - ev) through ldexp (no denormal factor; offsets beyond
    // any result's range, and that of an empty key range, bounded)
    const int e = (int)fmaxf(off[qt], -1.0e6f) - ev;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int c = 16 * ct + 4 * g + r;
        const float x = fmaf(O2[qt][ct][r], 1.0f / kSplitLowScale, T[qt][ct][r] - Tc[qt][ct][r]);
        if (c < cw) out[m * C + c] = ldexpf(x, e);
      }
  }
}

}  // namespace gs
