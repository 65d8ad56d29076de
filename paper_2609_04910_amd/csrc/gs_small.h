// gs_small.h -- small problems in one launch.
//
// k_small computes a whole call (the sum, the gradients with respect to one
// side, or both sides at once) from the caller's arrays: no prepared copies,
// no workspace, no split partials.  A small call is bound by launches -- each
// costs about 4 us of host time and 3 - 5 us of a dependent GPU queue, against
// a few microseconds of arithmetic -- so the work that the prepared path
// shares between workgroups (row norms, fp16 copies, transposes) is done again
// by every workgroup here, next to the loads it needs anyway.
//
// A workgroup is eight waves (sixteen where registers allow) that own the same
// 16 queries and take every eighth key step (32 keys) each: even a problem of
// a thousand points then keeps 63 CUs with eight waves busy.  A wave loads
// the 32 key rows as the A operands of the score MFMAs straight from the
// caller's row-major array (16-byte loads at element alignment), forms their
// half norms in fp64, and, for the contractions over keys, stores the same
// registers to its own piece of LDS and reads them back transposed
// (ds_read_b64_tr_b16); the next step's rows are loaded before the current
// step is computed.  At the end the waves' partial results are added in wave
// order through LDS, so results are reproducible bit for bit.
//
// Bound by instruction issue and latency, not by memory: per step the norms,
// conversions and masks take several times the prepared kernels' instructions,
// which is why larger calls prepare.  What that share cost and no longer does
// (sum over 4096 x 4096, D = 16, C = 1, the kernel alone): branches on the
// values' type per element and on a divergent wave index 27 -> 18 us; masks as
// scalar pairs and element-by-element loads at the arrays' ends 18 -> 13 us.
// Norms in fp32 would save 5 % and lose precision; key steps started at
// different places by different workgroups (so that they do not wait for the
// same cold lines) measured the same.
//
// Range: kernel values carry a running offset per row and wave (the row's
// largest exponent, rounded down, when it last grew by more than kSmallRaise), so no row
// check is needed: the values of a row that matter are within fp16's normal
// range whatever the row maximum is.  In the single-channel gradient the
// exponent is that of Phi |v| (log2 |v| is added to it, the sign goes onto the
// kernel value), so that this holds for unequal weights too: with an offset of
// Phi alone and v scaled by the largest |v| a row whose near neighbours weigh
// little had subnormal products (log-normal weights of sigma 4, N = 1000,
// D = 8: errors of 1.7e-2 of sum Phi |v|, now 5e-4; N = 1000, D = 3 as a flow 18.1 / 18.3 us).  The
// single-channel sum is formed in fp32 on the vector unit (no fp16 value
// anywhere) and needs no offset.
#pragma once

#include "gs_kernels.h"
#include "gs_prep.h"

namespace gs {

// Offsets move when an exponent exceeds the current one by more than this:
// kernel values stay at or below 2^6 and their products with w = <g, v> (less
// than 4 C <= 2^8 for the at most 64 channels here, after scaling) below
// fp16's largest number.
constexpr float kSmallRaise = 6.0f;
constexpr float kSmallCap = 64.0f;  // 2^kSmallRaise

enum SmallKind : int {
  kSmallFwd,    // s
  kSmallGrad,   // dq and, if wanted, s
  kSmallSvgd    // sum_n Phi score_n - tau sum_n Phi (k_n - q_m)
};

// One direction: rows q against keys k with values v (N x C), upstream
// gradients g (M x C) of the rows; NULL outputs are not written, g = NULL is
// a unit gradient.  b*: byte strides between problems of a batch.
struct SmallSide {
  const uint16_t *q, *k;
  const void *v, *g;
  float *out_s, *out_d;
  int64_t M, N;
  int64_t bq, bk, bv, bg, bs, bd;
  int v_dtype, g_dtype;
};

// Eight consecutive elements of a row as loaded (fp32 fills both halves, 16-bit
// types the first; the second is then whatever follows), at element alignment.
struct Raw8 {
  uint4 a, b;
};
typedef uint32_t u32x4_e2 __attribute__((ext_vector_type(4), aligned(2)));
__device__ __forceinline__ uint4 load16(const char* __restrict__ p) {
  const u32x4_e2 u = *reinterpret_cast<const u32x4_e2*>(p);
  return uint4{u.x, u.y, u.z, u.w};
}

// Elements idx .. idx+7; the caller knows that they lie inside the array (for
// load8_any: that the 32 bytes from element idx on do).
__device__ __forceinline__ uint4 load8_u16(const uint16_t* __restrict__ x, int64_t idx) {
  return load16(reinterpret_cast<const char*>(x + idx));
}
__device__ __forceinline__ Raw8 load8_any(const void* __restrict__ x, int esize, int64_t idx) {
  const char* p = static_cast<const char*>(x) + idx * esize;
  return Raw8{load16(p), load16(p + 16)};
}
// Sixteen bytes from element idx on (elements of 2^LG bytes, LG = 1 or 2) of an
// array of `count` elements, zeros beyond its end, reading inside it only: the
// array's last sixteen bytes where fewer are left, moved down by what they
// start too early (one load; one by one, eight loads and their selects took
// most of a step).
template <int LG>
__device__ __forceinline__ uint4 load16_end(const char* __restrict__ x, int64_t idx, int64_t count) {
  constexpr int PER = 16 >> LG;
  uint32_t w[4] = {0, 0, 0, 0};
  if (count < PER) {
    // a whole array of less than sixteen bytes
    for (int e = 0; e < PER; ++e)
      if (idx + e < count) {
        if constexpr (LG == 1)
          w[e >> 1] |= (uint32_t)reinterpret_cast<const uint16_t*>(x)[idx + e] << (16 * (e & 1));
        else
          w[e] = reinterpret_cast<const uint32_t*>(x)[idx + e];
      }
    return uint4{w[0], w[1], w[2], w[3]};
  }
  const int64_t from = idx < count - PER ? idx : count - PER;
  const int sh = (int)(idx - from < PER ? idx - from : PER);  // elements to drop
  const uint4 u = load16(x + (from << LG));
  w[0] = u.x;
  w[1] = u.y;
  w[2] = u.z;
  w[3] = u.w;
  const int d = sh >> (2 - LG);  // whole dwords
#pragma unroll
  for (int bit = 2; bit > 0; bit >>= 1)
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = d & bit ? (e + bit < 4 ? w[e + bit < 4 ? e + bit : 3] : 0u) : w[e];
  if constexpr (LG == 1) {
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = sh & 1 ? (w[e] >> 16) | (e < 3 ? w[e < 3 ? e + 1 : 3] << 16 : 0u) : w[e];
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) w[e] = sh >= PER ? 0u : w[e];
  return uint4{w[0], w[1], w[2], w[3]};
}
__device__ __forceinline__ uint4 load8_u16_end(const uint16_t* __restrict__ x, int64_t idx, int64_t count) {
  return load16_end<1>(reinterpret_cast<const char*>(x), idx, count);
}
__device__ __forceinline__ Raw8 load8_any_end(const void* __restrict__ x, int dtype, int64_t idx, int64_t count) {
  const char* p = static_cast<const char*>(x);
  if (dtype != 0) return Raw8{load16_end<1>(p, idx, count), uint4{0, 0, 0, 0}};
  return Raw8{load16_end<2>(p, idx, count), load16_end<2>(p, idx + 4, count)};
}
// Masks of the first `valid` of eight 16-bit elements (the rest of a loaded
// chunk belongs to the next row).  Kept in vector registers: as comparisons
// they took a scalar register pair each, more than there are.
__device__ __forceinline__ uint4 first_mask(int valid) {
  uint32_t w[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) w[e] = valid >= 2 * e + 2 ? ~0u : valid == 2 * e + 1 ? 0xffffu : 0u;
  return uint4{w[0], w[1], w[2], w[3]};
}
__device__ __forceinline__ uint4 and4(uint4 a, uint4 m) { return uint4{a.x & m.x, a.y & m.y, a.z & m.z, a.w & m.w}; }
// Loaded elements as floats.  One (uniform) branch on the type for all of
// them: a choice per element became a branch per element.
template <int N>
__device__ __forceinline__ void raw8_floats(const Raw8 (&r)[N], int dtype, float (&f)[N][8]) {
  auto dw = [&](int i, int e) {
    const uint32_t a[8] = {r[i].a.x, r[i].a.y, r[i].a.z, r[i].a.w, r[i].b.x, r[i].b.y, r[i].b.z, r[i].b.w};
    return a[e];
  };
  if (dtype == 0) {
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) f[i][e] = __builtin_bit_cast(float, dw(i, e));
  } else if (dtype == 1) {
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) f[i][e] = F16::to_float((uint16_t)(dw(i, e >> 1) >> (16 * (e & 1))));
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) f[i][e] = BF16::to_float((uint16_t)(dw(i, e >> 1) >> (16 * (e & 1))));
  }
}
__device__ __forceinline__ void bf16_floats(uint4 u, float (&f)[8]) {
  const uint32_t a[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int e = 0; e < 8; ++e) f[e] = BF16::to_float((uint16_t)(a[e >> 1] >> (16 * (e & 1))));
}
__device__ __forceinline__ uint4 scaled_f16(const float (&f)[8], float s) {
  return uint4{pack_f16(f[0] * s, f[1] * s), pack_f16(f[2] * s, f[3] * s), pack_f16(f[4] * s, f[5] * s),
               pack_f16(f[6] * s, f[7] * s)};
}

// Sum of squares of eight 16-bit values in fp64 (each square is exact).
template <typename T>
__device__ __forceinline__ double square_sum(uint4 u, double acc) {
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const double v = (double)T::to_float((uint16_t)(w[e >> 1] >> (16 * (e & 1))));
    acc += v * v;
  }
  return acc;
}
__device__ __forceinline__ double sum_over_g(double x) {
  x += __shfl_xor(x, 16, kWave);
  x += __shfl_xor(x, 32, kWave);
  return x;
}

// The 16 x 32 A operand of tile `t` (16 columns) of a contraction over keys,
// read transposed from a wave's row tiles in LDS: NC chunks of 32 columns per
// 16-key tile, the layout and swizzle of the key ring (see tr_lane).
typedef short short4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4v lds_short4;
template <int NC>
__device__ __forceinline__ uint4 read_transposed(const char* base, TrLane trl, int t) {
  const char* p = base + (t >> 1) * 1024 + ((t & 1) ? trl.odd : trl.even);
  const short4v x0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(p));
  const short4v x1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(p + NC * 1024));
  const uint2 a = __builtin_bit_cast(uint2, x0), b = __builtin_bit_cast(uint2, x1);
  return uint4{a.x, a.y, b.x, b.y};
}

// Waves of a workgroup: sixteen where their registers fit four to a SIMD (the
// fp16 gradient at D <= 32 with two spilled values; bf16 spilled 22, and runs
// 2 - 10 % faster with eight: all gradients at 3663 points, D = 20, C = 1
// 42.0 -> 39.3 us).
constexpr int small_waves(int DP, int CV, int kind, bool bf16) {
  return CV == 0 && ((DP == 1 && !(bf16 && kind == kSmallGrad)) || (DP == 2 && kind == kSmallFwd)) ? 16 : 8;
}

// DP: 32-wide chunks of D.  CV: 32-wide chunks of the values (0: the single
// channel, whose value multiplies the kernel value in fp32).
template <typename T, int DP, int CV, int KIND>
struct SmallShape {
  static constexpr int DT = KIND == kSmallFwd ? 0 : 2 * DP;  // 16-row tiles of dQ
  static constexpr int CT = 2 * CV;                          // 16-row tiles of the sum
  static constexpr int NT = DT + CT;
  static constexpr int W = small_waves(DP, CV, KIND, std::is_same<T, BF16>::value);
  // LDS: the waves' transposed pieces, later the waves' partial results
  static constexpr int WAVE_LDS = ((KIND == kSmallFwd ? 0 : 2 * DP) + 2 * CV) * 1024;
  static constexpr int RED = (4 * NT + 1) * kWave * 4;       // per wave
  static constexpr int BYTES = W * (WAVE_LDS > RED ? WAVE_LDS : RED);
};

template <typename T, int DP, int CV, int KIND>
__global__ __launch_bounds__(kWave * small_waves(DP, CV, KIND, std::is_same<T, BF16>::value)) void k_small(
    SmallSide sa, SmallSide sb, unsigned blocks0, float tau2, float tau, int D, int C) {
  using S = SmallShape<T, DP, CV, KIND>;
  constexpr int DT = S::DT, CT = S::CT, NT = S::NT, W = S::W;
  constexpr int NV = CV > 0 ? CV : 1, NTA = NT > 0 ? NT : 1;
  constexpr bool ONE = CV == 0;
  constexpr bool LOGV = ONE && KIND == kSmallGrad;  // |v| in the exponent
  constexpr bool BF = std::is_same<T, BF16>::value;
  static_assert(S::BYTES <= 160 * 1024, "LDS of a workgroup");
  static_assert(KIND != kSmallSvgd || CV > 0, "SVGD has D score channels");
  __shared__ __attribute__((aligned(1024))) char lds[S::BYTES];

  const bool first = blockIdx.x < blocks0;
  const SmallSide& s = first ? sa : sb;
  const int64_t z = blockIdx.z;
  auto at = [&](const void* p, int64_t bytes) { return static_cast<const char*>(p) + z * bytes; };
  const uint16_t* __restrict__ q = reinterpret_cast<const uint16_t*>(at(s.q, s.bq));
  const uint16_t* __restrict__ k = reinterpret_cast<const uint16_t*>(at(s.k, s.bk));
  const void* __restrict__ v = at(s.v, s.bv);
  const void* __restrict__ gr = s.g ? at(s.g, s.bg) : nullptr;
  const int64_t M = s.M, N = s.N;
  const int vdt = s.v_dtype, gdt = s.g_dtype;
  // (the wave's index in a scalar register: the branches on its steps then are scalar)
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int j = lane & 15, g = lane >> 4;
  const int64_t q0 = (int64_t)(first ? blockIdx.x : blockIdx.x - blocks0) * 16;
  const int steps = (int)((N + kStep - 1) / kStep);

  // columns of the lane's eight that belong to the row, per 32-wide chunk
  auto dcols = [&](int dc) { return D - 32 * dc - 8 * g; };
  auto ccols = [&](int cc) { return C - 32 * cc - 8 * g; };

  const int ves = vdt == 0 ? 4 : 2, ges = gdt == 0 ? 4 : 2;
  uint4 km[DP], vm[NV];
#pragma unroll
  for (int dc = 0; dc < DP; ++dc) km[dc] = first_mask(dcols(dc));
#pragma unroll
  for (int cc = 0; cc < NV; ++cc) vm[cc] = first_mask(ccols(cc));
  // the steps before `full` can be loaded whole: every 16 bytes that fetch
  // reads lie inside the arrays
  auto whole = [&](int st) {
    const int64_t last = (int64_t)(st + 1) * kStep;  // rows before it
    if (last > N || (last - 1) * D + 32 * DP > N * D) return false;
    return ONE ? (last - 4) * ves + 16 <= N * ves : ((last - 1) * C + 32 * CV - 8) * ves + 32 <= N * C * ves;
  };
  int full = steps;
  while (full > 0 && !whole(full - 1)) --full;

  // the next step's rows, as loaded (garbage beyond a row's end is masked at
  // the use, so that no load is waited for here)
  uint4 kn[2][DP];
  Raw8 vn[2][NV];
  uint4 v1n[2];
  auto fetch = [&](int st) {
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      const int64_t r0 = (int64_t)st * kStep + 16 * kt;
#pragma unroll
      for (int dc = 0; dc < DP; ++dc) kn[kt][dc] = load8_u16(k, (r0 + j) * D + 32 * dc + 8 * g);
      if constexpr (ONE) {
        v1n[kt] = load16(static_cast<const char*>(v) + (r0 + 4 * g) * ves);
      } else {
#pragma unroll
        for (int cc = 0; cc < CV; ++cc) vn[kt][cc] = load8_any(v, ves, (r0 + j) * C + 32 * cc + 8 * g);
      }
    }
  };
  auto fetch_end = [&](int st) {
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      const int64_t r0 = (int64_t)st * kStep + 16 * kt;
#pragma unroll
      for (int dc = 0; dc < DP; ++dc) kn[kt][dc] = load8_u16_end(k, (r0 + j) * D + 32 * dc + 8 * g, N * D);
      if constexpr (ONE) {
        v1n[kt] = vdt == 0 ? load16_end<2>(static_cast<const char*>(v), r0 + 4 * g, N)
                           : load16_end<1>(static_cast<const char*>(v), r0 + 4 * g, N);
      } else {
#pragma unroll
        for (int cc = 0; cc < CV; ++cc) vn[kt][cc] = load8_any_end(v, vdt, (r0 + j) * C + 32 * cc + 8 * g, N * C);
      }
    }
  };
  int st = wave;
  if (st < full) fetch(st);

  // queries: operands, half norms, upstream gradients
  uint4 qreg[DP];
  double qq = 0.0;
  if ((q0 + 15) * D + 32 * DP <= M * D) {
#pragma unroll
    for (int dc = 0; dc < DP; ++dc) qreg[dc] = load8_u16(q, (q0 + j) * D + 32 * dc + 8 * g);
#pragma unroll
    for (int dc = 0; dc < DP; ++dc) qreg[dc] = and4(qreg[dc], km[dc]);
  } else {
#pragma unroll
    for (int dc = 0; dc < DP; ++dc)
      qreg[dc] = and4(load8_u16_end(q, (q0 + j) * D + 32 * dc + 8 * g, M * D), km[dc]);
  }
#pragma unroll
  for (int dc = 0; dc < DP; ++dc) qq = square_sum<T>(qreg[dc], qq);
  const float bq = tau2 * (float)(-0.5 * sum_over_g(qq));
  uint4 greg[NV];
  int eg = 0;
  if constexpr (KIND == kSmallGrad && !ONE) {
    // scaled by the largest magnitude of the workgroup's own rows
    float f[NV][8];
    Raw8 r[NV];
    uint32_t mb = 0;
    const bool inside = ((q0 + 15) * C + 32 * CV - 8) * ges + 32 <= M * C * ges;
#pragma unroll
    for (int cc = 0; cc < CV; ++cc) {
      const int64_t idx = (q0 + j) * C + 32 * cc + 8 * g;
      r[cc] = inside ? load8_any(gr, ges, idx) : load8_any_end(gr, gdt, idx, M * C);
    }
    raw8_floats(r, gdt, f);
#pragma unroll
    for (int cc = 0; cc < CV; ++cc)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if (e >= ccols(cc)) f[cc][e] = 0.0f;
        mb = umax32(mb, __builtin_bit_cast(uint32_t, fabsf(f[cc][e])));
      }
    eg = scale_exponent(wave_umax(mb));
    const float sg = ldexpf(1.0f, eg);
#pragma unroll
    for (int cc = 0; cc < CV; ++cc) greg[cc] = scaled_f16(f[cc], sg);
  }

  // running scales (powers of two) of the fp16 values and of the fp16 copy of
  // bf16 keys: the exponent and the largest magnitude it is good for (they come
  // from single key steps, which may hold subnormal numbers only: kMaxScale)
  int ev = 0, ek = 0;
  float vlim = 0.0f, klim = 0.0f, sv = 1.0f, sk = 1.0f;

  char* kl = lds + wave * S::WAVE_LDS;                       // key rows (gradients)
  char* vl = kl + (KIND == kSmallFwd ? 0 : 2 * DP) * 1024;   // value rows
  const TrLane trl = tr_lane(lane);
  const int lrow = j * 64 + lds_col(j, g) * 16;              // the lane's place in a 1-KiB chunk

  floatx4 acc[NTA];  // dQ tiles, then tiles of the sum
#pragma unroll
  for (int t = 0; t < NTA; ++t) acc[t] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
  // off: whole numbers (-3e38 before any exponent above -inf); cap: kernel
  // value 1 relative to the offset, and no more than a raise leaves (where an
  // exponent's terms are so large that they round by whole units, 2^27 and up,
  // an exponent may come out above the offset taken from it)
  float rs = 0.0f, off = -3.0e38f, cap = kSmallCap;
  const int src = 16 * (j >> 2) + (j & 3);  // a lane that holds key j's single-channel value

  for (; st < steps; st += W) {
    if (st >= full) fetch_end(st);
    uint4 kr[2][DP];
    Raw8 vr[2][NV];
    float v1[2][4];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
      for (int dc = 0; dc < DP; ++dc) kr[kt][dc] = and4(kn[kt][dc], km[dc]);
      if constexpr (ONE) {
        vr[kt][0] = Raw8{v1n[kt], v1n[kt]};
      } else {
#pragma unroll
        for (int cc = 0; cc < CV; ++cc) vr[kt][cc] = vn[kt][cc];
      }
    }
    if constexpr (ONE) {
      float f[2][8];
      const Raw8 r1[2] = {vr[0][0], vr[1][0]};
      raw8_floats(r1, vdt, f);
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int e = 0; e < 4; ++e) v1[kt][e] = f[kt][e];
    }
    if (st + W < full) fetch(st + W);

    floatx4 sc[2];
    float lv[2][4];  // log2 |v| of the lane's keys
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      if constexpr (LOGV) {
        // each lane the logarithm of one key, handed out like the half norms
        const float x = j & 2 ? (j & 1 ? v1[kt][3] : v1[kt][2]) : (j & 1 ? v1[kt][1] : v1[kt][0]);
        const float l = log2f(fabsf(__shfl(x, src, kWave)));
#pragma unroll
        for (int e = 0; e < 4; ++e) lv[kt][e] = __shfl(l, 4 * g + e, kWave);
      }
      double kk = 0.0;
#pragma unroll
      for (int dc = 0; dc < DP; ++dc) kk = square_sum<T>(kr[kt][dc], kk);
      const int64_t r = (int64_t)st * kStep + 16 * kt + j;
      kk = sum_over_g(kk);
      const float nh = r < N ? (float)(-0.5 * kk) : kPadBias;
      floatx4 cin;
#pragma unroll
      for (int e = 0; e < 4; ++e) cin[e] = __shfl(nh, 4 * g + e, kWave);
      sc[kt] = score_tile<T, DP>(kr[kt], qreg, cin);
    }
    if constexpr (KIND == kSmallFwd && ONE) {
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int e = 0; e < 4; ++e) rs = fmaf(exp2_clamped(fmaf(sc[kt][e], tau2, bq)), v1[kt][e], rs);
      continue;
    }
    // values: a larger magnitude than any before moves the scale (exact).  What
    // lies beyond a row's end is elements of other rows, masked after packing.
    uint4 vh[2][NV];
    if constexpr (!ONE) {
      float vf[2][NV][8];
      float vmax = 0.0f;
      raw8_floats(vr[0], vdt, vf[0]);
      raw8_floats(vr[1], vdt, vf[1]);
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int cc = 0; cc < CV; ++cc)
#pragma unroll
          for (int e = 0; e < 8; ++e) vmax = fmaxf(vmax, fabsf(vf[kt][cc][e]));
      if (__any(vmax > vlim)) {
        const int e = scale_exponent(wave_umax(__builtin_bit_cast(uint32_t, vmax)));
        const int ne = vlim > 0.0f && e > ev ? ev : e;
        const float f = vlim > 0.0f ? ldexpf(1.0f, ne - ev) : 1.0f;
#pragma unroll
        for (int t = KIND == kSmallSvgd ? DT : 0; t < NT; ++t)
#pragma unroll
          for (int e4 = 0; e4 < 4; ++e4) acc[t][e4] *= f;
        if constexpr (KIND != kSmallSvgd) rs *= f;
        ev = ne;
        sv = ldexpf(1.0f, ev);
        vlim = ldexpf(1.99999988f, -ev);
      }
      // value rows as fp16: registers for w, LDS for the sum
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int cc = 0; cc < CV; ++cc) {
          vh[kt][cc] = and4(scaled_f16(vf[kt][cc], sv), vm[cc]);
          *reinterpret_cast<uint4*>(vl + (kt * CV + cc) * 1024 + lrow) = vh[kt][cc];
        }
    }
    if constexpr (KIND != kSmallFwd) {
      if constexpr (BF) {
        float kmax = 0.0f;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
          for (int dc = 0; dc < DP; ++dc) {
            float f[8];
            bf16_floats(kr[kt][dc], f);
#pragma unroll
            for (int e = 0; e < 8; ++e) kmax = fmaxf(kmax, fabsf(f[e]));
          }
        if (__any(kmax > klim)) {
          const int e = point_scale_exponent(wave_umax(__builtin_bit_cast(uint32_t, kmax)));
          const int ne = klim > 0.0f && e > ek ? ek : e;
          const float f = klim > 0.0f ? ldexpf(1.0f, ne - ek) : 1.0f;
#pragma unroll
          for (int t = 0; t < DT; ++t)
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) acc[t][e4] *= f;
          ek = ne;
          sk = ldexpf(1.0f, ek);
          klim = ldexpf(1.99999988f, kPointScaleHeadroom - ek);
        }
      }
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int dc = 0; dc < DP; ++dc) {
          uint4 h = kr[kt][dc];
          if constexpr (BF) {
            float f[8];
            bf16_floats(h, f);
            h = scaled_f16(f, sk);
          }
          *reinterpret_cast<uint4*>(kl + (kt * DP + dc) * 1024 + lrow) = h;
        }
    }
    // running offset of each row (see the top of the file)
    float y[2][4], top = -__builtin_inff();
    const float be = bq - off;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
      for (int e = 0; e < 4; ++e) y[kt][e] = fmaf(sc[kt][e], tau2, LOGV ? be + lv[kt][e] : be);
      top = max_into(top, floatx4{y[kt][0], y[kt][1], y[kt][2], y[kt][3]});
    }
    if (__any(top > kSmallRaise)) {
      float raw = -__builtin_inff();
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x = fmaf(sc[kt][e], tau2, bq), c = x > 0.0f ? 0.0f : x;  // (NaN stays, and is passed over)
          raw = fmaxf(raw, LOGV ? c + lv[kt][e] : c);
        }
      // whole numbers, so that all scaling by offsets is exact (a gradient
      // term's k - q then cancels exactly where it should)
      const float nw = fmaxf(off, floorf(wave_max_over_g(raw)));
      const float f = nw > off ? exp2f(off - nw) : 1.0f;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[t][e] *= f;
      rs *= f;
      off = nw;
      cap = exp2f(-nw);
      if constexpr (!LOGV) cap = fminf(cap, kSmallCap);
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int e = 0; e < 4; ++e) y[kt][e] = fmaf(sc[kt][e], tau2, LOGV ? bq - off + lv[kt][e] : bq - off);
    }
    // kernel values relative to the offset, clamped to [0, 1] in their own
    // units (LOGV: times |v|, to [0, |v|])
    float phi[2][4], p[2][4];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        phi[kt][e] = __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(y[kt][e]), 0.0f,
                                             LOGV ? fminf(fabsf(v1[kt][e]) * cap, kSmallCap) : cap);
      if constexpr (KIND == kSmallGrad) {
        if constexpr (ONE) {
#pragma unroll
          for (int e = 0; e < 4; ++e) p[kt][e] = copysignf(phi[kt][e], v1[kt][e]);
        } else {
          floatx4 w = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int cc = 0; cc < CV; ++cc) w = mfma_f16(vh[kt][cc], greg[cc], w);
#pragma unroll
          for (int e = 0; e < 4; ++e) p[kt][e] = phi[kt][e] * w[e];
        }
      }
    }
    const uint4 bphi = pack_tile_pair(phi);
    const uint4 b = KIND == kSmallGrad ? pack_tile_pair(p) : bphi;
    if constexpr (KIND != kSmallFwd) {
#pragma unroll
      for (int t = 0; t < DT; ++t) acc[t] = mfma_f16(read_transposed<DP>(kl, trl, t), b, acc[t]);
      rs = dot2_acc(b, uint4{0x3C003C00u, 0x3C003C00u, 0x3C003C00u, 0x3C003C00u}, rs);
    }
    if constexpr (!ONE) {
#pragma unroll
      for (int t = 0; t < CT; ++t) acc[DT + t] = mfma_f16(read_transposed<NV>(vl, trl, t), bphi, acc[DT + t]);
    }
  }

  // partial results of the waves without their offsets and scales
  // (2^off through ldexp: no denormal or infinite factor; offsets beyond any
  // result's range, and that of a wave without steps, bounded)
  const int eo = KIND == kSmallFwd && ONE ? 0 : (int)fmaxf(off, -1.0e6f);
  rs += __shfl_xor(rs, 16, kWave);
  rs += __shfl_xor(rs, 32, kWave);
  __syncthreads();  // every wave is done with its piece of LDS
  float* red = reinterpret_cast<float*>(lds);
  auto slot = [&](int i, int w) { return (i * W + w) * kWave + lane; };
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      red[slot(4 * t + e, wave)] =
          ldexpf(acc[t][e], eo - (t < DT ? ek : 0) - (KIND == kSmallSvgd && t < DT ? 0 : ev));
  red[slot(4 * NT, wave)] = ldexpf(rs, eo - (KIND == kSmallSvgd ? 0 : ev));
  __syncthreads();
  auto total = [&](int i) {
    float x = red[slot(i, 0)];
#pragma unroll
    for (int w = 1; w < W; ++w) x += red[slot(i, w)];
    return x;
  };
  const int64_t m = q0 + j;
  const float rm = total(4 * NT);
  if constexpr (ONE) {
    if (wave == 0 && g == 0 && m < M && s.out_s)
      reinterpret_cast<float*>(const_cast<char*>(at(s.out_s, s.bs)))[m] = rm;
  }
  if constexpr (KIND != kSmallFwd) {
    float* out = s.out_d ? reinterpret_cast<float*>(const_cast<char*>(at(s.out_d, s.bd))) : nullptr;
    float f = tau;
    if constexpr (KIND == kSmallGrad && ONE) {
      if (gr && m < M) f *= load_any(gr, m, gdt);
    }
        const bool v4 = vec4_rows(out, D);
    for (int t = wave; t < DT; t += W) {
      const int d0 = 16 * t + 4 * g;
      if (!s.out_d || m >= M || d0 >= D) continue;
      float o[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float qv = d0 + e < D ? T::to_float(q[m * D + d0 + e]) : 0.0f;
        const float d = total(4 * t + e) - qv * rm;
        if constexpr (KIND == kSmallSvgd)
          o[e] = (t < CT ? total(4 * (DT + t) + e) : 0.0f) - d * f;
        else
          o[e] = ldexpf(d * f, -eg);
      }
      store_row4(out + m * D, d0, D, v4, o[0], o[1], o[2], o[3]);
    }
  }
  if constexpr (KIND != kSmallSvgd && !ONE) {
    if (s.out_s) {
      float* out = reinterpret_cast<float*>(const_cast<char*>(at(s.out_s, s.bs)));
      const bool v4 = vec4_rows(out, C);
      for (int t = wave; t < CT; t += W) {
        const int c0 = 16 * t + 4 * g;
        if (m >= M || c0 >= C) continue;
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = total(4 * (DT + t) + e);
        store_row4(out + m * C, c0, C, v4, o[0], o[1], o[2], o[3]);
      }
    }
  }
}

}  // namespace gs
