// gs_prep.h -- per-call preparation of the operands (linear cost).
//
//  * points: padded RT-layout copy in the input dtype (operand of q.k), the
//    fp32 half squared norm -||x||^2/2 (from the exact input values, summed in
//    fp64), the key scalars of the passes these points are the keys of, a
//    sample of rows for the row bound, and optionally a KS-layout fp16 copy
//    (operand of sum_n P_mn k_n).  fp32 points: two fp16 parts instead.
//  * values: exact power-of-two scaling so the largest |value| lies in [1, 2)
//    (RT: w_headroom binades higher), then fp16 copies in RT layout
//    (contraction over C) and / or KS layout (contraction over keys).
//
// A call's whole preparation is one launch (k_prep), or two when the maxima
// that the scales come from take more than a workgroup's glance (k_prep_max
// first): the work is linear and short, so separate kernels (up to 17 of them
// for a forward and full gradient, each a dependent launch of 3 - 5 us and as
// much host time) cost ordinary calls much of their time.  Per call, before and
// after (the smallest calls do not prepare at all: gs_small.h): a sum at
// M = N = 9000, D = 16 47 -> 33 us, a flow of 6000 particles in D = 3 60 -> 35 us,
// an SVGD direction of 4000 in D = 45 53 -> 42 us, sum and gradients through
// autograd at M = 6001, N = 9003, D = 50, C = 10 214 - 262 -> 176 us, sum and
// gradients at M = N = 16384, D = C = 128 722 -> 687 us.
#pragma once

#include "gs_common.h"

namespace gs {

#if !defined(GS_PART) || GS_PART == 0  // (kernels that are no templates: in one build part only)
__global__ void k_fill_f32(float* __restrict__ p, int64_t n, float val) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = val;
}
#endif

// ---------------------------------------------------------------- maxima

// An array whose largest magnitude a scale comes from.
struct MaxSource {
  const void* x;
  int64_t bz;      // byte stride between problems
  int64_t count;
  int dtype;
  int slot;        // which maximum: 0 |v|, 1 |dout|, 2 |q|, 3 |k|
  int parts;       // partial maxima of k_prep_max (0: none, reduce the array itself)
};
constexpr int kMaxSlots = 4;
constexpr int kMaxBlock = 1024;     // threads of k_prep_max

// The larger of two magnitudes given as float bits (|x| >= 0, so unsigned
// comparison of the bit patterns orders them; NaN compares largest).
__device__ __forceinline__ uint32_t umax32(uint32_t a, uint32_t b) { return a > b ? a : b; }

__device__ __forceinline__ uint32_t wave_umax(uint32_t m) {
  for (int off = 32; off > 0; off >>= 1) m = umax32(m, (uint32_t)__shfl_xor((int)m, off, kWave));
  return m;
}

// Largest |x[i]| over the elements that thread `tid` of `stride` threads takes
// (float bits), 16-byte loads, four of them in flight, where x allows.
__device__ __forceinline__ uint32_t absmax_strided(const void* __restrict__ x, int64_t count, int dtype,
                                                   int64_t tid, int64_t stride) {
  uint32_t mb = 0;
  auto take = [&](float f) { mb = umax32(mb, __builtin_bit_cast(uint32_t, fabsf(f))); };
  int64_t done = 0;
  if ((reinterpret_cast<uintptr_t>(x) & 15) == 0) {
    const int per = dtype == 0 ? 4 : 8;
    const int64_t nv = count / per;
    const uint4* xv = static_cast<const uint4*>(x);
    auto vec = [&](const uint4 w) {
      const uint32_t u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (dtype == 0) {
          take(__builtin_bit_cast(float, u[e]));
        } else {
          const uint16_t lo = (uint16_t)(u[e] & 0xffffu), hi = (uint16_t)(u[e] >> 16);
          take(dtype == 1 ? F16::to_float(lo) : BF16::to_float(lo));
          take(dtype == 1 ? F16::to_float(hi) : BF16::to_float(hi));
        }
      }
    };
    int64_t j = tid;
    for (; j + 3 * stride < nv; j += 4 * stride) {
      const uint4 a = xv[j], b = xv[j + stride], c = xv[j + 2 * stride], d = xv[j + 3 * stride];
      vec(a);
      vec(b);
      vec(c);
      vec(d);
    }
    for (; j < nv; j += stride) vec(xv[j]);
    done = nv * per;
  }
  int64_t i = done + tid;
  for (; i + 3 * stride < count; i += 4 * stride) {
    float f[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) f[u] = load_any(x, i + u * stride, dtype);
#pragma unroll
    for (int u = 0; u < 4; ++u) take(f[u]);
  }
  for (; i < count; i += stride) take(load_any(x, i, dtype));
  return mb;
}

struct MaxArgs {
  int n;
  MaxSource src[kMaxSlots];
};

// Partial maxima: workgroup (b, i) of grid (blocks, arrays) reduces its share
// of array i into part[i * pitch + b].  No atomics, so nothing has
// to be cleared first.
#if !defined(GS_PART) || GS_PART == 0  // (kernels that are no templates: in one build part only)
__global__ __launch_bounds__(kMaxBlock) void k_prep_max(MaxArgs a, uint32_t* __restrict__ part, int pitch, Bz bz) {
  __shared__ uint32_t wmax[kMaxBlock / kWave];
  const MaxSource s = a.src[blockIdx.y];
  if ((int)blockIdx.x >= s.parts) return;
  part = zoff(part, bz.ws);
  uint32_t mb = wave_umax(absmax_strided(zoff(s.x, s.bz), s.count, s.dtype,
                                         (int64_t)blockIdx.x * kMaxBlock + threadIdx.x,
                                         (int64_t)s.parts * kMaxBlock));
  if ((threadIdx.x & (kWave - 1)) == 0) wmax[threadIdx.x / kWave] = mb;
  __syncthreads();
  if (threadIdx.x < kWave) {
    mb = wave_umax(threadIdx.x < kMaxBlock / kWave ? wmax[threadIdx.x] : 0u);
    if (threadIdx.x == 0) part[blockIdx.y * pitch + blockIdx.x] = mb;
  }
}
#endif

// ---------------------------------------------------------------- points

// Row r of a point set, columns 8c .. 8c+7 (zero beyond n rows or D columns).
// vec: rows start on 16-byte boundaries and D is a multiple of 8, so they are
// one 16-byte load.
__device__ __forceinline__ void load_cols8(const uint16_t* __restrict__ x, int64_t r, int64_t n, int D, int c,
                                           int vec, uint16_t (&h)[8]) {
  if (vec) {
    uint4 u = make_uint4(0, 0, 0, 0);
    if (r < n && 8 * c < D) u = *reinterpret_cast<const uint4*>(x + r * D + 8 * c);
    const uint32_t wd[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) h[e] = (uint16_t)(wd[e >> 1] >> (16 * (e & 1)));
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int w = 8 * c + e;
      h[e] = (r < n && w < D) ? x[r * D + w] : (uint16_t)0;
    }
  }
}

__device__ __forceinline__ uint4 pack8(const uint16_t (&h)[8]) {
  uint4 pk;
  pk.x = h[0] | ((uint32_t)h[1] << 16);
  pk.y = h[2] | ((uint32_t)h[3] << 16);
  pk.z = h[4] | ((uint32_t)h[5] << 16);
  pk.w = h[6] | ((uint32_t)h[7] << 16);
  return pk;
}

// Sum over the 2^lg consecutive lanes of a point row (whole rows lie in one
// wave), the same value in each of them.
__device__ __forceinline__ double row_sum(double acc, int lg) {
  for (int off = (1 << lg) >> 1; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kWave);
  return acc;
}

// Key row of sample position pos: rows floor(j N / kSampleRows), the coarse
// sample j = 0, 16, 32, ... (the rows floor(i N / kSampleCoarse)) at the first
// kSampleCoarse positions, the other j in increasing order after them, so
// that the coarse sample is the first kSampleCoarse / 16 RT tiles.
__device__ __forceinline__ int64_t sample_row(int pos, int64_t n) {
  constexpr int kStride = kSampleRows / kSampleCoarse;
  int j;
  if (pos < kSampleCoarse) {
    j = kStride * pos;
  } else {
    const int q = pos - kSampleCoarse;
    j = (q / (kStride - 1)) * kStride + q % (kStride - 1) + 1;
  }
  return ((int64_t)j * n) / kSampleRows;
}

// RT copy and half norms: thread (row r, chunk c) moves columns 8c .. 8c+7 of
// a row (one 16-byte store: those eight columns are contiguous in the RT
// copy) and sums their squares in fp64; the row's threads are consecutive
// lanes, so the half norm is rounded once to fp32.  Padding rows and columns
// are zero, padding rows get kPadBias.  src_row: the row of x that row r of
// the copy takes.  Returns the row's half norm (the same value in every lane
// of the row).
template <typename T>
__device__ __forceinline__ float rt_norm_item(const uint16_t* __restrict__ x, int64_t n, int D, int W, int lg,
                                              uint16_t* __restrict__ xs, float* __restrict__ nh, int vec,
                                              int64_t r, int c, int64_t src_row) {
  uint16_t h[8];
  load_cols8(x, src_row, n, D, c, vec, h);
  double acc = 0.0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const double v = (double)T::to_float(h[e]);
    acc += v * v;
  }
  acc = row_sum(acc, lg);
  *reinterpret_cast<uint4*>(xs + rt_index(r, 8 * c, W)) = pack8(h);
  const float half = src_row < n ? (float)(-0.5 * acc) : kPadBias;
  if (c == 0) nh[r] = half;
  return half;
}

// Position of key o (0 .. 31) of a step in the KS layout (its key slot).
__device__ __forceinline__ int key_slot(int o) { return 8 * ((o & 15) >> 2) + 4 * (o >> 4) + (o & 3); }
// Key of slot z of step s.
__device__ __forceinline__ int64_t slot_key(int64_t s, int z) {
  return s * 32 + 16 * ((z & 7) >> 2) + 4 * (z >> 3) + (z & 3);
}

// Per-step key scalars, 64 floats (256 bytes) per 32-key step:
//   [0, 32)  key bias b_n = -||k_n||^2/2, and for single-channel values
//            (v != NULL) additionally log2|v_n 2^e| / tau' with e putting
//            max |v 2^e| in [0.5, 1): the magnitude of v_n then enters the
//            exponent in fp32 (log2 0 = -inf gives an exact 0);
//   [32, 48) for single-channel values, sign(v_n) as fp16 +-1 in key-slot
//            order (the order of the MFMA B operand built from two score
//            tiles), two per float; otherwise not written;
//   [48, 64) not written.
// key_scalars writes the entries of key r (half norm `half`).
__device__ __forceinline__ void key_scalars(float* __restrict__ scal, float half, const void* __restrict__ v,
                                            int dtype, int64_t n, int64_t r, float sc, float tau2) {
  float* step = scal + (r >> 5) * 64;
  float bias = half;
  uint16_t sign = 0x3C00u;
  if (v && r < n) {
    const float val = load_any(v, r, dtype);
    bias += log2f(fabsf(val * sc)) / tau2;
    if (val < 0.0f) sign = 0xBC00u;
  }
  step[r & 31] = bias;
  if (v) reinterpret_cast<uint16_t*>(step + 32)[key_slot((int)(r & 31))] = sign;
}

// KS-layout fp16 copy of points scaled by s (bf16 points, whose range exceeds
// fp16; 1 for fp16 points) and, when sgn != NULL, multiplied by the sign of
// the single-channel value sgn[r] (exact).  Thread (32-key block, row w,
// quarter a) writes the eight key slots 8a .. 8a+7 of row w (one 16-byte
// store); consecutive threads write consecutive 16 bytes.
template <typename T>
__device__ __forceinline__ void points_ks_item(const uint16_t* __restrict__ x, int64_t n, int D, int lgR, float s,
                                               const void* __restrict__ sgn, int sgn_dtype,
                                               uint16_t* __restrict__ xt, int64_t t) {
  const int a = (int)(t & 3);
  const int64_t rest = t >> 2;
  const int64_t blk = rest >> lgR;
  const int w = (int)(rest & ((1 << lgR) - 1));
  uint16_t h[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int64_t r = slot_key(blk, 8 * a + e);
    float v = (r < n && w < D) ? T::to_float(x[r * D + w]) * s : 0.0f;
    if (sgn && r < n && load_any(sgn, r, sgn_dtype) < 0.0f) v = -v;
    h[e] = __builtin_bit_cast(uint16_t, (_Float16)v);
  }
  *reinterpret_cast<uint4*>(xt + (rest * 32 + 8 * a)) = pack8(h);
}

// ---------------------------------------------------------------- values

// fp16 copy of the values scaled by s, RT layout: thread (row, eight columns).
__device__ __forceinline__ void values_rt_item(const void* __restrict__ v, int dtype, int64_t n, int C, int W,
                                               float s, uint16_t* __restrict__ vs, int64_t r, int c) {
  uint16_t h[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int w = 8 * c + e;
    const float val = (r < n && w < C) ? load_any(v, r * C + w, dtype) * s : 0.0f;
    h[e] = __builtin_bit_cast(uint16_t, (_Float16)val);
  }
  *reinterpret_cast<uint4*>(vs + rt_index(r, 8 * c, W)) = pack8(h);
}

// KS layout; with sign_only (single-channel values, whose magnitudes enter
// the exponent through the step scalars) row 0 holds sign(v) = +-1 instead.
// Thread (32-key block, row w, quarter a) as points_ks_item.
__device__ __forceinline__ void values_ks_item(const void* __restrict__ v, int dtype, int64_t n, int C, int lgR,
                                               float s, int sign_only, uint16_t* __restrict__ vt, int64_t t) {
  const int a = (int)(t & 3);
  const int64_t rest = t >> 2;
  const int64_t blk = rest >> lgR;
  const int w = (int)(rest & ((1 << lgR) - 1));
  uint16_t h[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int64_t r = slot_key(blk, 8 * a + e);
    float val = (r < n && w < C) ? load_any(v, r * C + w, dtype) * s : 0.0f;
    if (sign_only) val = (r < n && w == 0) ? (val < 0.0f ? -1.0f : 1.0f) : 0.0f;
    h[e] = __builtin_bit_cast(uint16_t, (_Float16)val);
  }
  *reinterpret_cast<uint4*>(vt + (rest * 32 + 8 * a)) = pack8(h);
}

// ---------------------------------------------------------------- fp32 tier

// Scale exponent of the split copies: max |x| 2^e in [2^14, 2^15).
constexpr int kSplitHeadroom = 14;

// fp32 points -> scaled hi / lo fp16 copies (RT layout) and fp32 half norms
// -||x||^2/2 (exact fp32 inputs, squares summed in fp64); thread (row, eight
// columns) as rt_norm_item.  Returns the half norm.
__device__ __forceinline__ float split_item(const float* __restrict__ x, int64_t n, int D, int W, int lg, int e,
                                            uint16_t* __restrict__ hi, uint16_t* __restrict__ lo,
                                            float* __restrict__ nh, int64_t r, int c) {
  uint16_t h[8], l[8];
  double acc = 0.0;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int w = 8 * c + k;
    const float xv = (r < n && w < D) ? x[r * D + w] : 0.0f;
    acc += (double)xv * (double)xv;
    const float xs = ldexpf(xv, e);
    const _Float16 hh = (_Float16)xs;
    h[k] = __builtin_bit_cast(uint16_t, hh);
    l[k] = __builtin_bit_cast(uint16_t, (_Float16)(xs - (float)hh));
  }
  acc = row_sum(acc, lg);
  *reinterpret_cast<uint4*>(hi + rt_index(r, 8 * c, W)) = pack8(h);
  *reinterpret_cast<uint4*>(lo + rt_index(r, 8 * c, W)) = pack8(l);
  const float half = r < n ? (float)(-0.5 * acc) : kPadBias;
  if (c == 0) nh[r] = half;
  return half;
}

// Step scalars of the fp32 tier, 64 floats per 32-key step (v = NULL for
// several value channels: the bias is the scaled half norm alone, signs +1):
//   [0, 32)  2^es (b_n + log2 |v_n 2^ev| / tau'), the key bias in the scaled
//            units of the split scores (-inf for padding keys and for v_n = 0:
//            an exact zero term);
//   [32, 64) sign(v_n) as +-1.0f, key 32 s + i at position 32 + i (the row
//            order of the two 16-key score tiles).
// The bias is formed in fp64 and rounded once (the fp32 log2 and its division
// would add about one ulp of a systematic error to every term).
__device__ __forceinline__ void key_scalars32(float* __restrict__ scal, float half, const void* __restrict__ v,
                                              int dtype, int64_t n, int64_t r, int ev, int es, float tau2) {
  float* step = scal + (r >> 5) * 64;
  float bias = -__builtin_inff(), sign = 1.0f;
  if (r < n) {
    double lv = 0.0;
    if (v) {
      const float val = load_any(v, r, dtype);
      lv = log2(fabs((double)val)) + ev;
      if (val < 0.0f) sign = -1.0f;
    }
    bias = (float)ldexp((double)half + lv / (double)tau2, es);
  }
  step[r & 31] = bias;
  step[32 + (r & 31)] = sign;
}

// Values (several channels) for the fp32 tier: v 2^ev (max |v| 2^ev in [1, 2))
// split into fp16 hi + lo 2^-kSplitLow (scaled so that lo stays out of the
// subnormals), both in KS layout, written as values_ks_item does.
constexpr int kSplitLow = 11;
constexpr float kSplitLowScale = (float)(1 << kSplitLow);
__device__ __forceinline__ void values_ks_split_item(const void* __restrict__ v, int dtype, int64_t n, int C,
                                                     int lgR, int ev, uint16_t* __restrict__ vh,
                                                     uint16_t* __restrict__ vl, int64_t t) {
  const int a = (int)(t & 3);
  const int64_t rest = t >> 2;
  const int64_t blk = rest >> lgR;
  const int w = (int)(rest & ((1 << lgR) - 1));
  uint16_t h[8], l[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int64_t r = slot_key(blk, 8 * a + e);
    const float x = (r < n && w < C) ? ldexpf(load_any(v, r * C + w, dtype), ev) : 0.0f;
    const _Float16 hh = (_Float16)x;
    h[e] = __builtin_bit_cast(uint16_t, hh);
    l[e] = __builtin_bit_cast(uint16_t, (_Float16)((x - (float)hh) * kSplitLowScale));
  }
  *reinterpret_cast<uint4*>(vh + (rest * 32 + 8 * a)) = pack8(h);
  *reinterpret_cast<uint4*>(vl + (rest * 32 + 8 * a)) = pack8(l);
}

// ---------------------------------------------------------------- one launch

enum PrepKind : int {
  kJobPoints,        // RT copy, half norms, step scalars
  kJobSample,        // sampled rows and their half norms
  kJobPointsKs,
  kJobValuesRt,
  kJobValuesKs,
  kJobSplit,         // fp32 tier: split RT copies, half norms, step scalars
  kJobValuesKsSplit  // fp32 tier
};

// Key scalars a point job writes for a pass these points are the keys of.
struct KeyScalars {
  float* scal;       // NULL: none
  const void* val;   // single-channel values (NULL: several channels)
  int64_t bz;
  int dtype, slot;   // of val; slot: its maximum
};

// One array to prepare (grid-stride over `items` by the job's workgroups).
struct PrepJob {
  int kind;
  int width, lg;     // columns of src (D or C); log2 of the row length in items (points, RT values) or of R
  int dtype;         // of src (values)
  int vec;           // 16-byte row loads
  int slot;          // maximum the scale comes from (-1: no scale)
  int flag;          // values KS: signs only
  int64_t n, items;
  const void* src;
  int64_t bz;        // byte stride of src between problems
  uint16_t *out, *out2;
  float* nh;
  KeyScalars ks[2];  // kJobPoints: up to two; kJobSplit: the first; kJobPointsKs: ks[0].val = sign source
};
constexpr int kMaxJobs = 10;

struct PrepArgs {
  unsigned first[kMaxJobs + 1];  // first workgroup of each job; the grid's size from the last job on
  int jobs, nmax;
  float tau2;
  int pitch;
  int qslot, kslot;      // fp32 tier: maxima of the two point sets
  uint32_t* slots;       // the maxima themselves, for the main kernels
  const uint32_t* part;  // partial maxima of k_prep_max
  MaxSource mx[kMaxSlots];
  PrepJob job[kMaxJobs];
};

// The preparation of one launch group in one launch.  F32: the fp32 tier's
// jobs only; else T is the point dtype.  A workgroup first takes the maxima
// its job needs (each from at most kMaxBlock partials of k_prep_max, or from
// the array itself when it is short: see prep_launch), then its share of the
// job's items.  Items of a row are consecutive lanes of one wave and a job's
// item count is a multiple of the wave size, so whole waves run the same
// iterations and the row sums see every lane.
template <typename T, bool F32>
__global__ __launch_bounds__(256) void k_prep(const PrepArgs a, Bz bz) {
  // one row per maximum taken, so that each needs a single barrier
  __shared__ uint32_t wmax[kMaxSlots + 4][256 / kWave];
  int ji = 0;
#pragma unroll
  for (int i = 1; i < kMaxJobs; ++i) ji += blockIdx.x >= a.first[i];
  const PrepJob& J = a.job[ji];
  const unsigned block0 = a.first[ji], block_end = a.first[ji + 1];

  // maximum `slot` of this problem (float bits), by the whole workgroup
  int taken = 0;
  auto maximum = [&](int slot) -> uint32_t {
    for (int i = 0; i < a.nmax; ++i) {
      const MaxSource& s = a.mx[i];
      if (s.slot != slot) continue;
      uint32_t mb = 0;
      if (s.parts > 0) {
        const uint32_t* part = zoff(a.part, bz.ws) + i * a.pitch;
        for (int b = threadIdx.x; b < s.parts; b += 256) mb = umax32(mb, part[b]);
      } else {
        mb = absmax_strided(zoff(s.x, s.bz), s.count, s.dtype, threadIdx.x, 256);
      }
      mb = wave_umax(mb);
      uint32_t* row = wmax[taken++];
      if ((threadIdx.x & (kWave - 1)) == 0) row[threadIdx.x / kWave] = mb;
      __syncthreads();
      for (int w = 0; w < 256 / kWave; ++w) mb = umax32(mb, row[w]);
      return mb;
    }
    return 0u;
  };
  if (blockIdx.x == 0)
    for (int i = 0; i < a.nmax; ++i) {
      const uint32_t mb = maximum(a.mx[i].slot);
      if (threadIdx.x == 0) zoff(a.slots, bz.ws)[a.mx[i].slot] = mb;
    }

  const int64_t stride = (int64_t)(block_end - block0) * 256;
  const int64_t t0 = (int64_t)(blockIdx.x - block0) * 256 + threadIdx.x;
  const int64_t mask = ((int64_t)1 << J.lg) - 1;
  uint16_t* out = zoff(J.out, bz.ws);
  const void* src = zoff(J.src, J.bz);
  if constexpr (F32) {
    uint16_t* out2 = zoff(J.out2, bz.ws);
    if (J.kind == kJobSplit) {
      const int e = scale_exponent(maximum(J.slot)) + kSplitHeadroom;
      const KeyScalars& k = J.ks[0];
      int ev = 0, es = 0;
      if (k.scal) {
        if (k.val) ev = scale_exponent(maximum(k.slot)) - 1;
        es = scale_exponent(maximum(a.qslot)) + scale_exponent(maximum(a.kslot)) + 2 * kSplitHeadroom;
      }
      float* nh = zoff(J.nh, bz.ws);
      float* scal = zoff(k.scal, bz.ws);
      const void* val = zoff(k.val, k.bz);
      for (int64_t t = t0; t < J.items; t += stride) {
        const int64_t r = t >> J.lg;
        const int c = (int)(t & mask);
        const float half = split_item(static_cast<const float*>(src), J.n, J.width, 8 << J.lg, J.lg, e, out, out2,
                                      nh, r, c);
        if (scal && c == 0) key_scalars32(scal, half, val, k.dtype, J.n, r, ev, es, a.tau2);
      }
    } else {
      const int ev = scale_exponent(maximum(J.slot));
      for (int64_t t = t0; t < J.items; t += stride)
        values_ks_split_item(src, J.dtype, J.n, J.width, J.lg, ev, out, out2, t);
    }
  } else {
    const uint16_t* x16 = static_cast<const uint16_t*>(src);
    switch (J.kind) {
      case kJobPoints: {
        float* nh = zoff(J.nh, bz.ws);
        const KeyScalars &k0 = J.ks[0], &k1 = J.ks[1];
        float *scal0 = zoff(k0.scal, bz.ws), *scal1 = zoff(k1.scal, bz.ws);
        const void *val0 = zoff(k0.val, k0.bz), *val1 = zoff(k1.val, k1.bz);
        const float sc0 = scal0 && val0 ? ldexpf(1.0f, scale_exponent(maximum(k0.slot)) - 1) : 0.0f;
        const float sc1 = scal1 && val1 ? ldexpf(1.0f, scale_exponent(maximum(k1.slot)) - 1) : 0.0f;
        for (int64_t t = t0; t < J.items; t += stride) {
          const int64_t r = t >> J.lg;
          const int c = (int)(t & mask);
          const float half = rt_norm_item<T>(x16, J.n, J.width, 8 << J.lg, J.lg, out, nh, J.vec, r, c, r);
          if (scal0 && c == 0) key_scalars(scal0, half, val0, k0.dtype, J.n, r, sc0, a.tau2);
          if (scal1 && c == 1) key_scalars(scal1, half, val1, k1.dtype, J.n, r, sc1, a.tau2);
        }
        break;
      }
      case kJobSample: {
        float* nh = zoff(J.nh, bz.ws);
        for (int64_t t = t0; t < J.items; t += stride) {
          const int64_t r = t >> J.lg;
          (void)rt_norm_item<T>(x16, J.n, J.width, 8 << J.lg, J.lg, out, nh, J.vec, r, (int)(t & mask),
                                sample_row((int)r, J.n));
        }
        break;
      }
      case kJobPointsKs: {
        const float s = J.slot >= 0 ? ldexpf(1.0f, point_scale_exponent(maximum(J.slot))) : 1.0f;
        const void* sgn = zoff(J.ks[0].val, J.ks[0].bz);
        for (int64_t t = t0; t < J.items; t += stride)
          points_ks_item<T>(x16, J.n, J.width, J.lg, s, sgn, J.ks[0].dtype, out, t);
        break;
      }
      case kJobValuesRt: {
        const float s = ldexpf(1.0f, w_scale_exponent(maximum(J.slot), 1 << (J.lg - 2)));
        for (int64_t t = t0; t < J.items; t += stride)
          values_rt_item(src, J.dtype, J.n, J.width, 8 << J.lg, s, out, t >> J.lg, (int)(t & mask));
        break;
      }
      case kJobValuesKs: {
        const float s = ldexpf(1.0f, scale_exponent(maximum(J.slot)));
        for (int64_t t = t0; t < J.items; t += stride)
          values_ks_item(src, J.dtype, J.n, J.width, J.lg, s, J.flag, out, t);
        break;
      }
    }
  }
}

// Inner product sum_m v_m s_m in fp64, fixed order: thread t of workgroup b
// sums the elements b*T + t + k*gridDim*T in index order (T threads), then a
// fixed tree over the workgroup's threads; so the result does not depend on
// timing.  out receives one value per workgroup.
__device__ __forceinline__ void block_tree_sum(double acc, double* red, int threads, double* out) {
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = threads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0];
}

constexpr int kDotThreads = 1024;
#if !defined(GS_PART) || GS_PART == 0  // (kernels that are no templates: in one build part only)
__global__ __launch_bounds__(kDotThreads) void k_dot(const void* __restrict__ v, int dtype, const float* __restrict__ s,
                                                     int64_t n, double* __restrict__ out) {
  __shared__ double red[kDotThreads];
  double acc = 0.0;
  const int64_t stride = (int64_t)gridDim.x * kDotThreads;
  for (int64_t i = (int64_t)blockIdx.x * kDotThreads + threadIdx.x; i < n; i += stride)
    acc += (double)load_any(v, i, dtype) * (double)s[i];
  block_tree_sum(acc, red, kDotThreads, out + blockIdx.x);
}

// Sum of `parts` (at most 256) workgroup partials of k_dot, fixed tree.  One
// thread adding them in index order waited for 256 dependent loads (17 us).
__global__ __launch_bounds__(256) void k_dot_final(const double* __restrict__ part, int parts,
                                                   double* __restrict__ out) {
  __shared__ double red[256];
  block_tree_sum((int)threadIdx.x < parts ? part[threadIdx.x] : 0.0, red, 256, out);
}
#endif

// Split partials of one output: out[i] = sum_s part[s, i] in split order.
struct CombineSeg {
  const float* part;
  float* out;
  int64_t count;
  int64_t bz;       // byte stride of out between problems
};

// One workgroup's share (workgroup `block` of `blocks`) of a segment; four
// elements per thread where count allows 16-byte accesses, the loads of up to
// eight splits issued together before they are added in order.
__device__ __forceinline__ void combine_seg(const float* __restrict__ part, float* __restrict__ out, int64_t count,
                                            int splits, int64_t block, int64_t blocks) {
  int64_t i = block * 256 + threadIdx.x;
  const int64_t stride = blocks * 256;
  if ((count & 3) == 0) {
    // outputs are aligned to their elements only
    typedef float float4_elem __attribute__((ext_vector_type(4), aligned(4)));
    const int64_t c4 = count >> 2;
    const float4* p4 = reinterpret_cast<const float4*>(part);
    for (; i < c4; i += stride) {
      float4 acc = p4[i];
      for (int s0 = 1; s0 < splits; s0 += 8) {
        float4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (s0 + u < splits) v[u] = p4[(int64_t)(s0 + u) * c4 + i];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (s0 + u < splits) {
            acc.x += v[u].x;
            acc.y += v[u].y;
            acc.z += v[u].z;
            acc.w += v[u].w;
          }
      }
      reinterpret_cast<float4_elem*>(out)[i] = float4_elem{acc.x, acc.y, acc.z, acc.w};
    }
    return;
  }
  for (; i < count; i += stride) {
    float acc = part[i];
    for (int s0 = 1; s0 < splits; s0 += 8) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (s0 + u < splits) v[u] = part[(int64_t)(s0 + u) * count + i];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (s0 + u < splits) acc += v[u];
    }
    out[i] = acc;
  }
}

// The split partials of a pass's one or two outputs (a gradient and the
// forward sum it carries) in one launch: workgroups below blocks0 take the
// first.
#if !defined(GS_PART) || GS_PART == 0  // (kernels that are no templates: in one build part only)
__global__ __launch_bounds__(256) void k_combine(CombineSeg a, CombineSeg b, unsigned blocks0, int splits, Bz bz) {
  const bool first = blockIdx.x < blocks0;
  const CombineSeg s = first ? a : b;
  combine_seg(zoff(s.part, bz.ws), zoff(s.out, s.bz), s.count, splits, first ? blockIdx.x : blockIdx.x - blocks0,
              first ? blocks0 : gridDim.x - blocks0);
}
#endif

}  // namespace gs
