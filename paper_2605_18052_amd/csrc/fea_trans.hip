// Global Translation (Method > Global Translation).
//
// Relative translations.  With the global rotations fixed, each pair's unit
// relative translation u is chosen among candidate directions by the mean
// epipolar error of the pair's matches, eps(u) = x~2^T [u]x R_ij x~1.  By the
// scalar triple product eps(u) = u . n with n = (R_ij x~1) x x~2, so a pair
// with M matches and K candidates is the product of an M x 3 and a 3 x K
// matrix followed by |.| and a sum over M: a dense contraction of depth 3.
// It runs on the matrix cores, n computed once per match into LDS and |D|
// accumulated per lane in fp32: in large searches with both factors split into
// bf16 parts that carry fp32's 24 bits between them, the candidates that come
// out lowest scored once more with fp32 products (v_mfma_f32_16x16x4f32) and the
// choice made among those; else with fp32 products throughout (rt_split).  A
// direction and its opposite score the same; the sign comes from a cheirality
// vote (both triangulated depths positive) over the pair's matches.
//
// Camera centres.  The L1 direction loss of
// Eq. fastmap-global-translation-objective is minimised with Adam, one thread
// per (run, camera) wave: the lanes split the camera's pair terms and a fixed
// wave sum adds them (no atomics: the same order at every step), then the
// Adam step.  Several runs from independent random initial centres
// share each launch; they are aligned (centred, unit mean norm) and merged per
// camera by its mean pair loss (Multiple initializations), then the merged
// centres get a final loop.  Everything here is fp64: the work is O(pairs)
// per step and latency-bound.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <tuple>

#include "fea_device.h"
#include "fea_grid.h"
#include "fea_trans.h"

namespace fea {
namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int kRtThreads = 256;
constexpr int kRtLds = kRtItem + 32;              // LDS row stride (floats): a block past the last is readable
constexpr int kRtLds32 = kRtItem + 16;            // the same of fp32 products; rows land 16 banks apart
constexpr int kTaThreads = 256;

// ---- relative translations ---------------------------------------------------

// Per pair: R_ij = R_j R_i^T with the focal lengths and principal points, in
// fp32 for the scoring and fp64 for the vote.
__global__ void k_rt_pairs(int64_t n_pairs, const int32_t* __restrict__ pair_i, const int32_t* __restrict__ pair_j,
                           const double* __restrict__ R, const double* __restrict__ f,
                           const double* __restrict__ cx, const double* __restrict__ cy, float* __restrict__ rowf,
                           double* __restrict__ rowd) {
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= n_pairs) return;
  const int i = pair_i[n], j = pair_j[n];
  const double* Ri = R + 9 * (int64_t)i;
  const double* Rj = R + 9 * (int64_t)j;
  double row[kRtRow];
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b)
      row[3 * a + b] = Rj[3 * a] * Ri[3 * b] + Rj[3 * a + 1] * Ri[3 * b + 1] + Rj[3 * a + 2] * Ri[3 * b + 2];
  row[9] = f[i];
  row[10] = f[j];
  row[11] = cx[i];
  row[12] = cy[i];
  row[13] = cx[j];
  row[14] = cy[j];
  row[15] = 0.0;
  for (int k = 0; k < kRtRow; ++k) {
    rowd[kRtRow * n + k] = row[k];
    rowf[kRtRow * n + k] = (float)row[k];
  }
  rowf[kRtRow * n + 9] = (float)(1.0 / row[9]);
  rowf[kRtRow * n + 10] = (float)(1.0 / row[10]);
}

// A match's n = (R_ij x~1) x x~2 in fp32, x~2 = (b0, b1, 1).  The roundings
// are spelled out: the scoring and the second scoring of the lowest
// candidates form the same bits.
struct RtPair {
  float R[9], ifi, ifj, cxi, cyi, cxj, cyj;
  __device__ __forceinline__ explicit RtPair(const float* __restrict__ row) {
#pragma unroll
    for (int k = 0; k < 9; ++k) R[k] = row[k];
    ifi = row[9];
    ifj = row[10];
    cxi = row[11];
    cyi = row[12];
    cxj = row[13];
    cyj = row[14];
  }
  __device__ __forceinline__ void normal(float x1, float y1, float x2, float y2, float (&n)[3]) const {
    const float a0 = (x1 - cxi) * ifi, a1 = (y1 - cyi) * ifi;
    const float b0 = (x2 - cxj) * ifj, b1 = (y2 - cyj) * ifj;
    const float r0 = fmaf(R[0], a0, R[1] * a1) + R[2];
    const float r1 = fmaf(R[3], a0, R[4] * a1) + R[5];
    const float r2 = fmaf(R[6], a0, R[7] * a1) + R[8];
    n[0] = fmaf(-b1, r2, r1);
    n[1] = fmaf(b0, r2, -r0);
    n[2] = fmaf(b1, r0, -(b0 * r1));
  }
};

// x rounded to bf16 in both halves of a register.
__device__ __forceinline__ unsigned bf16_twice(float x) {
  return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){x, x}, bf16x2));
}

// fp32 x = h + m + l in bf16 parts (8 bits of the significand each).  The dot
// product of a match's (l l h m h m h m) and a candidate's (h m l l m m h h)
// is the product of the two but for l l, 2^-32 of it.
struct Bf16Parts {
  unsigned hm, ll, hh, mm;  // pairs of parts, the first in the low half
  __device__ __forceinline__ explicit Bf16Parts(float x) {
    hh = bf16_twice(x);
    const float r1 = x - __uint_as_float(hh & 0xffff0000u);
    mm = bf16_twice(r1);
    ll = bf16_twice(r1 - __uint_as_float(mm & 0xffff0000u));
    hm = (hh & 0xffffu) | (mm & 0xffff0000u);
  }
  __device__ __forceinline__ bf16x8 candidate() const {
    return __builtin_bit_cast(bf16x8, (u32x4){hm, ll, mm, hh});
  }
};
__device__ __forceinline__ bf16x8 match_operand(unsigned hm, unsigned ll) {
  return __builtin_bit_cast(bf16x8, (u32x4){ll, hm, hm, hm});
}

// Sums of kRtGroup candidates over one work item.  MFMA 32x32x16 (bf16): lane
// l supplies 8 contraction slots of match l%32 (A) and of candidate l%32 (B),
// the parts of one component: component l/32 in the first product, 2 (lanes
// 0-31; the others zero) in the second, which adds to it; the lane receives
// candidate l%32 at 16 of the 32 matches.  With CAP every product enters as
// min(|d|, tau) (one v_med3_f32 clamp each, the absolute value folded into
// the adds), else as |d| (folded into the adds).
//
// Bound by the vector unit: 8 instructions (32 cycles) per 256 products with
// the cap, beside 16 cycles of matrix unit; issue of the two overlaps only in
// part.  fp32 products (16x16x4, 32 cycles per 256, a quarter of its depth
// unused) held the vector unit up longer: the inner loop alone took 62.9
// cycles per 256 products, against 41.0 (capped) and 33.1 (plain) in this
// form; with 16x16x32 products 46.6, with 256 candidates per wave 86
// (registers).  30M matches, 2,048 candidates, cap 8 px: 5,971 -> 4,400 us.
// The sums' error against fp64 is not above the fp32 products' (relative,
// norm over all scores: 7.1e-8 for 1.8e-7 capped at 8 px, 4.8e-8 for 5.2e-8
// uncapped).
template <bool CAP>
__global__ __launch_bounds__(kRtThreads) void k_rt_score(const int4* __restrict__ items, int n_groups,
                                                         const float* __restrict__ rowf,
                                                         const float* __restrict__ x1, const float* __restrict__ y1,
                                                         const float* __restrict__ x2, const float* __restrict__ y2,
                                                         const float* __restrict__ cand, int n_cand, int kp, float tau,
                                                         float* __restrict__ partial, float* __restrict__ item_abs) {
  __shared__ unsigned s_hm[3][kRtLds], s_ll[3][kRtLds];  // n's parts
  __shared__ float s_abs[kRtThreads / 64];
  const int it = blockIdx.x / n_groups;
  const int grp = blockIdx.x - it * n_groups;
  const int4 rec = items[it];  // {pair, layout start, count, -}
  const int cnt = rec.z;
  const int nblk = (cnt + 31) >> 5;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  {
    const RtPair pr(rowf + (int64_t)kRtRow * rec.x);
    float sum = 0.f;
    for (int m = threadIdx.x; m < (nblk << 5); m += kRtThreads) {
      float n[3] = {0.f, 0.f, 0.f};
      if (m < cnt) {
        const int64_t s = (int64_t)rec.y + m;
        pr.normal(x1[s], y1[s], x2[s], y2[s], n);
      }
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const Bf16Parts p(n[k]);
        s_hm[k][m] = p.hm;
        s_ll[k][m] = p.ll;
      }
      sum += (__builtin_fabsf(n[0]) + __builtin_fabsf(n[1])) + __builtin_fabsf(n[2]);
    }
    if (grp == 0) {
      sum = wave_sum_f32(sum);
      if (lane == 0) s_abs[wave] = sum;
    }
  }
  __syncthreads();
  if (grp == 0 && threadIdx.x == 0) item_abs[it] = (s_abs[0] + s_abs[1]) + (s_abs[2] + s_abs[3]);

  const int hf = lane >> 5, col = lane & 31;
  const int cbase = grp * kRtGroup + wave * kRtWave;
  if (cbase >= n_cand) return;  // the whole wave: nothing but padding
  bf16x8 b01[kRtBlocks], b2[kRtBlocks];
#pragma unroll
  for (int q = 0; q < kRtBlocks; ++q) {
    const int k = cbase + 32 * q + col;
    b01[q] = Bf16Parts(cand[(int64_t)hf * kp + k]).candidate();
    b2[q] = Bf16Parts(hf ? 0.f : cand[(int64_t)2 * kp + k]).candidate();
  }
  float accf[kRtBlocks];
  double acc2[kRtBlocks];
#pragma unroll
  for (int q = 0; q < kRtBlocks; ++q) {
    accf[q] = 0.f;
    acc2[q] = 0.0;
  }
  const float ntau = -tau;
  // the rows of the next block are read while this one's products run (the
  // read past the last block stays inside the LDS row); in the second product
  // lanes 32-63 meet candidate parts of zero
  unsigned hm01 = s_hm[hf][col], ll01 = s_ll[hf][col], hm2 = s_hm[2][col], ll2 = s_ll[2][col];
  for (int mb = 0; mb < nblk; ++mb) {
    const bf16x8 a01 = match_operand(hm01, ll01), a2 = match_operand(hm2, ll2);
    const int nx = ((mb + 1) << 5) + col;
    hm01 = s_hm[hf][nx];
    ll01 = s_ll[hf][nx];
    hm2 = s_hm[2][nx];
    ll2 = s_ll[2][nx];
#pragma unroll
    for (int q = 0; q < kRtBlocks; ++q) {
      f32x16 d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a01, b01[q], (f32x16){}, 0, 0, 0);
      d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a2, b2[q], d, 0, 0, 0);
      float c[16];
      // |clamp(e, -tau, tau)| = min(|e|, tau): one v_med3 per product, the
      // absolute value rides on the add as a source modifier (fminf would
      // add a canonicalising max before every min)
#pragma unroll
      for (int r = 0; r < 16; ++r) c[r] = __builtin_fabsf(CAP ? __builtin_amdgcn_fmed3f(d[r], ntau, tau) : d[r]);
#pragma unroll
      for (int w = 8; w >= 1; w >>= 1)
#pragma unroll
        for (int r = 0; r < w; ++r) c[r] = c[2 * r] + c[2 * r + 1];
      accf[q] += c[0];
    }
    if ((mb & 7) == 7) {  // lane sums of at most 128 terms in fp32, those in fp64
#pragma unroll
      for (int q = 0; q < kRtBlocks; ++q) {
        acc2[q] += (double)accf[q];
        accf[q] = 0.f;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < kRtBlocks; ++q) {
    double s = acc2[q] + (double)accf[q];
    s += __shfl_xor(s, 32);
    if (hf == 0) partial[(int64_t)it * kp + cbase + 32 * q + col] = (float)s;
  }
}

// Four products of one candidate, capped or not, added.
__device__ __forceinline__ float rt_four(const f32x4 d, bool cap, float ntau, float tau) {
  if (cap) {
    const float c0 = __builtin_amdgcn_fmed3f(d[0], ntau, tau), c1 = __builtin_amdgcn_fmed3f(d[1], ntau, tau);
    const float c2 = __builtin_amdgcn_fmed3f(d[2], ntau, tau), c3 = __builtin_amdgcn_fmed3f(d[3], ntau, tau);
    return (__builtin_fabsf(c0) + __builtin_fabsf(c1)) + (__builtin_fabsf(c2) + __builtin_fabsf(c3));
  }
  return (__builtin_fabsf(d[0]) + __builtin_fabsf(d[1])) + (__builtin_fabsf(d[2]) + __builtin_fabsf(d[3]));
}

// The same with fp32 products, kRtGroup32 candidates over one work item, for
// the calls that rt_split leaves to them.  MFMA 16x16x4: lane l supplies
// component l/16 of match l%16 of the block (A) and of candidate l%16 (B),
// component 3 zero, and receives candidate l%16 at four matches.  Sums of at
// most 128 terms per lane in fp32, then at most 4 of those.
template <bool CAP>
__global__ __launch_bounds__(kRtThreads) void k_rt_score32(const int4* __restrict__ items, int n_groups,
                                                           const float* __restrict__ rowf,
                                                           const float* __restrict__ x1, const float* __restrict__ y1,
                                                           const float* __restrict__ x2, const float* __restrict__ y2,
                                                           const float* __restrict__ cand, int n_cand, int kp,
                                                           float tau, float* __restrict__ partial) {
  __shared__ float sn[3][kRtLds32];
  const int it = blockIdx.x / n_groups;
  const int grp = blockIdx.x - it * n_groups;
  const int4 rec = items[it];  // {pair, layout start, count, -}
  const int cnt = rec.z;
  const int nblk = (cnt + 15) >> 4;
  {
    const RtPair pr(rowf + (int64_t)kRtRow * rec.x);
    for (int m = threadIdx.x; m < (nblk << 4); m += kRtThreads) {
      float n[3] = {0.f, 0.f, 0.f};
      if (m < cnt) {
        const int64_t s = (int64_t)rec.y + m;
        pr.normal(x1[s], y1[s], x2[s], y2[s], n);
      }
#pragma unroll
      for (int k = 0; k < 3; ++k) sn[k][m] = n[k];
    }
  }
  __syncthreads();

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int kq = lane >> 4, col = lane & 15;
  const int cbase = grp * kRtGroup32 + wave * kRtWave32;
  if (cbase >= n_cand) return;  // the whole wave: nothing but padding
  float bop[kRtBlocks32];
#pragma unroll
  for (int q = 0; q < kRtBlocks32; ++q) bop[q] = kq < 3 ? cand[(int64_t)kq * kp + cbase + 16 * q + col] : 0.f;
  float accf[kRtBlocks32], acc2[kRtBlocks32];
#pragma unroll
  for (int q = 0; q < kRtBlocks32; ++q) {
    accf[q] = 0.f;
    acc2[q] = 0.f;
  }
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  const float ntau = -tau;
  // the row of the next block is read while this one's products run (the
  // read past the last block stays inside the LDS row)
  const float* srow = sn[kq < 3 ? kq : 0];
  float a_next = srow[col];
  for (int mb = 0; mb < nblk; ++mb) {
    const float a = kq < 3 ? a_next : 0.f;
    a_next = srow[((mb + 1) << 4) + col];
#pragma unroll
    for (int q = 0; q < kRtBlocks32; ++q) {
      const f32x4 d = __builtin_amdgcn_mfma_f32_16x16x4f32(a, bop[q], zero, 0, 0, 0);
      accf[q] += rt_four(d, CAP, ntau, tau);
    }
    if ((mb & 31) == 31) {
#pragma unroll
      for (int q = 0; q < kRtBlocks32; ++q) {
        acc2[q] += accf[q];
        accf[q] = 0.f;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < kRtBlocks32; ++q) {
    double s = (double)acc2[q] + (double)accf[q];
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    if (kq == 0) partial[(int64_t)it * kp + cbase + 16 * q + col] = (float)s;
  }
}

// Part of a candidate's (capped) sum over a run of matches with fp32
// products, one candidate per column, by one wave: kRtSeg blocks of 16
// matches from block mb0 on.  MFMA 16x16x4: lane l supplies component l/16
// of match l%16 and u = component l/16 of the column's candidate (component 3
// zero) and receives candidate l%16 at four matches.  The order of the sum is
// fixed, so it does not depend on the column or the wave.
constexpr int kRtSeg = 32;     // 128 terms per lane
constexpr int kRtRun = 2048;   // matches whose sum is rounded to fp32: kRtWaves segments
constexpr int kRtWaves = kRtThreads / 64;
static_assert(kRtRun == kRtWaves * kRtSeg * 16, "one segment of a run per wave");
__device__ float rt_segment_sum(const RtPair& pr, int64_t start, int cnt, int mb0, float u, bool cap, float tau,
                                int lane, float (*sn)[64], const float* __restrict__ x1,
                                const float* __restrict__ y1, const float* __restrict__ x2,
                                const float* __restrict__ y2) {
  const int kq = lane >> 4, col = lane & 15;
  const int nblk = min((cnt + 15) >> 4, mb0 + kRtSeg);
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  const float ntau = -tau;
  float acc = 0.f;
  // four blocks at a time: a match per lane, its n through the wave's rows
  // sn [4][64] in LDS (the fourth zero) to the lanes that supply it
  float q0 = 0.f, q1 = 0.f, q2 = 0.f, q3 = 0.f;
  auto load = [&](int mb) {
    const int64_t s = start + min((mb << 4) + lane, cnt - 1);
    q0 = x1[s];
    q1 = y1[s];
    q2 = x2[s];
    q3 = y2[s];
  };
  if (mb0 < nblk) load(mb0);
  for (int mb = mb0; mb < nblk; mb += 4) {
    float n[3];
    pr.normal(q0, q1, q2, q3, n);
    load(mb + 4);  // the next four blocks' coordinates, in flight meanwhile (clamped to the run)
    const bool in = (mb << 4) + lane < cnt;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();  // the rows' last reads come before
#pragma unroll
    for (int k = 0; k < 3; ++k) sn[k][lane] = in ? n[k] : 0.f;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    float a[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) a[b] = sn[kq][(b << 4) + col];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const f32x4 d = __builtin_amdgcn_mfma_f32_16x16x4f32(a[b], u, zero, 0, 0, 0);
      if (mb + b >= nblk) break;  // uniform
      acc += rt_four(d, cap, ntau, tau);
    }
  }
  return acc;
}

// Depth signs of one match for the translation direction u (camera j frame):
// the depths of the least-squares two-view triangulation
// l2 x~2 = l1 R_ij x~1 + u have the signs of -(a.u)(b.b) + (a.b)(b.u) and
// (a.a)(b.u) - (a.b)(a.u), a = R_ij x~1, b = x~2 (the determinant
// |a x b|^2 is positive unless the rays are parallel).
__device__ int cheirality_vote(const double* row, float fx1, float fy1, float fx2, float fy2, const double u[3],
                               double tau) {
  const double ax = ((double)fx1 - row[11]) / row[9], ay = ((double)fy1 - row[12]) / row[9];
  const double bx = ((double)fx2 - row[13]) / row[10], by = ((double)fy2 - row[14]) / row[10];
  const double a0 = row[0] * ax + row[1] * ay + row[2];
  const double a1 = row[3] * ax + row[4] * ay + row[5];
  const double a2 = row[6] * ax + row[7] * ay + row[8];
  // eps(u) = u . (a x b): only matches the chosen direction explains vote
  const double e = u[0] * (a1 - a2 * by) + u[1] * (a2 * bx - a0) + u[2] * (a0 * by - a1 * bx);
  if (!(fabs(e) < tau)) return 0;
  const double aa = a0 * a0 + a1 * a1 + a2 * a2, bb = bx * bx + by * by + 1.0;
  const double ab = a0 * bx + a1 * by + a2;
  const double au = a0 * u[0] + a1 * u[1] + a2 * u[2], bu = bx * u[0] + by * u[1] + u[2];
  const double det = aa * bb - ab * ab;
  if (!(det > 0.0)) return 0;
  const double l1 = -au * bb + ab * bu, l2 = aa * bu - ab * au;
  if (l1 > 0.0 && l2 > 0.0) return 1;
  if (l1 < 0.0 && l2 < 0.0) return -1;
  return 0;
}

// Per pair: mean score of every candidate (sum of the item partials over the
// pair's match count); the candidates whose mean may be the lowest in fp32
// arithmetic scored again with fp32 products (rt_segment_sum); of those the
// lowest (ties: lower index); then the vote of the matches with |eps| < tau
// at that direction.
//
// A product of the split parts is within 70 * 2^-24 |n|_1 of the fp32 one
// (|u| components at most 1; 24 terms added in fp32 against 3, and l l), the
// cap brings them no further apart, and the lane sums round by at most 200
// * 2^-24 of the score between both forms; so a candidate whose mean is more
// than twice that bound above the lowest mean cannot be the lowest one: of
// 2,048 a few remain, and the choice and its score are those of fp32
// products throughout.  Anything not finite leaves every candidate in.
// 10,600 pairs of 2,800 matches: 213 us with the vote alone, 367 us with the
// second scoring.
//
// SPLIT false: the sums are those of fp32 products, and the lowest is taken.
constexpr int kRtChunk = 1024;  // candidates looked through at a time
template <bool SPLIT>
__global__ __launch_bounds__(kRtThreads) void k_rt_select(int k_cand, int kp, double tau,
                                                          const int32_t* __restrict__ pair_item_off,
                                                          const int4* __restrict__ items,
                                                          const float* __restrict__ partial,
                                                          const float* __restrict__ item_abs,
                                                          const float* __restrict__ cand,
                                                          const float* __restrict__ rowf,
                                                          const double* __restrict__ rowd,
                                                          const float* __restrict__ x1, const float* __restrict__ y1,
                                                          const float* __restrict__ x2, const float* __restrict__ y2,
                                                          float* __restrict__ scores, int32_t* __restrict__ best,
                                                          int32_t* __restrict__ vote, double* __restrict__ t_rel,
                                                          double* __restrict__ score_best) {
  __shared__ double sv[kRtThreads];
  __shared__ int si[kRtThreads];
  const int tid = threadIdx.x;
  const int64_t n = blockIdx.x;
  const int i0 = pair_item_off[n], i1 = pair_item_off[n + 1];
  const int64_t start = items[i0].y;  // the pair's items are one run of the layout
  int cnt = 0;
  double abs1 = 0.0;
  for (int it = i0; it < i1; ++it) {
    cnt += items[it].z;
    if (SPLIT) abs1 += (double)item_abs[it];
  }
  auto mean_of = [&](int k) {
    double s = 0.0;
    for (int it = i0; it < i1; ++it) s += (double)partial[(int64_t)it * kp + k];
    return s / (double)cnt;
  };
  double bv = 0.0;
  int bk = -1;
  if constexpr (!SPLIT) {
    for (int k = tid; k < k_cand; k += kRtThreads) {
      const double mean = mean_of(k);
      if (scores) scores[n * k_cand + k] = (float)mean;
      if (bk < 0 || mean < bv) {
        bv = mean;
        bk = k;
      }
    }
  } else {
    __shared__ int s_list[kRtChunk];      // contenders of the chunk
    __shared__ double s_mean[kRtChunk];   // and their means in fp32 arithmetic
    __shared__ int s_slot[kRtChunk];      // candidate of the chunk -> its place in the list, -1 when ruled out
    __shared__ float s_seg[kRtWaves][64];
    __shared__ float s_rows[kRtWaves][4][64];
    __shared__ int s_n;
    const int lane = tid & 63, wave = tid >> 6;
    double lo = INFINITY;
    bool odd = false;
    for (int k = tid; k < k_cand; k += kRtThreads) {
      const double mean = mean_of(k);
      if (scores) scores[n * k_cand + k] = (float)mean;
      if (mean < lo) lo = mean;
      odd = odd || !isfinite(mean);
    }
    sv[tid] = lo;
    __syncthreads();
    for (int s = kRtThreads / 2; s > 0; s >>= 1) {
      if (tid < s && sv[tid + s] < sv[tid]) sv[tid] = sv[tid + s];
      __syncthreads();
    }
    const double low = sv[0];
    s_rows[wave][3][lane] = 0.f;
    __syncthreads();
    const double limit = low + 2.0 * 0x1p-24 * (70.0 * (abs1 / (double)cnt) + 200.0 * low);
    const bool none = !odd && lo > limit;  // none of this thread's candidates remains
    const RtPair pr(rowf + (int64_t)kRtRow * n);
    const bool cap = !isinf(tau);
    const float tauf = cap ? (float)tau : 0.f;
    for (int c0 = 0; c0 < k_cand; c0 += kRtChunk) {
      if (tid == 0) s_n = 0;
      __syncthreads();
      const int ce = min(c0 + kRtChunk, k_cand);
      for (int k = c0 + tid; k < ce; k += kRtThreads) {
        int slot = -1;
        if (!none && !(mean_of(k) > limit)) {
          slot = atomicAdd(&s_n, 1);
          s_list[slot] = k;
          s_mean[slot] = 0.0;
        }
        s_slot[k - c0] = slot;
      }
      __syncthreads();
      const int nc = s_n;
      for (int b = 0; b < nc; b += 16) {
        // 16 contenders at a time over runs of kRtRun matches, a segment per
        // wave: the full segments' lane sums are added in order, then the
        // last, shorter one's and the lanes' in fp64
        const int kq = lane >> 4, mine = b + (lane & 15);
        const float u = kq < 3 && mine < nc ? cand[(int64_t)kq * kp + s_list[mine]] : 0.f;
        for (int m0 = 0; m0 < cnt; m0 += kRtRun) {
          const int rc = min(kRtRun, cnt - m0), nblk = (rc + 15) >> 4;
          s_seg[wave][lane] =
              rt_segment_sum(pr, start + m0, rc, wave * kRtSeg, u, cap, tauf, lane, s_rows[wave], x1, y1, x2, y2);
          __syncthreads();
          if (wave == 0) {
            float acc2 = 0.f;
            const int full = nblk / kRtSeg;
            for (int w = 0; w < full; ++w) acc2 += s_seg[w][lane];
            const float accf = full < kRtWaves ? s_seg[full][lane] : 0.f;
            double s = (double)acc2 + (double)accf;
            s += __shfl_xor(s, 16);
            s += __shfl_xor(s, 32);
            if (lane < 16 && mine < nc) s_mean[mine] += (double)(float)s;
          }
          __syncthreads();
        }
      }
      for (int k = c0 + tid; k < ce; k += kRtThreads) {
        const int slot = s_slot[k - c0];
        if (slot < 0) continue;
        const double mean = s_mean[slot] / (double)cnt;
        if (scores) scores[n * k_cand + k] = (float)mean;
        if (bk < 0 || mean < bv) {
          bv = mean;
          bk = k;
        }
      }
      __syncthreads();
    }
  }
  sv[tid] = bv;
  si[tid] = bk;
  __syncthreads();
  for (int s = kRtThreads / 2; s > 0; s >>= 1) {
    if (tid < s) {
      const double v2 = sv[tid + s];
      const int k2 = si[tid + s];
      const int k1 = si[tid];
      if (k2 >= 0 && (k1 < 0 || v2 < sv[tid] || (v2 == sv[tid] && k2 < k1))) {
        sv[tid] = v2;
        si[tid] = k2;
      }
    }
    __syncthreads();
  }
  const int kb = si[0];
  const double vb = sv[0];
  const double u[3] = {(double)cand[kb], (double)cand[kp + kb], (double)cand[2 * kp + kb]};
  const double* row = rowd + (int64_t)kRtRow * n;
  int v = 0;
  for (int m = tid; m < cnt; m += kRtThreads) {
    const int64_t s = start + m;
    v += cheirality_vote(row, x1[s], y1[s], x2[s], y2[s], u, tau);
  }
  __syncthreads();
  si[threadIdx.x] = v;
  __syncthreads();
  for (int s = kRtThreads / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) si[threadIdx.x] += si[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const int vs = si[0];
    const double sg = vs >= 0 ? 1.0 : -1.0;
    best[n] = kb;
    vote[n] = vs;
    score_best[n] = vb;
    for (int k = 0; k < 3; ++k) t_rel[3 * n + k] = sg * u[k];
  }
}

// ---- camera centres -------------------------------------------------------------

__device__ __forceinline__ double sgn(double x) { return x > 0.0 ? 1.0 : (x < 0.0 ? -1.0 : 0.0); }

// o^{i->j} = -R_j^T t^{i->j} / |t^{i->j}|
__global__ void k_ta_targets(int64_t n_pairs, const int32_t* __restrict__ pair_j, const double* __restrict__ R,
                             const double* __restrict__ t_rel, double* __restrict__ target) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n_pairs) return;
  const double* t = t_rel + 3 * p;
  const double nt = sqrt(t[0] * t[0] + t[1] * t[1] + t[2] * t[2]);
  const double u[3] = {t[0] / nt, t[1] / nt, t[2] / nt};
  const double* Rj = R + 9 * (int64_t)pair_j[p];
  for (int k = 0; k < 3; ++k) target[3 * p + k] = -(Rj[k] * u[0] + Rj[3 + k] * u[1] + Rj[6 + k] * u[2]);
}

__global__ void k_ta_counters(TaCounters* ctr, double lr) {
  ctr->lr[0] = ctr->lr[1] = lr;
  ctr->b1t[0] = ctr->b1t[1] = 1.0;
  ctr->b2t[0] = ctr->b2t[1] = 1.0;
}

// The targets in the order the cameras' entries are read: camera c's block
// starts at 3 off[c] and holds entry k of its deg at [coordinate][k], and the
// entries themselves as {2 * pair + side, other camera}.
__global__ __launch_bounds__(kTaThreads) void k_ta_entries(int n_cams, const int32_t* __restrict__ cam_off,
                                                           const int32_t* __restrict__ cam_ent,
                                                           const int32_t* __restrict__ ent_other,
                                                           const double* __restrict__ target,
                                                           int2* __restrict__ ent2, double* __restrict__ tgt) {
  const int lane = threadIdx.x & 63;
  const int c = blockIdx.x * (kTaThreads / 64) + (threadIdx.x >> 6);
  if (c >= n_cams) return;
  const int e0 = cam_off[c], deg = cam_off[c + 1] - e0;
  double* out = tgt + 3 * (int64_t)e0;
  for (int k = lane; k < deg; k += 64) {
    const int ent = cam_ent[e0 + k];
    ent2[e0 + k] = make_int2(ent, ent_other[e0 + k]);
    for (int a = 0; a < 3; ++a) out[(int64_t)a * deg + k] = target[3 * (int64_t)(ent >> 1) + a];
  }
}

// One wave per (camera, run = blockIdx.y): the lanes split the camera's pair
// terms (s - n (n.s)) / |d| with s = sign(n - o^{i->j}) / |P|, added for j and
// subtracted for i; a fixed-order wave sum; lanes 0-2 take the Adam step of
// x, y, z.  A chain of dependent loads (the camera's range, its entries, the
// other cameras' centres) and fp64 roots: the camera is uniform over the
// wave, so its own data arrives by scalar loads, and two trips' entries are
// in flight together.  500 cameras of 125 pairs, 2 runs, 2,000 steps: 10.3 ->
// 8.6-9.0 ms.
__global__ __launch_bounds__(kTaThreads) void k_ta_step(int n_cams, int64_t n_pairs,
                                                        const int32_t* __restrict__ cam_off,
                                                        const int2* __restrict__ ent2,
                                                        const double* __restrict__ tgt,
                                                        const double* __restrict__ o_in, double* __restrict__ o_out,
                                                        double* __restrict__ m, double* __restrict__ v,
                                                        TaCounters* ctr, int p, double beta1, double beta2,
                                                        double eps, double decay) {
  const int lane = threadIdx.x & 63;
  const int c = blockIdx.x * (kTaThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const double lr = ctr->lr[p];
  const double b1t = ctr->b1t[p] * beta1, b2t = ctr->b2t[p] * beta2;
  if (c == 0 && blockIdx.y == 0 && lane == 0) {  // the other parity's slot: read by the next step only
    ctr->lr[p ^ 1] = lr * decay;
    ctr->b1t[p ^ 1] = b1t;
    ctr->b2t[p ^ 1] = b2t;
  }
  if (c >= n_cams) return;
  const int64_t base = (int64_t)blockIdx.y * n_cams * 3;
  const double* __restrict__ o = o_in + base;
  const int e0 = cam_off[c], deg = cam_off[c + 1] - e0;
  const int2* __restrict__ ec = ent2 + e0;
  const double* __restrict__ tc = tgt + 3 * (int64_t)e0;
  const double inv_np = 1.0 / (double)n_pairs;
  double g0 = 0.0, g1 = 0.0, g2 = 0.0;
  const double oc0 = o[3 * c], oc1 = o[3 * c + 1], oc2 = o[3 * c + 2];
  // the optimiser state of this camera's coordinate (lanes 0..2), loaded
  // before the pair loop so that it arrives meanwhile
  const int64_t a = base + 3 * c + (lane < 3 ? lane : 0);
  double m_old = 0.0, v_old = 0.0, o_old = 0.0;
  if (lane < 3) {
    m_old = m[a];
    v_old = v[a];
    o_old = o_in[a];
  }
  for (int k0 = lane; k0 < deg; k0 += 128) {
    int ent[2];
    double x[2][3], t[2][3];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int k = min(k0 + 64 * u, deg - 1);
      const int2 en = ec[k];
      ent[u] = en.x;
      for (int b = 0; b < 3; ++b) {
        t[u][b] = tc[(int64_t)b * deg + k];
        x[u][b] = o[3 * en.y + b];
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (k0 + 64 * u >= deg) break;
      // d = o_j - o_i; this camera is j of the pair when the entry is odd
      const bool cj = ent[u] & 1;
      const double x0 = x[u][0], x1 = x[u][1], x2 = x[u][2];
      const double d0 = cj ? oc0 - x0 : x0 - oc0, d1 = cj ? oc1 - x1 : x1 - oc1, d2 = cj ? oc2 - x2 : x2 - oc2;
      const double nd = sqrt(d0 * d0 + d1 * d1 + d2 * d2);
      if (!(nd > 0.0)) continue;
      const double inv = 1.0 / nd;
      const double n0 = d0 * inv, n1 = d1 * inv, n2 = d2 * inv;
      const double s0 = sgn(n0 - t[u][0]) * inv_np, s1 = sgn(n1 - t[u][1]) * inv_np, s2 = sgn(n2 - t[u][2]) * inv_np;
      const double ns = n0 * s0 + n1 * s1 + n2 * s2;
      const double sd = cj ? inv : -inv;
      g0 += (s0 - n0 * ns) * sd;
      g1 += (s1 - n1 * ns) * sd;
      g2 += (s2 - n2 * ns) * sd;
    }
  }
  double g[3] = {g0, g1, g2};
  wave_sum_f64_scatter(g);
  if (lane < 3) {
    const double gk = lane == 0 ? g[0] : (lane == 1 ? g[1] : g[2]);
    const double mk = beta1 * m_old + (1.0 - beta1) * gk;
    const double vk = beta2 * v_old + (1.0 - beta2) * gk * gk;
    m[a] = mk;
    v[a] = vk;
    const double mh = mk / (1.0 - b1t), vh = vk / (1.0 - b2t);
    o_out[a] = o_old - lr * mh / (sqrt(vh) + eps);
  }
}

// One workgroup per run: centre at the origin, rescale to unit mean norm.
__global__ __launch_bounds__(kTaThreads) void k_ta_align(int n_cams, double* __restrict__ o_all,
                                                         int32_t* __restrict__ err) {
  __shared__ double red[3][kTaThreads];
  double* o = o_all + (int64_t)blockIdx.x * n_cams * 3;
  double s0 = 0.0, s1 = 0.0, s2 = 0.0;
  for (int i = threadIdx.x; i < n_cams; i += kTaThreads) {
    s0 += o[3 * i];
    s1 += o[3 * i + 1];
    s2 += o[3 * i + 2];
  }
  red[0][threadIdx.x] = s0;
  red[1][threadIdx.x] = s1;
  red[2][threadIdx.x] = s2;
  __syncthreads();
  for (int s = kTaThreads / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s)
      for (int k = 0; k < 3; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + s];
    __syncthreads();
  }
  const double c0 = red[0][0] / n_cams, c1 = red[1][0] / n_cams, c2 = red[2][0] / n_cams;
  __syncthreads();
  double sn = 0.0;
  for (int i = threadIdx.x; i < n_cams; i += kTaThreads) {
    const double d0 = o[3 * i] - c0, d1 = o[3 * i + 1] - c1, d2 = o[3 * i + 2] - c2;
    sn += sqrt(d0 * d0 + d1 * d1 + d2 * d2);
  }
  red[0][threadIdx.x] = sn;
  __syncthreads();
  for (int s = kTaThreads / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[0][threadIdx.x] += red[0][threadIdx.x + s];
    __syncthreads();
  }
  const double scale = red[0][0] / n_cams;
  if (!(scale > 0.0)) {
    if (threadIdx.x == 0) *err = 1;
    return;
  }
  for (int i = threadIdx.x; i < n_cams; i += kTaThreads) {
    o[3 * i] = (o[3 * i] - c0) / scale;
    o[3 * i + 1] = (o[3 * i + 1] - c1) / scale;
    o[3 * i + 2] = (o[3 * i + 2] - c2) / scale;
  }
}

// L1 term of every (run, pair).
__global__ void k_ta_pair_loss(int runs, int n_cams, int64_t n_pairs, const int32_t* __restrict__ pair_i,
                               const int32_t* __restrict__ pair_j, const double* __restrict__ target,
                               const double* __restrict__ o_all, double* __restrict__ pair_loss) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)runs * n_pairs) return;
  const int64_t r = idx / n_pairs, q = idx - r * n_pairs;
  const double* o = o_all + r * n_cams * 3;
  const int i = pair_i[q], j = pair_j[q];
  const double d0 = o[3 * j] - o[3 * i], d1 = o[3 * j + 1] - o[3 * i + 1], d2 = o[3 * j + 2] - o[3 * i + 2];
  const double nd = sqrt(d0 * d0 + d1 * d1 + d2 * d2);
  double l = 0.0;
  if (nd > 0.0) {
    l += fabs(d0 / nd - target[3 * q]);
    l += fabs(d1 / nd - target[3 * q + 1]);
    l += fabs(d2 / nd - target[3 * q + 2]);
  }
  pair_loss[idx] = l;
}

// Mean pair loss of every (camera, run = blockIdx.y), summed in pair order: a
// wave loads 64 terms at a time and adds them one after another (one thread
// walking the list took 68 us for 500 cameras of 125 pairs, now 6).
__global__ __launch_bounds__(kTaThreads) void k_ta_cam_loss(int n_cams, int64_t n_pairs,
                                                            const int32_t* __restrict__ cam_off,
                                                            const int32_t* __restrict__ cam_ent,
                                                            const double* __restrict__ pair_loss,
                                                            double* __restrict__ cam_loss) {
  const int lane = threadIdx.x & 63;
  const int c = blockIdx.x * (kTaThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (c >= n_cams) return;
  const double* __restrict__ pl = pair_loss + (int64_t)blockIdx.y * n_pairs;
  const int e0 = cam_off[c], deg = cam_off[c + 1] - e0;
  double s = 0.0;
  for (int k = 0; k < deg; k += 64)
    s = wave_serial_sum(s, k + lane < deg ? pl[cam_ent[e0 + k + lane] >> 1] : 0.0, min(64, deg - k));
  if (lane == 0) cam_loss[(int64_t)blockIdx.y * n_cams + c] = deg ? s / (double)deg : 0.0;
}

// One workgroup per run: L_t = sum of the pair terms / |P|.
__global__ __launch_bounds__(kTaThreads) void k_ta_run_loss(int64_t n_pairs, const double* __restrict__ pair_loss,
                                                            double* __restrict__ run_loss) {
  __shared__ double red[kTaThreads];
  const double* pl = pair_loss + (int64_t)blockIdx.x * n_pairs;
  double s = 0.0;
#pragma unroll 8
  for (int64_t q = threadIdx.x; q < n_pairs; q += kTaThreads) s += pl[q];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int k = kTaThreads / 2; k > 0; k >>= 1) {
    if (threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) run_loss[blockIdx.x] = n_pairs > 0 ? red[0] / (double)n_pairs : 0.0;
}

// Per camera: the run with the lowest mean loss (ties: the lower run).
__global__ void k_ta_merge(int runs, int n_cams, const double* __restrict__ o_runs,
                           const double* __restrict__ cam_loss, double* __restrict__ o_out,
                           int32_t* __restrict__ run_of_cam) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n_cams) return;
  int b = 0;
  for (int r = 1; r < runs; ++r)
    if (cam_loss[(int64_t)r * n_cams + c] < cam_loss[(int64_t)b * n_cams + c]) b = r;
  run_of_cam[c] = b;
  for (int k = 0; k < 3; ++k) o_out[3 * c + k] = o_runs[((int64_t)b * n_cams + c) * 3 + k];
}

unsigned blocks_for(int64_t n, int threads) { return (unsigned)((n + threads - 1) / threads); }

}  // namespace

hipError_t launch_rt_pairs(hipStream_t st, int64_t n_pairs, const int32_t* pair_i, const int32_t* pair_j,
                           const double* R, const double* f, const double* cx, const double* cy, float* rowf,
                           double* rowd) {
  if (n_pairs == 0) return hipSuccess;
  k_rt_pairs<<<blocks_for(n_pairs, 256), 256, 0, st>>>(n_pairs, pair_i, pair_j, R, f, cx, cy, rowf, rowd);
  return hipGetLastError();
}

// Split products save products' time and cost the second scoring.  The
// former, per (match, candidate): 98 fs with fp32 products, padded to a wave's
// 256 candidates, 74 with split ones, to 128 (30M matches, 2,048 candidates:
// 5.97 and 4.4 ms); and 23 ns per match of the longest item, the chain that a
// small call waits for (28 pairs of 2,800 matches 117 and 73 us).  The latter,
// in a pair's workgroup: 1.3 us per chunk of candidates and 4.4 us per run of
// kRtRun matches (a segment's part of it where the run is shorter), more with
// the contenders that many candidates leave; all of it in sequence for the
// longest pair, some 768 workgroups' worth at once over all pairs.  So fp32
// products are for a few long pairs (one of 3M matches: 7.0 and 13.3 ms), many
// candidates of few matches (4M of 14,000: 34 and 43.7 ms) and pairs of a few
// dozen matches (1,225 of 50: 72 and 75 us).  Over 1 to 1,225 pairs of 50 to
// 60,000 matches and 1 to 8,192 candidates the choice is within 4% of the
// better one.
//
// A cap below 2e-3 (1 px at 500 px) takes fp32 products too: a mean's error
// bound grows with |n|, its spread over the candidates with the cap's square,
// and where one reaches the other every candidate is scored twice (2,000
// outlier pairs of 20,000 matches, 2,048 candidates, at a cap of 2e-3 8.5 ms
// either way, at 1.4e-3 8.5 with fp32 products and 25.7 split).
bool rt_split(int64_t n_pairs, int64_t n_matches, int64_t longest, int n_cand, double tau) {
  if (!(tau >= 2e-3)) return false;
  const double P = (double)n_pairs, M = (double)n_matches, L = (double)longest;
  const auto padded = [&](int unit) { return (double)((n_cand + unit - 1) / unit * (int64_t)unit); };
  const double saved = M * (98e-15 * padded(kRtWave32) - 74e-15 * padded(kRtWave)) + 23e-9 * std::min(L, (double)kRtItem);
  const double chunks = 1.3e-6 * (double)((n_cand + kRtChunk - 1) / kRtChunk);
  const double run = 4.4e-6 * (1.0 + n_cand / 16384.0);
  const double segment = (double)kRtRun / kRtWaves, full = std::floor(L / kRtRun);
  const double one = chunks + run * (full + std::min((L - full * kRtRun) / segment, 1.0));
  const double all = (P * chunks + run * std::min(P + M / kRtRun, M / segment)) / 768;
  return saved > std::max(one, all);
}

// `kernel` over the items, in slices that a grid holds, from item `first` on
// with the rest of its arguments shifted by `shifted(first)`.
template <class... Params, class Shift>
hipError_t launch_rt_slices(hipStream_t st, void (*kernel)(Params...), int64_t n_items, int n_groups, hipEvent_t ev0,
                            hipEvent_t ev1, Shift shifted) {
  const dim3 block(kRtThreads);
  const int64_t most = grid_rows(n_groups, kRtThreads);
  hipError_t e = hipSuccess;
  for (int64_t i = 0; i < n_items && e == hipSuccess; i += most) {
    const int64_t n = std::min(most, n_items - i);
    const dim3 grid((unsigned)(n * n_groups));
    std::apply(
        [&](auto... a) {
          if (ev0)
            hipExtLaunchKernelGGL(kernel, grid, block, 0, st, i == 0 ? ev0 : nullptr, i + n == n_items ? ev1 : nullptr,
                                  0, a...);
          else
            kernel<<<grid, block, 0, st>>>(a...);
        },
        shifted(i));
    e = hipGetLastError();
  }
  return e;
}

hipError_t launch_rt_score(hipStream_t st, bool split, int64_t n_items, int n_groups, const int4* items,
                           const float* rowf, const float* x1, const float* y1, const float* x2, const float* y2,
                           const float* cand, int n_cand, int kp, double tau, float* partial, float* item_abs,
                           hipEvent_t ev0, hipEvent_t ev1) {
  const bool cap = !std::isinf(tau);
  const float tauf = cap ? (float)tau : 0.f;
  if (split)
    return launch_rt_slices(st, cap ? k_rt_score<true> : k_rt_score<false>, n_items, n_groups, ev0, ev1,
                            [&](int64_t i) {
                              return std::make_tuple(items + i, n_groups, rowf, x1, y1, x2, y2, cand, n_cand, kp, tauf,
                                                     partial + i * kp, item_abs + i);
                            });
  return launch_rt_slices(st, cap ? k_rt_score32<true> : k_rt_score32<false>, n_items, n_groups, ev0, ev1,
                          [&](int64_t i) {
                            return std::make_tuple(items + i, n_groups, rowf, x1, y1, x2, y2, cand, n_cand, kp, tauf,
                                                   partial + i * kp);
                          });
}

hipError_t launch_rt_select(hipStream_t st, bool split, int64_t n_pairs, int k, int kp, double tau,
                            const int32_t* pair_item_off, const int4* items, const float* partial,
                            const float* item_abs, const float* cand, const float* rowf, const double* rowd,
                            const float* x1, const float* y1, const float* x2, const float* y2, float* scores,
                            int32_t* best, int32_t* vote, double* t_rel, double* score_best) {
  if (n_pairs == 0) return hipSuccess;
  const auto kernel = split ? k_rt_select<true> : k_rt_select<false>;
  kernel<<<(unsigned)n_pairs, kRtThreads, 0, st>>>(k, kp, tau, pair_item_off, items, partial, item_abs, cand, rowf,
                                                   rowd, x1, y1, x2, y2, scores, best, vote, t_rel, score_best);
  return hipGetLastError();
}

hipError_t launch_ta_targets(hipStream_t st, int64_t n_pairs, const int32_t* pair_j, const double* R,
                             const double* t_rel, double* target) {
  if (n_pairs == 0) return hipSuccess;
  k_ta_targets<<<blocks_for(n_pairs, 256), 256, 0, st>>>(n_pairs, pair_j, R, t_rel, target);
  return hipGetLastError();
}

hipError_t launch_ta_counters(hipStream_t st, TaCounters* ctr, double lr) {
  k_ta_counters<<<1, 1, 0, st>>>(ctr, lr);
  return hipGetLastError();
}

hipError_t launch_ta_entries(hipStream_t st, int n_cams, const int32_t* cam_off, const int32_t* cam_ent,
                             const int32_t* ent_other, const double* target, int2* ent2, double* tgt) {
  k_ta_entries<<<blocks_for(n_cams, kTaThreads / 64), kTaThreads, 0, st>>>(n_cams, cam_off, cam_ent, ent_other, target,
                                                                           ent2, tgt);
  return hipGetLastError();
}

hipError_t launch_ta_step(hipStream_t st, int runs, int n_cams, int64_t n_pairs, const int32_t* cam_off,
                          const int2* ent2, const double* tgt, const double* o_in, double* o_out, double* m, double* v,
                          TaCounters* ctr, int parity, double beta1, double beta2, double eps, double decay) {
  k_ta_step<<<dim3(blocks_for(n_cams, kTaThreads / 64), runs), kTaThreads, 0, st>>>(
      n_cams, n_pairs, cam_off, ent2, tgt, o_in, o_out, m, v, ctr, parity, beta1, beta2, eps, decay);
  return hipGetLastError();
}

hipError_t launch_ta_align(hipStream_t st, int runs, int n_cams, double* o, int32_t* err) {
  k_ta_align<<<runs, kTaThreads, 0, st>>>(n_cams, o, err);
  return hipGetLastError();
}

hipError_t launch_ta_losses(hipStream_t st, int runs, int n_cams, int64_t n_pairs, const int32_t* cam_off,
                            const int32_t* cam_ent, const int32_t* pair_i, const int32_t* pair_j,
                            const double* target, const double* o, double* pair_loss, double* cam_loss,
                            double* run_loss) {
  if (n_pairs > 0)
    k_ta_pair_loss<<<blocks_for((int64_t)runs * n_pairs, 256), 256, 0, st>>>(runs, n_cams, n_pairs, pair_i, pair_j,
                                                                             target, o, pair_loss);
  if (cam_loss)
    k_ta_cam_loss<<<dim3(blocks_for(n_cams, kTaThreads / 64), runs), kTaThreads, 0, st>>>(
        n_cams, n_pairs, cam_off, cam_ent, pair_loss, cam_loss);
  k_ta_run_loss<<<runs, kTaThreads, 0, st>>>(n_pairs, pair_loss, run_loss);
  return hipGetLastError();
}

hipError_t launch_ta_merge(hipStream_t st, int runs, int n_cams, const double* o_runs, const double* cam_loss,
                           double* o_out, int32_t* run_of_cam) {
  k_ta_merge<<<blocks_for(n_cams, 256), 256, 0, st>>>(runs, n_cams, o_runs, cam_loss, o_out, run_of_cam);
  return hipGetLastError();
}

}  // namespace fea
