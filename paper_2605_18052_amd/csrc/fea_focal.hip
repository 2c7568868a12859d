// Focal-length vote (Method > Focal Length Estimation, Eq. fastmap-focal-vote).
//
// A 3x3 matrix is an essential matrix exactly when its two non-zero singular
// values are equal, so a candidate focal length f is scored by
//   v(f) = sum over pairs of exp((1 - s1/s2) / tau),
// s1 >= s2 the two largest singular values of E = K_j^T F K_i with
// K = diag(f, f, 1) in centred pixel coordinates.  Per intrinsics group g the
// group's cameras take the candidate and every other camera keeps its
// group's current focal length; with one group this is the shared-intrinsics
// vote.  One wave per (run of a group's pairs, 64 candidates): each lane
// holds one candidate and walks the run's pairs in pair order with the rest
// of the wave (the pair's record is the same for every lane and arrives by
// scalar loads), so every lane works and a candidate's sum over the run is a
// plain serial one; the runs' sums are added in order (no atomics).  All in
// fp64; bound by the fp64 instructions of a problem.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "fea_focal.h"
#include "fea_grid.h"

namespace fea {
namespace {

constexpr int kFvThreads = 256;
// A group's pairs are cut into runs only as far as fewer than kFvWaves waves
// (4 on each of the 1,024 SIMDs) would run otherwise, and to no fewer than
// kFvMinRun pairs: past that the runs' partial sums cost more than the waves
// they add.  The votes of 1,000 one-camera groups stay uncut (16,000 waves);
// one group of 5,200 pairs becomes 250 runs.
constexpr int64_t kFvWaves = 4096;
constexpr int64_t kFvMinRun = 8;

// For any rank: s1 / s2 of a 3x3 matrix from the eigenvalues e1 >= e2 >= e3 of M = E^T E:
// with q = tr(M)/3 and p^2 = |M - qI|_F^2 / 6, the eigenvalues of
// B = (M - qI)/p are 2 cos(phi + 2 pi k/3) with cos(3 phi) = det(B)/2.
// Infinite when s2 = 0 (rank below 2).  A function of its own, so that the
// rank-2 forms keep 65 registers and 7 waves per SIMD (inlined: 98 and 4, and
// 72 -> 85 us for the votes of 1,000 cameras), its matrix passed in registers
// (through private memory 408 us for full-rank matrices, now 278; a kernel of
// the cubic alone 290).
__device__ __noinline__ double sv_ratio_full(double x0, double x1, double x2, double x3, double x4, double x5,
                                             double x6, double x7, double x8) {
  const double E[9] = {x0, x1, x2, x3, x4, x5, x6, x7, x8};
  const double m00 = E[0] * E[0] + E[3] * E[3] + E[6] * E[6];
  const double m11 = E[1] * E[1] + E[4] * E[4] + E[7] * E[7];
  const double m22 = E[2] * E[2] + E[5] * E[5] + E[8] * E[8];
  const double m01 = E[0] * E[1] + E[3] * E[4] + E[6] * E[7];
  const double m02 = E[0] * E[2] + E[3] * E[5] + E[6] * E[8];
  const double m12 = E[1] * E[2] + E[4] * E[5] + E[7] * E[8];
  const double q = (m00 + m11 + m22) / 3.0;
  const double a = m00 - q, b = m11 - q, c = m22 - q;
  const double p2 = (a * a + b * b + c * c + 2.0 * (m01 * m01 + m02 * m02 + m12 * m12)) / 6.0;
  if (!(q > 0.0)) return INFINITY;
  if (!(p2 > 0.0)) return 1.0;  // M = qI: all singular values equal
  const double p = sqrt(p2);
  const double det = a * (b * c - m12 * m12) - m01 * (m01 * c - m12 * m02) + m02 * (m01 * m12 - b * m02);
  double r = det / (2.0 * p2 * p);
  r = r < -1.0 ? -1.0 : (r > 1.0 ? 1.0 : r);
  const double phi = acos(r) / 3.0;
  const double e1 = q + 2.0 * p * cos(phi);
  const double e3 = q + 2.0 * p * cos(phi + 2.0943951023931957);  // + 2 pi / 3
  const double e2 = 3.0 * q - e1 - e3;
  if (!(e2 > 0.0)) return INFINITY;
  return sqrt(e1 / e2);
}

// One entry of a group's list, reduced as far as it goes before a candidate
// is known.  A fundamental matrix has rank 2: with the fixed focal lengths
// applied and the candidate's sides at a reference f0 it is E0 = Q B, Q 3x2
// with orthonormal columns, B 2x3, and a candidate f scales the candidate's
// sides by D = diag(g, g, 1), g = f/f0.  With phi = g^2:
//  - one side (E = Q B D; for the other side E0 is transposed first): s1^2
//    and s2^2 are the eigenvalues of S = B D^2 B^T = phi P + R, a symmetric
//    2x2 matrix, and det S = phi (phi c2 + c1) with c2, c1 sums of squared
//    minors of B (Cauchy-Binet: no cancellation);
//  - both sides (E = D Q B D): those of G H, G = Q^T D^2 Q, H = B D^2 B^T,
//    or of the symmetric L^T H L with G = L L^T, here times G00 so that no
//    root is taken.
// Then d = s1^2 - s2^2 = sqrt((S00 - S11)^2 + 4 S01^2) and
// s1/s2 = (S00 + S11 + d) / (2 sqrt(det S)).  Nothing small is formed from
// large terms that nearly cancel: s1/s2 - 1 comes out to ~1e-15, where the
// cubic's closed form fixes it to ~1e-8 near s1 = s2.  A matrix of full
// rank, or with focal lengths beyond what these products carry, keeps the
// cubic.
enum : int { kFvOneSide = 0, kFvBothSides = 1, kFvFull = 2 };

struct FvEntry {
  // one side: P00 P01 P11 R00 R01 R11 c2 c1; both sides: the same of H, then
  // of G; full rank: F with the fixed focal lengths applied
  double v[16];
  int32_t kind, cand_i, cand_j, pad;
};

__device__ __forceinline__ double dot3(const double* a, const double* b) { return a[0] * b[0] + a[1] * b[1] + a[2] * b[2]; }

// The eight coefficients of B D^2 B^T and its determinant from the rows of B.
__device__ void form_coeffs(const double* b0, const double* b1, double* v) {
  v[0] = b0[0] * b0[0] + b0[1] * b0[1];
  v[1] = b0[0] * b1[0] + b0[1] * b1[1];
  v[2] = b1[0] * b1[0] + b1[1] * b1[1];
  v[3] = b0[2] * b0[2];
  v[4] = b0[2] * b1[2];
  v[5] = b1[2] * b1[2];
  const double m01 = b0[0] * b1[1] - b0[1] * b1[0];
  const double m02 = b0[0] * b1[2] - b0[2] * b1[0], m12 = b0[1] * b1[2] - b0[2] * b1[1];
  v[6] = m01 * m01;
  v[7] = m02 * m02 + m12 * m12;
}

__global__ __launch_bounds__(kFvThreads) void k_fv_entries(int64_t n_entries, const int32_t* __restrict__ ent_group,
                                                           const int32_t* __restrict__ ent_pair,
                                                           const int32_t* __restrict__ pair_i,
                                                           const int32_t* __restrict__ pair_j,
                                                           const int32_t* __restrict__ group,
                                                           const double* __restrict__ F,
                                                           const double* __restrict__ f_cur, double f0,
                                                           FvEntry* __restrict__ ent) {
  const int64_t e = (int64_t)blockIdx.x * kFvThreads + threadIdx.x;
  if (e >= n_entries) return;
  const int p = ent_pair[e], g = ent_group[e];
  const int gi = group[pair_i[p]], gj = group[pair_j[p]];
  const bool ci = gi == g, cj = gj == g;
  const double fi = ci ? 1.0 : f_cur[gi], fj = cj ? 1.0 : f_cur[gj];
  const double si[3] = {fi, fi, 1.0}, sj[3] = {fj, fj, 1.0};
  FvEntry r;
  for (int k = 0; k < 16; ++k) r.v[k] = 0.0;
  r.kind = kFvFull;
  r.cand_i = ci;
  r.cand_j = cj;
  r.pad = 0;
  // F may come at any scale; brought near 1 by a power of two, which changes no
  // bit of a ratio (the cubic's products go to the sixth order in F)
  double top = 0.0;
  for (int k = 0; k < 9; ++k) top = fmax(top, fabs(F[9 * (int64_t)p + k]));
  const int ex = top > 0.0 ? -ilogb(top) : 0;
  double E[9];  // columns of E0 (of its transpose when only side j takes the candidate), at f0
  for (int k = 0; k < 3; ++k)
    for (int c = 0; c < 3; ++c) {
      const double x = sj[k] * ldexp(F[9 * (int64_t)p + 3 * k + c], ex) * si[c];
      r.v[3 * k + c] = x;
      const double y = x * (cj && k < 2 ? f0 : 1.0) * (ci && c < 2 ? f0 : 1.0);
      E[ci ? 3 * c + k : 3 * k + c] = y;
    }
  double nrm = 0.0;
  for (int k = 0; k < 9; ++k) nrm += E[k] * E[k];
  // f0 = 0: the candidates' range rules the reduced forms out
  if (f0 > 0.0 && nrm > 1e-200 && nrm < 1e200) {
    const double inv = 1.0 / sqrt(nrm);
    for (int k = 0; k < 9; ++k) E[k] *= inv;
    // Q by Gram-Schmidt: the largest column, then the largest remainder
    // (projected twice), and the third direction to see the rank
    int c0 = 0;
    double n0 = dot3(E, E);
    for (int c = 1; c < 3; ++c) {
      const double n = dot3(E + 3 * c, E + 3 * c);
      if (n > n0) {
        n0 = n;
        c0 = c;
      }
    }
    double q0[3], q1[3] = {0.0, 0.0, 0.0}, q2[3];
    const double i0 = 1.0 / sqrt(n0);
    for (int k = 0; k < 3; ++k) q0[k] = E[3 * c0 + k] * i0;
    double n1 = 0.0;
    for (int c = 0; c < 3; ++c) {
      if (c == c0) continue;
      double u[3] = {E[3 * c], E[3 * c + 1], E[3 * c + 2]};
      for (int rep = 0; rep < 2; ++rep) {
        const double d = dot3(q0, u);
        for (int k = 0; k < 3; ++k) u[k] -= d * q0[k];
      }
      const double n = dot3(u, u);
      if (n > n1) {
        n1 = n;
        for (int k = 0; k < 3; ++k) q1[k] = u[k];
      }
    }
    if (n1 > 1e-20) {  // s2/s1 above ~1e-10
      const double i1 = 1.0 / sqrt(n1);
      for (int k = 0; k < 3; ++k) q1[k] *= i1;
      q2[0] = q0[1] * q1[2] - q0[2] * q1[1];
      q2[1] = q0[2] * q1[0] - q0[0] * q1[2];
      q2[2] = q0[0] * q1[1] - q0[1] * q1[0];
      double b0[3], b1[3], b2[3];
      for (int c = 0; c < 3; ++c) {
        b0[c] = dot3(q0, E + 3 * c);
        b1[c] = dot3(q1, E + 3 * c);
        b2[c] = dot3(q2, E + 3 * c);
      }
      if (dot3(b2, b2) < 1e-28 * n1) {  // s3/s2 below ~1e-14: rank 2 to rounding
        r.kind = ci && cj ? kFvBothSides : kFvOneSide;
        form_coeffs(b0, b1, r.v);
        if (ci && cj) form_coeffs(q0, q1, r.v + 8);
      }
    }
  }
  ent[e] = r;
}

// 1/sqrt(x) and sqrt(x) of a positive normal x: the hardware's reciprocal
// root with one coupled Newton step and a last residual step each (within an
// ulp or two; the general forms rescale their argument, twice the work).
__device__ __forceinline__ double fast_rsqrt(double x) {
  double y = __builtin_amdgcn_rsq(x);
  double e = fma(-x * y, y, 1.0);
  y = fma(y * e, fma(e, 0.375, 0.5), y);
  e = fma(-x * y, y, 1.0);
  return fma(0.5 * y, e, y);
}
__device__ __forceinline__ double fast_sqrt(double x) {
  const double y = fast_rsqrt(x);
  const double g = x * y;
  return fma(0.5 * y, fma(-g, g, x), g);
}

// One wave per (work item, 64 candidates); an item is a run of one group's
// entries.  partial[item][k] = the run's votes for candidate k.  Bound by
// fp64 instructions: ~75 a problem on one side, 25 of them the exponential's
// (the cubic with acos and two cosines took ~540).  Measured, kernel alone:
// 1,000 cameras, 10,600 pairs, a group per camera, 1,024 candidates 299 ->
// 74 us; 5,200 pairs in one group 6,865 -> 31.5 us, most of it because the
// group's list is cut into runs (one list per group left 16 waves).
__global__ __launch_bounds__(kFvThreads) void k_fv_vote(int n_items, int n_cand, const int2* __restrict__ items,
                                                        const FvEntry* __restrict__ ent,
                                                        const double* __restrict__ cand, double inv_tau, double inv_f0,
                                                        double* __restrict__ partial) {
  const int lane = threadIdx.x & 63;
  const int nb = (n_cand + 63) >> 6;
  // uniform over the wave: the entries arrive by scalar loads
  const int64_t w = (int64_t)blockIdx.x * (kFvThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (w >= (int64_t)n_items * nb) return;
  const int it = (int)(w / nb), k = (int)(w - (int64_t)it * nb) * 64 + lane;
  const double f = cand[k < n_cand ? k : n_cand - 1];
  const double phi = (f * inv_f0) * (f * inv_f0);
  const int2 run = items[it];
  double s = 0.0;
  for (int e = run.x; e < run.y; ++e) {
    const FvEntry& r = ent[e];
    const double* v = r.v;
    double ratio;
    if (r.kind == kFvOneSide) {
      const double a = fma(phi, v[0], v[3]), b = fma(phi, v[1], v[4]), c = fma(phi, v[2], v[5]);
      const double det = phi * fma(phi, v[6], v[7]);
      const double d = fast_sqrt(fmax(fma(4.0 * b, b, (a - c) * (a - c)), 1e-290));
      ratio = 0.5 * (a + c + d) * fast_rsqrt(det);
    } else if (r.kind == kFvBothSides) {
      const double h00 = fma(phi, v[0], v[3]), h01 = fma(phi, v[1], v[4]), h11 = fma(phi, v[2], v[5]);
      const double dh = phi * fma(phi, v[6], v[7]);
      const double g00 = fma(phi, v[8], v[11]), g01 = fma(phi, v[9], v[12]);
      const double dg = phi * fma(phi, v[14], v[15]);
      const double u = fma(g00, h01, g01 * h11);              // (G H)_01
      const double a = fma(g00, fma(g00, h00, g01 * h01), g01 * u);  // G00 (L^T H L)_00
      const double c = dg * h11;
      const double d = fast_sqrt(fmax(fma(4.0 * dg, u * u, (a - c) * (a - c)), 1e-290));
      ratio = 0.5 * (a + c + d) * fast_rsqrt(dg * dh * g00 * g00);
    } else {
      const double fi = r.cand_i ? f : 1.0, fj = r.cand_j ? f : 1.0;
      ratio = sv_ratio_full(v[0] * fj * fi, v[1] * fj * fi, v[2] * fj, v[3] * fj * fi, v[4] * fj * fi, v[5] * fj,
                            v[6] * fi, v[7] * fi, v[8]);
    }
    s += exp((1.0 - ratio) * inv_tau);
  }
  if (k < n_cand) partial[(int64_t)it * n_cand + k] = s;
}

// votes[g][k] = the partials of group g's items, 16 waves each adding rows
// q, q + 16, ... and the 16 sums added in order (a fixed order: no atomics).
constexpr int kFvSumWaves = 16;
__global__ __launch_bounds__(64 * kFvSumWaves) void k_fv_sum(int n_cand, const int32_t* __restrict__ grp_item_off,
                                                             const double* __restrict__ partial,
                                                             double* __restrict__ votes) {
  __shared__ double red[kFvSumWaves][64];
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int nb = (n_cand + 63) >> 6;
  const int g = blockIdx.x / nb, k = (blockIdx.x - g * nb) * 64 + lane;
  double s = 0.0;
  if (k < n_cand)
    for (int it = grp_item_off[g] + q; it < grp_item_off[g + 1]; it += kFvSumWaves) s += partial[(int64_t)it * n_cand + k];
  red[q][lane] = s;
  __syncthreads();
  if (q == 0 && k < n_cand) {
    double t = 0.0;
#pragma unroll
    for (int r = 0; r < kFvSumWaves; ++r) t += red[r][lane];
    votes[(int64_t)g * n_cand + k] = t;
  }
}

// Per group: the candidate with the highest vote (ties: the lower index).
__global__ __launch_bounds__(kFvThreads) void k_fv_best(int n_cand, const double* __restrict__ votes,
                                                        const double* __restrict__ cand, double* __restrict__ f_best,
                                                        int32_t* __restrict__ k_best) {
  __shared__ double sv[kFvThreads];
  __shared__ int si[kFvThreads];
  const double* v = votes + (int64_t)blockIdx.x * n_cand;
  double bv = 0.0;
  int bk = -1;
  for (int k = threadIdx.x; k < n_cand; k += kFvThreads)
    if (bk < 0 || v[k] > bv) {
      bv = v[k];
      bk = k;
    }
  sv[threadIdx.x] = bv;
  si[threadIdx.x] = bk;
  __syncthreads();
  for (int s = kFvThreads / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      const int k2 = si[threadIdx.x + s], k1 = si[threadIdx.x];
      const double v2 = sv[threadIdx.x + s];
      if (k2 >= 0 && (k1 < 0 || v2 > sv[threadIdx.x] || (v2 == sv[threadIdx.x] && k2 < k1))) {
        sv[threadIdx.x] = v2;
        si[threadIdx.x] = k2;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    f_best[blockIdx.x] = cand[si[0]];
    k_best[blockIdx.x] = si[0];
  }
}

}  // namespace

size_t fv_entry_bytes() { return sizeof(FvEntry); }

int fv_items_chunk(int64_t n_entries, int n_cand) {
  const int64_t nb = (n_cand + 63) / 64;
  return (int)std::max<int64_t>(kFvMinRun, (n_entries * nb + kFvWaves - 1) / kFvWaves);
}

hipError_t launch_fv_vote(hipStream_t st, int n_groups, int n_items, int64_t n_entries, int n_cand,
                          const int32_t* ent_group, const int32_t* ent_pair, const int2* items,
                          const int32_t* grp_item_off, const int32_t* pair_i, const int32_t* pair_j,
                          const int32_t* group, const double* F, const double* f_cur, const double* cand, double f0,
                          double tau, void* ent, double* partial, double* votes, hipEvent_t ev0, hipEvent_t ev1) {
  const int64_t nb = (n_cand + 63) / 64;
  FvEntry* fe = static_cast<FvEntry*>(ent);
  k_fv_entries<<<(unsigned)((n_entries + kFvThreads - 1) / kFvThreads), kFvThreads, 0, st>>>(
      n_entries, ent_group, ent_pair, pair_i, pair_j, group, F, f_cur, f0, fe);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  double* out = n_items == n_groups ? votes : partial;
  const double inv_f0 = f0 > 0.0 ? 1.0 / f0 : 1.0;
  // slices of the items, and of the groups below, that a grid holds
  constexpr int kWaves = kFvThreads / 64;
  const int64_t most = std::max<int64_t>(grid_rows(1, kFvThreads) * kWaves / nb, 1);
  for (int64_t i = 0; i < n_items; i += most) {
    const int n = (int)std::min<int64_t>(most, n_items - i);
    const dim3 grid((unsigned)((n * nb + kWaves - 1) / kWaves)), block(kFvThreads);
    if (ev0)
      hipExtLaunchKernelGGL(k_fv_vote, grid, block, 0, st, i == 0 ? ev0 : nullptr, i + n == n_items ? ev1 : nullptr, 0,
                            n, n_cand, items + i, fe, cand, 1.0 / tau, inv_f0, out + i * n_cand);
    else
      k_fv_vote<<<grid, block, 0, st>>>(n, n_cand, items + i, fe, cand, 1.0 / tau, inv_f0, out + i * n_cand);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (n_items == n_groups) return e;
  const int64_t most_groups = grid_rows(nb, 64 * kFvSumWaves);
  for (int64_t g = 0; g < n_groups && e == hipSuccess; g += most_groups) {
    const int64_t n = std::min<int64_t>(most_groups, n_groups - g);
    k_fv_sum<<<(unsigned)(n * nb), 64 * kFvSumWaves, 0, st>>>(n_cand, grp_item_off + g, partial, votes + g * n_cand);
    e = hipGetLastError();
  }
  return e;
}

hipError_t launch_fv_best(hipStream_t st, int n_groups, int n_cand, const double* votes, const double* cand,
                          double* f_best, int32_t* k_best) {
  k_fv_best<<<n_groups, kFvThreads, 0, st>>>(n_cand, votes, cand, f_best, k_best);
  return hipGetLastError();
}

}  // namespace fea
