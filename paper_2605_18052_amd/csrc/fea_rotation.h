// Global rotation (Method > Global Rotation): kernels and launchers in
// fea_rotation.hip.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "fea_trans.h"  // TaCounters: the Adam step counters

namespace fea {

// The pair graph as the kernels read it (device arrays): per camera its
// entries (2 * pair + side, side 1 = the pair's second camera), each entry's
// other camera, and the relative rotations in entry order (launch_ra_entries).
struct LzGraph {
  int n_cams;
  const int32_t *cam_off, *cam_ent, *ent_other;
  const double* Rent;
};
hipError_t launch_ra_entries(hipStream_t st, int n_cams, const int32_t* cam_off, const int32_t* cam_ent,
                             const double* Rrel, double* Rent);

// A Lanczos step j on A = wm M + wp diag(c1 c1^T) (c1 nullable: wp unused),
// in two parts.  launch_lz_apply: w = A V_j; where lz_fused_next(n), for
// j > 0 it first completes step j - 1 from that step's vector w_prev (V_j,
// alpha[j-1] = its coefficient on V_{j-1}, beta[j-1] = |w_prev|).
// launch_lz_orthogonalise: w orthogonalised twice against V_0..V_j (and, where
// not fused, the step completed).  launch_lz_finish completes step j without
// another step (V_{j+1}, alpha[j], beta[j]).  V holds (j+2) * n doubles,
// n = 3 n_cams; h1/h2 j+1, part lz_orth_blocks(n) scratch.
int lz_orth_blocks(int64_t n);
bool lz_fused_next(int64_t n);
hipError_t launch_lz_apply(hipStream_t st, const LzGraph& g, const double* c1, double wm, double wp, double* V, int j,
                           double* w_prev, double* w, double* h1, double* h2, double* part, double* alpha,
                           double* beta);
hipError_t launch_lz_orthogonalise(hipStream_t st, int64_t n, double* V, int j, double* w, double* h1, double* h2,
                                   double* part, double* alpha, double* beta);
hipError_t launch_lz_finish(hipStream_t st, int64_t n, double* V, int j, double* w, double* h1, double* h2,
                            double* part, double* alpha, double* beta);
// y = sum over i < m of s[i] V_i.
hipError_t launch_lz_combine(hipStream_t st, int64_t n, int m, const double* V, const double* s, double* y);
hipError_t launch_ra_columns(hipStream_t st, int n_cams, const double* c, const double* c1, double* out,
                             int32_t* err);
hipError_t launch_ra_step(hipStream_t st, const LzGraph& g, int64_t n_pairs, const double* a_in, double* a_out,
                          double* m, double* v, TaCounters* ctr, int parity, double beta1, double beta2, double eps,
                          double decay);
// dist: n_pairs doubles of scratch.
hipError_t launch_ra_loss(hipStream_t st, int64_t n_pairs, const int32_t* pair_i, const int32_t* pair_j,
                          const double* Rrel, const double* a6, double* dist, double* loss);
hipError_t launch_ra_to_R(hipStream_t st, int n_cams, const double* a6, double* R);

}  // namespace fea
