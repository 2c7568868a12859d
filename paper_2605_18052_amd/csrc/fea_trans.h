// Global Translation stages (Method > Global Translation): the
// relative-translation candidate search and the camera-centre alignment with
// multiple random initialisations.  Kernels and launchers in fea_trans.hip.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace fea {

// Candidate search: one scoring workgroup covers one work item (a run of at
// most kRtItem matches of one pair) and a group of candidates.  Split products
// (bf16 parts): a pair is cut into equal runs, kRtGroup candidates (4 waves x
// kRtBlocks blocks of 32).  Items of 1,536 (four workgroups per CU instead of
// three) took 2% less time for the scoring, and as much more for the sums of
// the additional items.  fp32 products: runs of kRtItem, kRtGroup32 candidates
// (4 waves x kRtBlocks32 blocks of 16).
constexpr int kRtItem = 2048;
constexpr int kRtBlocks = 4;
constexpr int kRtWave = kRtBlocks * 32;  // candidates of one wave
constexpr int kRtGroup = 4 * kRtWave;
constexpr int kRtBlocks32 = 16;
constexpr int kRtWave32 = kRtBlocks32 * 16;
constexpr int kRtGroup32 = 4 * kRtWave32;
constexpr int kRtRow = 16;  // per-pair row: R_ij (9), 1/f_i, 1/f_j, cx_i, cy_i, cx_j, cy_j, pad

// Adam state shared by all cameras of one alignment phase, one slot per step
// parity: the learning rate of the step and the running powers of the betas.
struct TaCounters {
  double lr[2];
  double b1t[2];
  double b2t[2];
};

hipError_t launch_rt_pairs(hipStream_t st, int64_t n_pairs, const int32_t* pair_i, const int32_t* pair_j,
                           const double* R, const double* f, const double* cx, const double* cy, float* rowf,
                           double* rowd);
// Whether a search of n_matches in n_pairs (the longest with `longest`) takes
// split products or fp32 ones; tau in normalised units.
bool rt_split(int64_t n_pairs, int64_t n_matches, int64_t longest, int n_cand, double tau);
// partial [n_items * kp]: every candidate's (capped) sum over the item, kp the
// candidates rounded up to a wave's.  Split
// products also leave item_abs [n_items]: the sum of |n|_1 over the item's
// matches, which bounds how far those sums are from fp32 products' (see
// launch_rt_select).
hipError_t launch_rt_score(hipStream_t st, bool split, int64_t n_items, int n_groups, const int4* items,
                           const float* rowf, const float* x1, const float* y1, const float* x2, const float* y2,
                           const float* cand, int n_cand, int kp, double tau, float* partial, float* item_abs,
                           hipEvent_t ev0, hipEvent_t ev1);
// Per pair: the mean scores; of split products the candidates within the sums'
// error bound of the lowest scored again with fp32 products; the lowest of
// those, its vote.
hipError_t launch_rt_select(hipStream_t st, bool split, int64_t n_pairs, int k, int kp, double tau,
                            const int32_t* pair_item_off, const int4* items, const float* partial,
                            const float* item_abs, const float* cand, const float* rowf, const double* rowd,
                            const float* x1, const float* y1, const float* x2, const float* y2, float* scores,
                            int32_t* best, int32_t* vote, double* t_rel, double* score_best);

hipError_t launch_ta_targets(hipStream_t st, int64_t n_pairs, const int32_t* pair_j, const double* R,
                             const double* t_rel, double* target);
hipError_t launch_ta_counters(hipStream_t st, TaCounters* ctr, double lr);
// The entries and targets in the order launch_ta_step reads them: ent2
// [2 n_pairs], tgt [6 n_pairs].
hipError_t launch_ta_entries(hipStream_t st, int n_cams, const int32_t* cam_off, const int32_t* cam_ent,
                             const int32_t* ent_other, const double* target, int2* ent2, double* tgt);
hipError_t launch_ta_step(hipStream_t st, int runs, int n_cams, int64_t n_pairs, const int32_t* cam_off,
                          const int2* ent2, const double* tgt, const double* o_in, double* o_out, double* m, double* v,
                          TaCounters* ctr, int parity, double beta1, double beta2, double eps, double decay);
hipError_t launch_ta_align(hipStream_t st, int runs, int n_cams, double* o, int32_t* err);
hipError_t launch_ta_losses(hipStream_t st, int runs, int n_cams, int64_t n_pairs, const int32_t* cam_off,
                            const int32_t* cam_ent, const int32_t* pair_i, const int32_t* pair_j,
                            const double* target, const double* o, double* pair_loss, double* cam_loss,
                            double* run_loss);
hipError_t launch_ta_merge(hipStream_t st, int runs, int n_cams, const double* o_runs, const double* cam_loss,
                           double* o_out, int32_t* run_of_cam);

}  // namespace fea
