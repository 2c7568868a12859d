// Focal-length vote (Method > Focal Length Estimation): kernels and
// launchers in fea_focal.hip.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace fea {

// Longest run of one group's entries a work item takes; bytes of one entry
// record.
int fv_items_chunk(int64_t n_entries, int n_cand);
size_t fv_entry_bytes();
// Votes of every group's candidates.  The groups' lists are concatenated:
// entry e is pair ent_pair[e] of group ent_group[e]; items [n_items] are runs
// {first, end} of entries of one group, in order, at least one (possibly
// empty) per group, group g's being grp_item_off[g]..grp_item_off[g + 1].
// f0: a focal length amid the candidates, or 0 where they span more than the
// rank-2 forms are scaled for.  ent: n_entries records of scratch; partial: [n_items * n_cand] scratch,
// unused when every group has one item.
hipError_t launch_fv_vote(hipStream_t st, int n_groups, int n_items, int64_t n_entries, int n_cand,
                          const int32_t* ent_group, const int32_t* ent_pair, const int2* items,
                          const int32_t* grp_item_off, const int32_t* pair_i, const int32_t* pair_j,
                          const int32_t* group, const double* F, const double* f_cur, const double* cand, double f0,
                          double tau, void* ent, double* partial, double* votes, hipEvent_t ev0, hipEvent_t ev1);
hipError_t launch_fv_best(hipStream_t st, int n_groups, int n_cand, const double* votes, const double* cand,
                          double* f_best, int32_t* k_best);

}  // namespace fea
