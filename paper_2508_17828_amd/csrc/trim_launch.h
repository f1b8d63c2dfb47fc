// What the translation units of libtrim share on the host side: the launch plan of a search,
// the error bookkeeping, and the launchers of the search kernel's instances.  The instances are
// compiled in translation units of their own (trim_search_inst.hip, once per search mode,
// result-set width and code width), so that they build in parallel.
#pragma once

#include <hip/hip_runtime.h>

#include "../../include/trim.h"
#include "trim_passes.h"
#include "trim_search.h"

namespace trim {

// Table phases, block size and LDS layout of a search launch (made by make_plan).
struct Plan {
    int threads;
    int P, Mp, vec;
    size_t lds;
    uint32_t off_q, off_segp, off_segd, off_rest, off_seglb, off_spos, off_sd2, off_sidx, off_rd2, off_rid, off_ctl;
    uint32_t off_plb, off_cnt, off_wq;
    int span, wqcap, cruise, poss_cap, scap, rcap, bucket;
    int use_rest;    // see rest_holds
    int lean;    // a LeanKind; kNN, up to 128 results: launch an 80-register instance (six waves per SIMD, or short codes)
};

// Records a failed HIP call for trim_last_hip_error and returns TRIM_HIP_ERROR.
int hip_fail(hipError_t e);

#define HIP_TRY(expr)                                         \
    do {                                                      \
        hipError_t _e = (expr);                               \
        if (_e != hipSuccess) return ::trim::hip_fail(_e);    \
    } while (0)

constexpr size_t kLdsBytes = 160 * 1024;  // LDS per workgroup on gfx950

// Lets a kernel be launched with `bytes` of dynamic LDS (up to 64 KB it may be without asking).
inline hipError_t allow_lds(const void *fn, size_t bytes) {
    return bytes <= 65536 ? hipSuccess : hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// launch_search_<mode>_e<result entries per lane>_c<bits per code>: enqueue the matching
// instance of search_kernel (with or without the work counters, by SearchArgs::work).
#define TRIM_DECLARE_LAUNCH(name) \
    int name(const SearchArgs &a, const Plan &pl, dim3 grid, hipStream_t st)
// The separate passes (trim_mark_inst.hip).
int launch_finish(const FinishArgs &a, int vec, bool fs, int threads, size_t lds, int64_t slots, hipStream_t st);
int launch_lut(const LutArgs &a, int dsub, bool fs, bool verify, hipStream_t st);
int launch_totals(const FinishArgs &a, hipStream_t st);
int launch_filter_operands(const FilterArgs &a, hipStream_t st);
int launch_filter(const FilterArgs &a, hipStream_t st);
int launch_invert(const InvertArgs &a, hipStream_t st);
int launch_measure(const FilterArgs &a, hipStream_t st);
int launch_range_exact(ReplayArgs a, int64_t nslots, int nchunk, hipStream_t st);
size_t replay_lds(int d, int k, int nseg);      // LDS of one of their workgroups
// The search of few queries (trim_few_inst.hip).
bool few_fits(int d, int M, bool fs, int k, int nseg);
int launch_bound(FewArgs a, bool fs, hipStream_t st);
int launch_settle(FewArgs a, hipStream_t st);
int launch_few_rows(FewArgs a, hipStream_t st);
int launch_replay(ReplayArgs a, hipStream_t st);
int launch_pick(ReplayArgs a, hipStream_t st);

TRIM_DECLARE_LAUNCH(launch_search_knnlean_e1_c8);
TRIM_DECLARE_LAUNCH(launch_search_knnlean_e2_c8);
TRIM_DECLARE_LAUNCH(launch_search_knnlean_e2_c4);
TRIM_DECLARE_LAUNCH(launch_search_knnleanlong_e2_c8);
TRIM_DECLARE_LAUNCH(launch_search_knnleanlong_e2_c4);
TRIM_DECLARE_LAUNCH(launch_search_knnlean_e1_c4);
TRIM_DECLARE_LAUNCH(launch_search_knnleanlong_e1_c8);
TRIM_DECLARE_LAUNCH(launch_search_knnleanlong_e1_c4);
TRIM_DECLARE_LAUNCH(launch_search_knn_e1_c8);
TRIM_DECLARE_LAUNCH(launch_search_knn_e2_c8);
TRIM_DECLARE_LAUNCH(launch_search_knn_e4_c8);
TRIM_DECLARE_LAUNCH(launch_search_knn_e16_c8);
TRIM_DECLARE_LAUNCH(launch_search_range_e1_c8);
TRIM_DECLARE_LAUNCH(launch_search_knn_e1_c4);
TRIM_DECLARE_LAUNCH(launch_search_knn_e2_c4);
TRIM_DECLARE_LAUNCH(launch_search_knn_e4_c4);
TRIM_DECLARE_LAUNCH(launch_search_knn_e16_c4);
TRIM_DECLARE_LAUNCH(launch_search_range_e1_c4);

}  // namespace trim
