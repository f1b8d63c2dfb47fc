// The instances of the passes and their launchers (see trim_mark.h).
#include <algorithm>
#include <atomic>

#include "trim_launch.h"
#include "trim_mark.h"

namespace trim {

int launch_invert(const InvertArgs &a, hipStream_t st) {
    const int64_t total = a.nslots * a.nseg;
    const size_t lds = a.nlist <= kInvLists ? (size_t)a.nlist * 4 : 0;
    hipLaunchKernelGGL(invert_count_kernel, dim3((unsigned)((total + kInvPer - 1) / kInvPer)), dim3(1024), lds, st, a);
    hipLaunchKernelGGL(invert_scan_kernel, dim3(1), dim3(1024), 0, st, a);
    hipLaunchKernelGGL(invert_place_kernel, dim3((unsigned)((a.nslots + kInvQueries - 1) / kInvQueries)), dim3(1024), lds, st, a);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

template <bool PICK>
static void (*finish_of(int vec, bool fs))(const FinishArgs) {
    if (fs) return vec == 4 ? finish_kernel<4, true, PICK> : finish_kernel<2, true, PICK>;
    return vec == 4 ? finish_kernel<4, false, PICK> : vec == 2 ? finish_kernel<2, false, PICK> : finish_kernel<1, false, PICK>;
}
int launch_finish(const FinishArgs &a, int vec, bool fs, int threads, size_t lds, int64_t slots, hipStream_t st) {
    if (fs && vec == 1) return TRIM_UNSUPPORTED_SHAPE;
    void (*fn)(const FinishArgs) = a.only ? finish_of<true>(vec, fs) : finish_of<false>(vec, fs);
    // (the table must start at LDS address 0: see launch_instance)
    static std::atomic<int> lds_checked[12];
    std::atomic<int> &seen = lds_checked[(a.only ? 6 : 0) + (fs ? 3 : 0) + (vec == 4 ? 2 : vec == 2 ? 1 : 0)];
    if (seen.load(std::memory_order_acquire) == 0) {
        hipFuncAttributes fa;
        HIP_TRY(hipFuncGetAttributes(&fa, reinterpret_cast<const void *>(fn)));
        seen.store(fa.sharedSizeBytes == 0 ? 1 : -1, std::memory_order_release);
    }
    if (seen.load(std::memory_order_acquire) < 0) return TRIM_INTERNAL;
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(fn), lds));
    hipLaunchKernelGGL(fn, dim3((unsigned)slots), dim3(threads), lds, st, a);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

template <bool VERIFY>
static int launch_lut_as(const LutArgs &a, int dsub, bool fs, hipStream_t st) {
    void (*fn)(const LutArgs) = fs ? lut_tile_kernel<2, true, VERIFY>
                                : dsub == 4 ? lut_tile_kernel<4, false, VERIFY>
                                : dsub == 8 ? lut_tile_kernel<8, false, VERIFY> : lut_tile_kernel<16, false, VERIFY>;
    const int64_t entries = (int64_t)a.nsub * (fs ? kC4 : kC);
    LutArgs b = a;
    for (int64_t s0 = 0; s0 < a.nslots; s0 += (int64_t)kLutQueries * 65535) {       // (grid.y)
        b.nslots = std::min<int64_t>(a.nslots - s0, (int64_t)kLutQueries * 65535);
        b.slot0 = a.slot0 + s0;
        if (a.by_slot) b.lut = a.lut + (size_t)s0 * entries;
        hipLaunchKernelGGL(fn, dim3((unsigned)((entries + 255) / 256), (unsigned)((b.nslots + kLutQueries - 1) / kLutQueries)),
                           dim3(256), 0, st, b);
        HIP_TRY(hipGetLastError());
    }
    return TRIM_OK;
}
int launch_lut(const LutArgs &a, int dsub, bool fs, bool verify, hipStream_t st) {
    if (!lut_tiled(dsub, fs)) return TRIM_UNSUPPORTED_SHAPE;
    return verify ? launch_lut_as<true>(a, dsub, fs, st) : launch_lut_as<false>(a, dsub, fs, st);
}

int launch_totals(const FinishArgs &a, hipStream_t st) {
    hipLaunchKernelGGL(totals_kernel, dim3((unsigned)((a.nslots + 3) / 4)), dim3(256), 0, st, a);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

// The operands of the filter (once per slab of queries).
int launch_filter_operands(const FilterArgs &a, hipStream_t st) {
    hipLaunchKernelGGL(filter_means_kernel, dim3((unsigned)a.nsub), dim3(256), 0, st, a);
    hipLaunchKernelGGL(filter_operands_kernel, dim3((unsigned)(a.kpad / a.padded + a.nslots)), dim3(256), 0, st, a);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

template <int AL, bool CERTAIN>
static void (*filter_of(const FilterArgs &a))(const FilterArgs) {
    switch (a.padded) {
        case 4: return filter_kernel<4, false, AL, CERTAIN>;
        case 8: return filter_kernel<8, false, AL, CERTAIN>;
        case 16: return filter_kernel<16, false, AL, CERTAIN>;
        case 32: return filter_kernel<32, false, AL, CERTAIN>;
        default: return nullptr;
    }
}
int launch_filter(const FilterArgs &a, hipStream_t st) {
    const int64_t blocks = 256 * 4;      // (one per CU at a time)
    // (4-bit codes have a multiple of eight bytes)
    void (*fn)(const FilterArgs);
    if (a.certain) fn = a.ncent == kC4 ? filter_kernel<2, true, 2, true> : a.M % 8 == 0 ? filter_of<2, true>(a) : filter_of<1, true>(a);
    else fn = a.ncent == kC4 ? filter_kernel<2, true, 2, false> : a.M % 8 == 0 ? filter_of<2, false>(a) : filter_of<1, false>(a);
    if (!fn) return TRIM_UNSUPPORTED_SHAPE;
    hipLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(kFltThreads), 0, st, a);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

int launch_measure(const FilterArgs &a, hipStream_t st) {
    // 256 queries at a time where a row tile meets that many (rows are then read half as often: 500 queries x 300,000 x
    // 960: 906 -> 547 us), else 128 and two workgroups per CU (2500 queries in 1024 lists, 768: 414 -> 405, 332 -> 285 us).
    // Without lists:
    //   - 512 queries by 128 rows from 320 queries on, where that makes three tiles for four CUs: 300,000 x 960, 260 queries
    //     308 -> 338 us, 320 441 -> 353, 400 537 -> 373, 500 555 -> 404, 1000 872 -> 684; 28,672 rows x 500 108 -> 87, 3,584 rows 53 -> 75;
    //   - otherwise the queries are cut finer while there are fewer row tiles than CUs, and the rows too while all tiles are resident at
    //     once (500 queries: 612 rows 52 -> 35 us, 3,584 rows 53 -> 36; 11,700 rows, 368 tiles, 43 -> 49).
    const int64_t hi = std::min<int64_t>(a.n, a.hi), row_tiles = (hi + kMsrRows - 1) / kMsrRows;
    const int64_t half_tiles = (std::max<int64_t>(hi - a.lo, 0) + kMsrRows / 2 - 1) / (kMsrRows / 2);
    const double share = a.list_offsets ? (double)a.nslots * a.nseg / a.nlist : (double)a.nslots;
    const bool few_rows = !a.list_offsets && row_tiles < 256;
    const bool wide = !a.list_offsets && a.nslots >= 320 && half_tiles >= 192 && measure_lds(a.d, 8, 2) <= kLdsBytes;
    const bool few = few_rows && !wide && half_tiles * ((a.nslots + 127) / 128) <= 256;
    // (the means of more than 21,000 values leave the LDS no room for 256)
    const int wr = wide || few ? 2 : 4, wq = wide ? 8 : share >= 192.0 && !few_rows && measure_lds(a.d, 4, 4) <= kLdsBytes ? 4 : 2;
    FilterArgs b = a;
    b.msr_block = few_rows && !wide ? 64 * wq : kMsrBlock;
    void (*fn)(const FilterArgs) = wide ? measure_kernel<8, 2, 1, 4> : few ? measure_kernel<2, 2, 4, 2> :
                                   wq == 4 ? measure_kernel<4, 4, 2, 4> : measure_kernel<2, 4, 1, 4>;
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, a.d * 4));
    hipLaunchKernelGGL(fn, dim3(256 * 4), dim3(64 * wq * wr), (size_t)a.d * 4, st, b);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

namespace {
// LDS of the replay and range_exact passes.
size_t replay_carve(ReplayArgs &a) {
    const int ns = a.nseg > 0 ? a.nseg : 1, E = result_slots(a.k);
    auto up = [](size_t x) { return (x + 15) & ~size_t(15); };
    size_t off = 0;
    a.off_segp = (uint32_t)off; off += up((size_t)(ns + 1) * 4);
    a.off_segd = (uint32_t)off; off += up((size_t)ns * 4);
    a.off_q = (uint32_t)off;    off += up((size_t)a.d * 4);
    a.off_cl = (uint32_t)off;   off += kReplayCap * 4;
    a.off_key = (uint32_t)off;  off += (size_t)kReplayCap * 8;
    a.off_g = (uint32_t)off;    off += kReplayCap * 4;
    a.off_d2 = (uint32_t)off;   off += kReplayCap * 4;
    a.off_id = (uint32_t)off;   off += kReplayCap * 4;
    a.off_rd2 = (uint32_t)off;  off += (size_t)kWave * E * 4;
    a.off_rid = (uint32_t)off;  off += (size_t)kWave * E * 4;
    a.off_todo = (uint32_t)off; off += (size_t)kReplayCap * 2;
    return off;
}
}  // namespace

size_t replay_lds(int d, int k, int nseg) {
    ReplayArgs a{};
    a.d = d; a.k = k; a.nseg = nseg;
    return replay_carve(a) + 256;        // (and the kernels' static part)
}

int launch_range_exact(ReplayArgs a, int64_t nslots, int nchunk, hipStream_t st) {
    a.k = 1;
    replay_carve(a);
    const size_t off = a.off_g;          // (what follows is the replay's)
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(range_exact_kernel), off));
    hipLaunchKernelGGL(range_exact_kernel, dim3((unsigned)nslots, (unsigned)nchunk), dim3(kReplayThreads), off, st, a);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

int launch_pick(ReplayArgs a, hipStream_t st) {
    replay_carve(a);
    const size_t off = a.off_cl;          // (what follows is the replay's)
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(pick_kernel), off));
    hipLaunchKernelGGL(pick_kernel, dim3((unsigned)((a.nslots + kXcds - 1) / kXcds * kXcds)), dim3(kReplayThreads), off, st, a);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

int launch_replay(ReplayArgs a, hipStream_t st) {
    const int E = result_slots(a.k);
    const size_t off = replay_carve(a);
    void (*fn)(const ReplayArgs) = E == 1 ? replay_kernel<1> : E == 2 ? replay_kernel<2> : E == 4 ? replay_kernel<4> : replay_kernel<16>;
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(fn), off));
    hipLaunchKernelGGL(fn, dim3((unsigned)a.nslots), dim3(kReplayThreads), off, st, a);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

}  // namespace trim
