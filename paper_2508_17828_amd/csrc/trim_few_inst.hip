// The instances of the few-queries kernels and their launchers (see trim_few.h).
#include <atomic>
#include <type_traits>

#include "trim_few.h"
#include "trim_launch.h"

namespace trim {

namespace {
size_t up(size_t x) { return (x + 15) & ~size_t(15); }
// bound_kernel: table phases of rows that leave room for two workgroups per CU; 0: no room.
size_t bound_carve(FewArgs &a, bool fs) {
    const int row_bytes = fs ? (int)kByteRow<true> : (int)kByteRow<false>, ns = a.nseg > 0 ? a.nseg : 1;
    for (a.P = 1; a.P <= a.M / 4; ++a.P) {
        if (a.M % a.P || (a.M / a.P) % 4) continue;
        a.Mp = a.M / a.P;
        size_t off = (size_t)a.Mp * row_bytes;
        a.off_q = (uint32_t)off;    off += up((size_t)a.d * 4);
        a.off_segp = (uint32_t)off; off += up((size_t)(ns + 1) * 4);
        a.off_segd = (uint32_t)off; off += up((size_t)ns * 4);
        if (off <= 81920) return off;
    }
    return 0;
}
size_t settle_carve(FewArgs &a) {
    const int ns = a.nseg > 0 ? a.nseg : 1, E = result_slots(a.k);
    size_t off = 0;
    a.off_q = (uint32_t)off;    off += up((size_t)a.d * 4);
    a.off_segp = (uint32_t)off; off += up((size_t)(ns + 1) * 4);
    a.off_segd = (uint32_t)off; off += up((size_t)ns * 4);
    a.off_rd2 = (uint32_t)off;  off += (size_t)kWave * E * 4;
    a.off_rid = (uint32_t)off;  off += (size_t)kWave * E * 4;
    a.off_fd2 = (uint32_t)off;  off += kSettleFirst * 4;
    a.off_key = (uint32_t)off;  off += kSettleFirst * 8;
    a.off_todo = (uint32_t)off; off += kSettleFirst * 2;
    static_assert(kSettleFirst * 8 >= kSettleList * 16, "the stretch lists lie over the keys");
    return off;
}
}  // namespace

bool few_fits(int d, int M, bool fs, int k, int nseg) {
    FewArgs a{};
    a.d = d; a.M = M; a.k = k; a.nseg = nseg;
    return bound_carve(a, fs) != 0 && settle_carve(a) + 2048 <= kLdsBytes;      // (and the static part)
}

int launch_bound(FewArgs a, bool fs, hipStream_t st) {
    const size_t lds = bound_carve(a, fs);
    // As many workgroups as are resident at once (three per CU where their tables fit, else two), no more, over all
    // queries, each with a candidate per thread at the least.  Searches, us, two per CU rounded up / this: 48 code bytes, 384 values: 20
    // queries 73.7 / 72.8, 33 82.4 / 78.3, 48 91.4 / 88.7, 67 100.4 / 96.5; 32 code bytes: 20 89.7 / 85.1, 60 124.5 / 112.9; 96 code
    // bytes, 768 values: 20 365.6 / 353.3, 67 518.8 / 504.2, 100 629.6 / 609.3.
    const int64_t resident = 256 * (3 * lds <= kLdsBytes ? 3 : 2);
    const int64_t nsplit = std::max<int64_t>(1, std::min<int64_t>(resident / a.nq, ((int64_t)a.max_cand + kBoundThreads - 1) / kBoundThreads));
    const int vec = (a.M % 16 == 0 && a.Mp % 16 == 0) ? 4 : (a.M % 8 == 0 && a.Mp % 8 == 0) ? 2 : 1;
    void (*fn)(const FewArgs) = nullptr;
    if (fs) {
        if (vec == 1) return TRIM_UNSUPPORTED_SHAPE;
        fn = vec == 4 ? bound_kernel<4, true> : bound_kernel<2, true>;
    } else {
        fn = vec == 4 ? bound_kernel<4, false> : vec == 2 ? bound_kernel<2, false> : bound_kernel<1, false>;
    }
    // (the table must start at LDS address 0: see launch_instance)
    static std::atomic<int> lds_checked[6];
    std::atomic<int> &seen = lds_checked[(fs ? 3 : 0) + (vec == 4 ? 2 : vec == 2 ? 1 : 0)];
    if (seen.load(std::memory_order_acquire) == 0) {
        hipFuncAttributes fa;
        HIP_TRY(hipFuncGetAttributes(&fa, reinterpret_cast<const void *>(fn)));
        seen.store(fa.sharedSizeBytes == 0 ? 1 : -1, std::memory_order_release);
    }
    if (seen.load(std::memory_order_acquire) < 0) return TRIM_INTERNAL;
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(fn), lds));
    hipLaunchKernelGGL(fn, dim3((unsigned)nsplit, (unsigned)a.nq), dim3(kBoundThreads), lds, st, a);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

int launch_settle(FewArgs a, hipStream_t st) {
    const size_t lds = settle_carve(a);
    const int E = result_slots(a.k);
    auto of = [&](auto part) {
        constexpr int P = decltype(part)::value;
        return E == 1 ? settle_kernel<1, P> : E == 2 ? settle_kernel<2, P> : E == 4 ? settle_kernel<4, P> : settle_kernel<16, P>;
    };
    void (*fn)(const FewArgs) = !a.d2_all ? of(std::integral_constant<int, 0>{}) : a.lo == 0 ? of(std::integral_constant<int, 1>{})
                                                                                             : of(std::integral_constant<int, 2>{});
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(fn), lds));
    hipLaunchKernelGGL(fn, dim3((unsigned)a.nq), dim3(settle_threads(E)), lds, st, a);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

int launch_few_rows(FewArgs a, hipStream_t st) {
    settle_carve(a);
    const size_t lds = a.off_rd2;         // (what follows is settle's)
    // as many workgroups as are resident at once, no more than there are groups of 64
    const int64_t groups = ((int64_t)a.hi - a.lo + 63) / 64 + 1, nsplit = std::max<int64_t>(1, std::min<int64_t>(256 * 6 / a.nq, groups));
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(few_rows_kernel), lds));
    hipLaunchKernelGGL(few_rows_kernel, dim3((unsigned)nsplit, (unsigned)a.nq), dim3(kFewRowsThreads), lds, st, a);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

}  // namespace trim
