// C ABI of libtrim (see include/trim.h): argument checks, LDS carve-up, launches.
// No device allocation, no synchronisation, no state between calls.
#include "../../include/trim.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <mutex>

#include "trim_aux.h"
#include "trim_gamma.h"
#include "trim_probe.h"
#include "trim_launch.h"
#include "trim_update.h"
#include "trim_assign.h"

// Scratch area of trim_search_range_static (see below): device memory inside the library's code
// object; every GPU the library runs on holds its own copy at its own address.
static __device__ __align__(256) unsigned char scratch[TRIM_STATIC_SCRATCH_BYTES];

namespace trim {
thread_local int g_last_hip_error = 0;
int hip_fail(hipError_t e) {
    g_last_hip_error = (int)e;
    return TRIM_HIP_ERROR;
}
}  // namespace trim

namespace {

using namespace trim;

static_assert(kWorkCounters == TRIM_WORK_COUNTERS && kWorkFirstPass == TRIM_WORK_FIRST_PASS &&
              kWorkSkipped == TRIM_WORK_SKIPPED && kWorkCodeBytes == TRIM_WORK_CODE_BYTES &&
              kWorkLookups == TRIM_WORK_LOOKUPS && kWorkRows == TRIM_WORK_ROWS &&
              kWorkFullCode == TRIM_WORK_FULL_CODE, "header and kernel disagree on the work counters");



inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline size_t up16(size_t x) { return (x + 15u) & ~size_t(15); }


// Decide table phases, block size and LDS layout for a search launch.
// cap = survivor-list capacity (max(batch,k) for kNN, round size for range).
// batch = candidates per threshold update (range: = cap).  The span of candidates bounded
// between two barriers on the span-by-span path is the largest multiple of batch up to the
// span target (at least one batch, at most kMaxBatchesPerSpan batches).  In kNN mode that
// path only serves the first stretch after the seed and the rare overflow of a cruise
// stretch, so its span is kept short and the LDS goes to residency instead: the layout is
// fitted to the smallest footprint tier (most workgroups per CU) that holds it.
constexpr int kSpanKnn = 1024;
constexpr int kSpanRange = 4096;
constexpr int kSpanLong = 4096;   // kNN span target when the table leaves one workgroup per CU anyway
constexpr int kMaxBatchesPerSpan = 1024;
constexpr int kPossMin = 512;    // smallest possibles list worth cruising with
constexpr int kPossMax = 2048;
constexpr int64_t kCus = 256;
constexpr double kOneGoScan = 16384.0;
constexpr int kOneGoBatch = 128;

// Block size and LDS bytes per workgroup for 4, 3, 2 and 1 workgroups per CU (LDS is handed
// out in 1280-byte granules).  Three 512-thread workgroups, or two of 768 threads, are 6 waves
// per SIMD: only the kernel instances built for that register budget (result_slots <= 2) can use
// those tiers (two entries per lane: k = 100, 8000 queries, 1M x 128, M = 32, 1652 -> 1182 us; 4000 x 500,000 x 384, M = 48, 970 ->
// 839).  The second is for tables too long for three workgroups (M = 40..60): with 24
// instead of 16 waves per CU more rows and code blocks are in flight (5M x 384, M = 48: the
// scan went 5.06 -> 4.70 ms); it is kept to codes under 64 bytes, which the 80-register
// instance is the better one for anyway.
struct Tier { int threads; size_t lds; bool needs_6_waves; bool short_codes_only; };
constexpr Tier kTiers[] = {{256, 40960, false, false}, {512, 53760, true, false}, {768, 81920, true, true},
                           {512, 81920, false, false}, {1024, kLdsBytes, false, false}};

// Thresholds that count on the remaining table minima (and list summaries) rest on an error
// bound of 2 * (table additions) * 2^-24 <= 3.1e-5 (see abandon_threshold): at most 256
// additions per table sum (4-bit codes: two a byte), and the whole table resident.  The 80-register
// instances have them compiled in.
bool rest_holds(int P, int M, int row_bytes) { return P == 1 && M * (row_bytes == (int)kByteRow<true> ? 2 : 1) <= 256; }

// One attempt: table phases P, a footprint tier, a span; need_poss: only layouts with a possibles
// list (a cruise) count.
bool fit_plan(int d, int M, int row_bytes, int nsegs, int cap, int batch, int k, bool range, int P,
              const Tier &tier, int span, bool need_poss, Plan *pl) {
    const int Mp = M / P;
    const int nbatch = span / batch;
    // cruise stretches (kNN): up to 61440 candidates (16-bit queue entries).  Their possibles
    // are counted per bucket of `bucket` candidates (a whole number of batches, at most 1024
    // buckets).
    int cruise = 61440 / batch * batch;
    if (range || cruise < 2 * span) cruise = 0;
    int bucket = batch;
    if (cruise / batch > 1024) bucket = batch * (((cruise + 1023) / 1024 + batch - 1) / batch);
    const int nbucket = cruise > 0 ? (cruise + bucket - 1) / bucket : 0;
    const int ncnt = nbucket > nbatch ? nbucket : nbatch;
    // (4-bit codes: 8 KB in front of the table for the pair table of the first filter pass)
    const size_t tab = (size_t)Mp * row_bytes + (row_bytes == (int)kByteRow<true> ? 8 * kC * 4 : 0);
    const bool rest_ok = rest_holds(P, M, row_bytes);
    if (tier.needs_6_waves && !rest_ok) return false;
    const bool can_cruise = cruise > 0 && P == 1;  // table phases need block-wide barriers
    if (need_poss && !can_cruise) return false;
    const int nwaves = tier.threads / 64;
    // a wave's share of a span is rounded up to 64; two queue arrays of 16-bit entries
    const int wqcap = ((span + nwaves - 1) / nwaves + 63) / 64 * 64;
    size_t wq_min = (size_t)2 * nwaves * wqcap * 2;
    if (can_cruise && wq_min < (size_t)nwaves * kRing * 4) wq_min = (size_t)nwaves * kRing * 4;
    const size_t rest = tab + up16((size_t)d * 4) + up16((size_t)(nsegs + 1) * 4) +
                        up16((size_t)nsegs * 4) + up16((size_t)(Mp / 4 + 1) * 4) +
                        up16((size_t)nsegs * 8) +
                        (range ? up16((size_t)cap * 4) : 0) +
                        up16((size_t)kWave * result_slots(k) * 4) * 2 + up16(sizeof(Ctl)) +
                        up16((size_t)ncnt * 4);
    // The possibles list of a cruise stretch takes what is left, largest first.  Its
    // capacity p also sizes the arrays of the stretch's replay: spos[] holds p entries,
    // and the queue area holds p exact distances and p bounds (queues are only live
    // while bounds are computed, distances and bounds only afterwards).
    static const int kPossTry[] = {kPossMax, 1536, 1024, 768, kPossMin, 0};
    for (int p : kPossTry) {
        if (p > 0 && !can_cruise) continue;
        if (p == 0 && need_poss) continue;
        const int scap = cap > p ? cap : p;
        size_t wq_bytes = wq_min;
        if (wq_bytes < (size_t)(scap + p) * 4) wq_bytes = (size_t)(scap + p) * 4;
        // a span that ends in a replay keeps up to min(scap, span) bounds behind the
        // scap exact distances
        const int span_poss = scap < span ? scap : span;
        if (!range && wq_bytes < (size_t)(scap + span_poss) * 4) wq_bytes = (size_t)(scap + span_poss) * 4;
        wq_bytes = up16(wq_bytes);
        size_t plb = up16((size_t)span * 4);             // bounds of a span / the possibles list
        if (plb < (size_t)p * 8) plb = (size_t)p * 8;
        const size_t total = rest + up16((size_t)scap * 4) + plb + wq_bytes;
        if (total > tier.lds) continue;
        pl->P = P;
        pl->Mp = Mp;
        pl->vec = (M % 16 == 0 && Mp % 16 == 0) ? 4 : (M % 8 == 0 && Mp % 8 == 0) ? 2 : (!range && M % 8 != 0 && Mp >= 16) ? kDwordRows : 1;
        // (kDwordRows: 32 of 1024 lists, 1.18M x 100, M = 20, k = 100: 200 queries 159 -> 136 us, 1000 459 -> 336, 8000 2058 -> 1345;
        // k = 10, 1000 382 -> 241; 100 queries, no lists, 8226 -> 3684.  Range searches, which abandon little early, lose 2 %: 1629 / 1675)
        size_t off = tab;
        pl->off_q = (uint32_t)off;    off += up16((size_t)d * 4);
        pl->off_segp = (uint32_t)off; off += up16((size_t)(nsegs + 1) * 4);
        pl->off_segd = (uint32_t)off; off += up16((size_t)nsegs * 4);
        pl->off_rest = (uint32_t)off; off += up16((size_t)(Mp / 4 + 1) * 4);
        pl->off_seglb = (uint32_t)off; off += up16((size_t)nsegs * 8);
        pl->off_spos = (uint32_t)off; off += up16((size_t)scap * 4);
        pl->off_sidx = (uint32_t)off; if (range) off += up16((size_t)cap * 4);
        pl->off_rd2 = (uint32_t)off;  off += up16((size_t)kWave * result_slots(k) * 4);
        pl->off_rid = (uint32_t)off;  off += up16((size_t)kWave * result_slots(k) * 4);
        pl->off_ctl = (uint32_t)off;  off += up16(sizeof(Ctl));
        pl->off_plb = (uint32_t)off;  off += plb;
        pl->off_cnt = (uint32_t)off;  off += up16((size_t)ncnt * 4);
        pl->off_wq = (uint32_t)off;   off += wq_bytes;
        pl->off_sd2 = pl->off_wq;
        pl->span = span;
        pl->lds = off;
        pl->threads = tier.threads;
        // the 80-register instance: needed for three workgroups per CU, and the better one for short
        // codes in any case (the other's bulk rounds and deeper refine pipelines pay from 64 code bytes on)
        pl->use_rest = rest_ok;
        pl->lean = !(rest_ok && (tier.needs_6_waves || M < 64)) ? kFullInstance
                   : d <= 128 ? kLeanShortRows : kLeanLongRows;
        pl->wqcap = wqcap;
        pl->cruise = p > 0 ? cruise : 0;
        pl->poss_cap = p;
        pl->scap = scap;
        pl->rcap = (int)(wq_bytes / 4) - scap;
        pl->bucket = bucket;
        return true;
    }
    return false;
}

// M counts code bytes; fs: 4-bit codes (two subspaces of 16 centroids per byte), else 8-bit.  scanned: candidates of a query, lists as long
// as each other.
bool make_plan(int d, int M, bool fs, int nseg, int cap, int batch, int k, bool range, int64_t nq, double scanned, Plan *pl) {
    if (d <= 0 || M <= 0 || d % 4 || M % 4) return false;
    if (fs ? (d % (2 * M) || M % 8 || d / (2 * M) > 64) : (d % M || d / M > 64)) return false;
    const int row_bytes = fs ? (int)kByteRow<true> : (int)kByteRow<false>;
    const int nsegs = nseg > 0 ? nseg : 1;
    int nbatch = (range ? kSpanRange : kSpanKnn) / batch;
    if (nbatch < 1) nbatch = 1;
    if (nbatch > kMaxBatchesPerSpan) nbatch = kMaxBatchesPerSpan;
    const int span = nbatch * batch;
    if (span > 65535) return false;
    constexpr int nt = (int)(sizeof(kTiers) / sizeof(kTiers[0]));
    for (int P = 1; P <= M / 4; ++P) {
        if (M % P || (M / P) % 4) continue;
        for (int t = 0; t < nt; ++t) {
            const Tier &tier = kTiers[t];
            if (tier.needs_6_waves && (range || result_slots(k) > 2)) continue;
            if (tier.short_codes_only && M >= 64) continue;
            // Fewer queries than workgroups that fit side by side: more threads a query, one or two workgroups per CU (32 lists of 1024, k = 10,
            // M = 32: 256 queries 125 -> 109 us, 512 142 -> 128; 4-bit codes 94 -> 82, 102 -> 98; 350 queries one per CU: 126 -> 150; 700
            // two per CU: 150 -> 187; k = 100, 200 queries: M = 32 159 -> 128, M = 20 351 -> 159, 4-bit codes 224 -> 139).
            if (!range && result_slots(k) <= 2 && (nq <= kCus ? t + 1 < nt : nq <= 2 * kCus && tier.lds < kLdsBytes / 2)) continue;
            // A short table would fit four small workgroups per CU (16 waves); the instances built
            // for six waves per SIMD do better as three 512-thread ones (24 waves), which also have twice the threads for
            // a query where all are resident at once.  32 of 1024 lists: 1.18M x 100, M = 20, k = 10: 600 queries 333 -> 230 us, 1000 230 ->
            // 229, 8000 2266 -> 1841, k = 100: 200 351 -> 159, 700 404 -> 276, 1000 336 -> 293; M = 16, k = 100, 1000 228 -> 196, 4000 510 ->
            // 462; 4-bit codes, k = 100, 700 260 -> 210, 3000 650 -> 586, 8000 1363 -> 1279.  But not with 8-bit codes
            // between 768 and 1024 queries, which four a CU take in one go, where there is little to scan (three a CU / four, M = 20, 900
            // queries, 7 of 275 lists of 47,000: k = 1 124 / 98, 10 103 / 83, 50 126 / 95, 100 112 / 89; 20 of 640 of 400,000, gamma 0.5, 1024: k = 10 131 /
            // 119, 64 202 / 157, 100 152 / 158; 20 of 900 of 800,000, 775, gamma 0.1: k = 10 157 / 183, 100 180 / 197), batches are short (of 128, k = 64:
            // those 800,000 238 / 216, 30,000 without lists 505 / 403) or codes are shorter and k up to 64 (M = 8, 900 queries 121 / 104; M = 16, 800
            // 127 / 124).
            const bool one_go = !fs && nq > 3 * kCus && nq <= 4 * kCus &&
                                (scanned <= kOneGoScan || batch <= kOneGoBatch || (M <= 16 && result_slots(k) == 1));
            if (t == 0 && !range && result_slots(k) <= 2 && !one_go) continue;
            if (t + 1 < nt) {
                // below the last tier a layout must leave room for a cruise when one is possible
                // at all (else the next tier is tried first)
                const bool cruise_possible = !range && P == 1 && 61440 / batch * batch >= 2 * span;
                if (fit_plan(d, M, row_bytes, nsegs, cap, batch, k, range, P, tier, span, cruise_possible, pl)) return true;
                continue;
            }
            // One workgroup per CU whatever the span: kNN takes the longest span that fits (fewer
            // barriers and more survivors per refine step on the span-by-span path), first among the
            // layouts that keep a possibles list, then among those without.
            if (!range) {
                for (int pass = 0; pass < 2; ++pass)
                    for (int target = kSpanLong; target > span; target -= 1024) {
                        const int longer = target / batch * batch;
                        if (longer <= span || longer / batch > kMaxBatchesPerSpan) continue;
                        if (fit_plan(d, M, row_bytes, nsegs, cap, batch, k, range, P, tier, longer, pass == 0, pl)) return true;
                    }
            }
            if (fit_plan(d, M, row_bytes, nsegs, cap, batch, k, range, P, tier, span, false, pl)) return true;
        }
    }
    return false;
}

// The search kernel's instances are compiled in translation units of their own
// (trim_search_inst.hip); this picks the one for a launch.
int launch_search(bool range, bool fs, const SearchArgs &a, const Plan &pl, dim3 grid, hipStream_t st) {
    if (range) return fs ? launch_search_range_e1_c4(a, pl, grid, st) : launch_search_range_e1_c8(a, pl, grid, st);
    // k decides how many result entries a lane of the merging wave holds (result_slots)
    switch (result_slots(a.k)) {
        case 1:
            if (pl.lean == kLeanLongRows) return fs ? launch_search_knnleanlong_e1_c4(a, pl, grid, st) : launch_search_knnleanlong_e1_c8(a, pl, grid, st);
            if (pl.lean) return fs ? launch_search_knnlean_e1_c4(a, pl, grid, st) : launch_search_knnlean_e1_c8(a, pl, grid, st);
            return fs ? launch_search_knn_e1_c4(a, pl, grid, st) : launch_search_knn_e1_c8(a, pl, grid, st);
        case 2:
            if (pl.lean == kLeanLongRows) return fs ? launch_search_knnleanlong_e2_c4(a, pl, grid, st) : launch_search_knnleanlong_e2_c8(a, pl, grid, st);
            if (pl.lean) return fs ? launch_search_knnlean_e2_c4(a, pl, grid, st) : launch_search_knnlean_e2_c8(a, pl, grid, st);
            return fs ? launch_search_knn_e2_c4(a, pl, grid, st) : launch_search_knn_e2_c8(a, pl, grid, st);
        case 4: return fs ? launch_search_knn_e4_c4(a, pl, grid, st) : launch_search_knn_e4_c8(a, pl, grid, st);
        default: return fs ? launch_search_knn_e16_c4(a, pl, grid, st) : launch_search_knn_e16_c8(a, pl, grid, st);
    }
}

// 4-bit codes (two per byte, 16 centroids per subspace)?  Bytes of one stored code.
inline bool is_fs(const trim_index_view *ix) { return ix->code_bits == 4; }
inline int code_bytes(const trim_index_view *ix) { return is_fs(ix) ? ix->M / 2 : ix->M; }

// A query's share of the base set, lists as long as each other.
inline double scanned_per_query(const trim_index_view *ix, const trim_candidates *cand) {
    return cand ? (double)ix->n * std::min(1.0, (double)cand->nprobe / cand->nlist) : (double)ix->n;
}

int check_index(const trim_index_view *ix) {
    if (!ix) return TRIM_INVALID_ARG;
    if (ix->n < 0 || ix->n >= (int64_t(1) << 31)) return TRIM_INVALID_ARG;
    if (ix->d <= 0 || ix->M <= 0) return TRIM_INVALID_ARG;
    if (ix->code_bits != 0 && ix->code_bits != 8 && ix->code_bits != 4) return TRIM_INVALID_ARG;
    if (!(is_fs(ix) ? trim_fs_shape_supported(ix->d, ix->M) : trim_shape_supported(ix->d, ix->M)))
        return TRIM_UNSUPPORTED_SHAPE;
    if (ix->n > 0 && (!ix->base || !ix->codes || !ix->dlx)) return TRIM_INVALID_ARG;
    if (!aligned16(ix->base) || !aligned16(ix->codes) || !aligned16(ix->codebooks))
        return TRIM_INVALID_ARG;
    if (ix->scan_head && ((reinterpret_cast<uintptr_t>(ix->scan_head) & 3u) || code_bytes(ix) % 8))
        return TRIM_INVALID_ARG;
    if (ix->codes_tiled && (!aligned16(ix->codes_tiled) || code_bytes(ix) % 16)) return TRIM_INVALID_ARG;
    return TRIM_OK;
}

int check_cand(const trim_candidates *c) {
    if (!c) return TRIM_OK;
    if (c->nlist <= 0 || c->nprobe <= 0 || c->nprobe > TRIM_MAX_NPROBE) return TRIM_INVALID_ARG;
    if (!c->list_offsets || !c->probes) return TRIM_INVALID_ARG;
    if (c->list_bounds && !aligned16(c->list_bounds)) return TRIM_INVALID_ARG;
    return TRIM_OK;
}

void fill_common(SearchArgs &a, const trim_index_view *ix, const float *queries, const float *lut,
                 const trim_candidates *cand, float gamma, const trim_stats *stats,
                 uint32_t *mask, int64_t mask_words, const Plan &pl) {
    a.base = ix->base; a.codes = ix->codes; a.dlx = ix->dlx; a.ids = ix->ids;
    a.codebooks = ix->codebooks; a.head = static_cast<const uint32_t *>(ix->scan_head);
    a.codes_tiled = static_cast<const uint8_t *>(ix->codes_tiled); a.n = ix->n; a.d = ix->d;
    a.M = code_bytes(ix);       // the kernel counts code bytes
    a.dsub = ix->d / ix->M;     // length of one subspace's sub-vectors (8- or 4-bit codes alike)
    a.queries = queries; a.lut = lut; a.order = nullptr;
    a.list_offsets = cand ? cand->list_offsets : nullptr;
    a.probes = cand ? cand->probes : nullptr;
    a.nlist = cand ? cand->nlist : 0;
    a.nseg = cand ? cand->nprobe : 0;
    const int64_t hard = (int64_t(1) << 31) - 1 - TRIM_MAX_BATCH - 2048;
    int64_t mc = cand ? cand->max_candidates : ix->n;
    if (mc <= 0 || mc > hard) mc = hard;
    a.max_cand = (int32_t)mc;
    a.P = pl.P; a.Mp = pl.Mp;
    a.two_gamma = 2.0f * gamma;
    a.n_scanned = stats ? stats->n_scanned : nullptr;
    a.n_exact = stats ? stats->n_exact : nullptr;
    a.work = stats ? stats->work : nullptr;
    a.mask = mask; a.mask_words = mask_words;
    a.off_q = pl.off_q; a.off_segp = pl.off_segp; a.off_segd = pl.off_segd; a.off_rest = pl.off_rest;
    a.off_seglb = pl.off_seglb;
    a.list_bounds = cand ? static_cast<const uint8_t *>(cand->list_bounds) : nullptr;
    a.off_spos = pl.off_spos; a.off_sd2 = pl.off_sd2; a.off_sidx = pl.off_sidx;
    a.off_rd2 = pl.off_rd2; a.off_rid = pl.off_rid; a.off_ctl = pl.off_ctl;
    a.off_plb = pl.off_plb; a.off_cnt = pl.off_cnt; a.span = pl.span;
    a.off_wq = pl.off_wq; a.wqcap = pl.wqcap; a.cruise = pl.cruise; a.poss_cap = pl.poss_cap; a.scap = pl.scap; a.rcap = pl.rcap; a.bucket = pl.bucket;
    a.bucket_inv = pl.bucket > 1 ? (uint32_t)(((uint64_t(1) << 32) + pl.bucket - 1) / pl.bucket) : 0;      // (stretches have buckets of 60 and more)
    a.small_addr = ix->n < (int64_t(1) << 24) && ix->n * (int64_t)ix->M < (int64_t(1) << 32) &&
                   ix->M < (1 << 24);
    a.use_rest = pl.use_rest;
}

int fill_u32(uint32_t *p, size_t count, uint32_t v, hipStream_t st) {
    if (count == 0) return TRIM_OK;
    size_t blocks = (count + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p, count, v);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

int zero_areas(const ZeroAreas &z, hipStream_t st) {
    if (z.count > ZeroAreas::kMost) return TRIM_INTERNAL;
    size_t most = 0;
    for (int i = 0; i < z.count; ++i) most = std::max(most, z.words[i]);
    if (most == 0) return TRIM_OK;
    hipLaunchKernelGGL(zero_areas_kernel, dim3((unsigned)std::min<size_t>((most + 255) / 256, 4096)), dim3(256), 0, st, z);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

// Clusters per workgroup of the k-means update: as many as 32 (every workgroup reads all the
// assignments), fewer until there is a workgroup per CU or one cluster is left, and never
// more than 48 KB of float64 sums.
template <int ABYTES>
int launch_kmeans_update(const float *x, int64_t ns, int d, int dim, const void *assign, int64_t astride, int64_t ystride, int K,
                         int ny, float *cent, hipStream_t st) {
    const int cols = dim < kUpdCols ? dim : kUpdCols, nz = (dim + kUpdCols - 1) / kUpdCols;
    int lg = kUpdMaxLog2;
    while (lg > 0 && ((int64_t)((K + (1 << lg) - 1) >> lg) * ny * nz < 256 || ((size_t)cols << lg) * 8 > 48 * 1024)) --lg;
    UpdateArgs a{};
    a.vals = (int32_t)std::min<int64_t>(kUpdVals, (ns * cols + 63) / 64 * 64);
    a.x = x; a.assign = assign; a.ns = ns; a.stride = d; a.astride = astride; a.ystride = ystride;
    a.dim = dim; a.K = K; a.cg_log2 = lg; a.groups = (K + (1 << lg) - 1) >> lg; a.ny = ny; a.cent = cent;
    const int64_t total = (int64_t)a.groups * ny * nz;
    if (total > 0x7fffffff - kXcds) return TRIM_UNSUPPORTED_SHAPE;
    a.total = (int32_t)total;
    // (no more workgroups than CUs: room beside them is none's, and the other instance has more loads in flight: 8192 x 128, 64 x 16 x 2
    // coordinates, 4 iterations: 361 us, 388 with the few)
    const bool few = ns <= kUpdFew && total > 256;
    const size_t lds = kmeans_update_lds(lg, cols, few ? kUpdFew : kUpdList, a.vals);
    void (*fn)(UpdateArgs) = few ? kmeans_update_kernel<ABYTES, kUpdFew> : kmeans_update_kernel<ABYTES, kUpdList>;
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(fn), lds));
    hipLaunchKernelGGL(fn, dim3((unsigned)((total + kXcds - 1) / kXcds * kXcds)), dim3(kUpdThreads), lds,
                       st, a);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

// Work space of the update step (trim_update.h): the clusters' first places, the rows' numbers in cluster order, and (short rows) the
// sub-vectors clustering by clustering.
struct UpdateLayout {
    bool brief;                   // short rows
    int loops, threads, rows, nchunk;
    size_t off_list, off_columns, total;      // total: 0 where the update goes without
};
UpdateLayout update_layout(int64_t ns, int dim, int K, int ny) {
    UpdateLayout L{};
    if (ns <= 0 || dim <= 0 || K <= 0 || ny <= 0 || ny > 65535 || ns > 0x7fffffff - 65536) return L;
    // Few rows, or few to a cluster: kmeans_update_kernel, one launch instead of two (4 iterations of training, us, without / with:
    // codebooks, 300 x 128 76 / 90, 4096 x 128 98 / 106, 8192 x 128 109 / 118, 8192 x 1024 430 / 409, 65,536 x 128 513 / 418, 16 centroids:
    // 16,384 x 512 1186 / 1223, 65,536 x 128 1080 / 1014; coarse lists, 8000 x 768 in 4096 5214 / 5354, 4096 x 128 in 64 168 / 133).
    if (ny > 1 ? ns <= 4096 || ny * ns < (1 << 19) || (K < kC && ns < 32768) : ns < 8 * (int64_t)K) return L;
    L.brief = dim <= kShortRow;
    // 4096 rows a chunk; 1024 where a workgroup has one clustering's assignments only, and there are few chunks
    L.loops = ny > 1 || ns > 256 * kSortThreads ? 4 : 1;
    for (L.threads = kSortThreads; kmeans_sort_lds(L.threads, K) > (size_t)kSortCounters; L.threads >>= 1)
        if (L.threads == kWave) return L;
    if (L.threads < kSortThreads) L.loops = 4;
    L.rows = L.loops * L.threads;
    L.nchunk = (int)((ns + L.rows - 1) / L.rows);
    if ((int64_t)K * ny * ((dim + kUpdCols - 1) / kUpdCols) > 0x7fffffff - kXcds) return L;
    L.off_list = ((size_t)ny * L.nchunk * (K + 1) * 2 + 255) & ~size_t(255);
    L.off_columns = (L.off_list + (size_t)ny * ns * 2 + 255) & ~size_t(255);
    L.total = L.off_columns + (L.brief && ny > 1 ? (size_t)ny * ns * dim * 4 : 0);
    return L;
}
// What is laid out once per training.
int kmeans_columns(const float *x, int64_t ns, int d, int dim, int ny, const UpdateLayout &L, unsigned char *ws, hipStream_t st) {
    if (!ws || !L.brief || ny == 1 || !aligned16(x)) return TRIM_OK;
    hipLaunchKernelGGL(kmeans_columns_kernel, dim3((unsigned)((ns + kWave - 1) / kWave)), dim3(256), 0, st, x, ns, (int64_t)d, dim, ny,
                       reinterpret_cast<float *>(ws + L.off_columns));
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}
template <int ABYTES>
int launch_kmeans_sorted(const float *x, int64_t ns, int d, int dim, const void *assign, int64_t astride, int64_t ystride, int K, int ny,
                         float *cent, const UpdateLayout &L, unsigned char *ws, hipStream_t st) {
    SortArgs a{};
    a.x = x; a.assign = assign; a.ns = ns; a.stride = d; a.astride = astride; a.ystride = ystride;
    a.xstep = dim;
    if (L.brief && ny > 1 && aligned16(x)) { a.x = reinterpret_cast<const float *>(ws + L.off_columns); a.stride = dim; a.xstep = ns * dim; }
    a.dim = dim; a.K = K; a.ny = ny; a.nchunk = L.nchunk; a.rows = L.rows; a.cent = cent;
    while ((1 << a.kbits) < K) ++a.kbits;
    a.starts = reinterpret_cast<uint16_t *>(ws);
    a.list = reinterpret_cast<uint16_t *>(ws + L.off_list);
    void (*sort)(SortArgs) = L.loops == 4 ? kmeans_sort_kernel<ABYTES, 4> : kmeans_sort_kernel<ABYTES, 1>;
    const size_t lds = kmeans_sort_lds(L.threads, K);
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(sort), lds));
    hipLaunchKernelGGL(sort, dim3((unsigned)L.nchunk, (unsigned)ny), dim3(L.threads), lds, st, a);
    HIP_TRY(hipGetLastError());
    if (L.brief) {
        // clusters per workgroup: as many as there are threads to add for, fewer until there is a workgroup per CU
        a.cg_log2 = kSumMaxLog2;
        while (a.cg_log2 > 0 && ((dim << a.cg_log2) > kSumThreads || (int64_t)((K + (1 << a.cg_log2) - 1) >> a.cg_log2) * ny < 512)) --a.cg_log2;
        const int64_t groups = (int64_t)((K + (1 << a.cg_log2) - 1) >> a.cg_log2) * ny;
        const bool vec = dim % 4 == 0 && (a.stride | a.xstep) % 4 == 0 && aligned16(a.x);
        void (*sums)(SortArgs) = vec ? (dim == 4 ? kmeans_sums_kernel<4, true> : dim == 8 ? kmeans_sums_kernel<8, true> : kmeans_sums_kernel<0, true>)
                                     : dim == 2 ? kmeans_sums_kernel<2, false> : kmeans_sums_kernel<0, false>;
        hipLaunchKernelGGL(sums, dim3((unsigned)((groups + kXcds - 1) / kXcds * kXcds)), dim3(kSumThreads), 0, st, a);
    } else {
        const int nz = (dim + kUpdCols - 1) / kUpdCols, cols = dim < kUpdCols ? dim : kUpdCols;
        hipLaunchKernelGGL(kmeans_rows_kernel, dim3((unsigned)(K * nz), (unsigned)ny), dim3(cols <= 64 ? 64 : cols <= 128 ? 128 : kUpdCols), 0, st, a);
    }
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}
// The update with a work space (null: without) that update_layout's size was asked for.
template <int ABYTES>
int kmeans_update(const float *x, int64_t ns, int d, int dim, const void *assign, int64_t astride, int64_t ystride, int K, int ny,
                  float *cent, unsigned char *ws, hipStream_t st) {
    if (ws) return launch_kmeans_sorted<ABYTES>(x, ns, d, dim, assign, astride, ystride, K, ny, cent, update_layout(ns, dim, K, ny), ws, st);
    return launch_kmeans_update<ABYTES>(x, ns, d, dim, assign, astride, ystride, K, ny, cent, st);
}
// A caller's work space from its first multiple of 256 on, or null where it is too small for that.
unsigned char *update_space(void *ws, size_t bytes, size_t need) {
    if (!ws || need == 0 || bytes < need + 256) return nullptr;
    return reinterpret_cast<unsigned char *>((reinterpret_cast<uintptr_t>(ws) + 255) & ~uintptr_t(255));
}

// Encoding with the matrix-core filter: T vectors per workgroup, 512 or 256 (which prepare a subspace's centroids twice as often).
template <int D, int T>
int launch_encode_t(const float *base, int64_t n, int d, const float *codebooks, int M, int jper, uint8_t *codes, int64_t across,
                    float *dlx, hipStream_t st) {
    void (*fn)(const float *, int64_t, int, const float *, int, int, uint8_t *, int64_t, float *) =
        across ? encode_mfma_kernel<D, T, true> : encode_mfma_kernel<D, T, false>;
    const size_t lds = sizeof(EncodeLds<D, T>);
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(fn), lds));
    hipLaunchKernelGGL(fn, dim3((unsigned)((n + T - 1) / T), (unsigned)((M + jper - 1) / jper)), dim3(T), lds, st, base, n, d,
                       codebooks, M, jper, codes, across, dlx);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}
template <int D>
int launch_encode(const float *base, int64_t n, int d, const float *codebooks, int M, uint8_t *codes, int64_t across, float *dlx,
                  hipStream_t st) {
    // Subspaces per workgroup: all, or fewer until there are enough workgroups: two thirds again as many as are resident, or more where
    // nobody wants the landmark distances, which take a pass of their own then (us, whole / split: 49,152 x 128 80 / 58, 40,000 x 1536
    // 733 / 515, 65,536 x 128 82 / 72, 60,000 x 1536 762 / 780; training, 65,536 x 128, four iterations 480 / 354).
    const int64_t many = (n + 511) / 512, few = (n + 255) / 256;
    int jper = M;
    if (many <= (dlx ? 112 : 512)) {
        const int64_t split = std::min<int64_t>(M / 4, ((dlx ? 768 : 1024) + many - 1) / many);
        jper = (int)((M / 4 + split - 1) / split) * 4;
    }
    // 512 vectors a workgroup, unless few are there (us, 256 / 512: 4096 x 128 18 / 20, 16,384 x 128 27 / 26) or 256 share the CUs out better:
    // a step with 256 costs 9/8 of one with 512 (160,000 x 128 115 / 125, 200,000 x 128 142 / 125, 1,000,000 x 128 599 / 547).
    const bool wide = jper < M ? many * (M / jper) > 128 : 9 * ((few + 255) / 256) >= 16 * ((many + 255) / 256);
    const int rc = wide ? launch_encode_t<D, 512>(base, n, d, codebooks, M, jper, codes, across, dlx, st)
                        : launch_encode_t<D, 256>(base, n, d, codebooks, M, jper, codes, across, dlx, st);
    if (rc) return rc;
    if (jper < M && dlx)
        hipLaunchKernelGGL(encode_dlx_kernel, dim3((unsigned)((n + kDlxRows - 1) / kDlxRows)), dim3(256), 0, st, base, n, d,
                           codebooks, M, D, codes, dlx);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

template <bool PACKED>
int launch_encode_fs(const float *base, int64_t n, int d, const float *codebooks, int m, uint8_t *codes, int64_t across, float *dlx,
                     hipStream_t st) {
    const int dsub = d / m;
    if (dsub == 2)
        hipLaunchKernelGGL(encode_fs2_kernel<PACKED>, dim3((unsigned)((n + kFsRows - 1) / kFsRows)), dim3(kFsRows), 0, st, base,
                           n, d, codebooks, m, codes, across, dlx);
    else
        hipLaunchKernelGGL(encode_fs_kernel<PACKED>, dim3((unsigned)((n + 255) / 256)), dim3(256), (size_t)2 * kC4 * dsub * 4,
                           st, base, n, d, codebooks, m, dsub, codes, across, dlx);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

// trim_encode past its checks.  dlx may be null where the caller needs the codes only (training).
int encode_codes(const float *base, int64_t n, int d, const float *codebooks, int M, uint8_t *codes, int64_t across, float *dlx,
                 hipStream_t st) {
    const int dsub = d / M;
    switch (dsub) {
        case 4: return launch_encode<4>(base, n, d, codebooks, M, codes, across, dlx, st);
        case 5: return launch_encode<5>(base, n, d, codebooks, M, codes, across, dlx, st);
        case 6: return launch_encode<6>(base, n, d, codebooks, M, codes, across, dlx, st);
        case 8: return launch_encode<8>(base, n, d, codebooks, M, codes, across, dlx, st);
        default: break;
    }
    hipLaunchKernelGGL(encode_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), (size_t)kC * dsub * 4, st, base, n, d,
                       codebooks, M, dsub, codes, across, dlx);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

constexpr int kRangeRound = 2048;   // survivor-list capacity per round in range mode
constexpr int kRangeSplitTarget = 2048;  // aim for at least this many workgroups

int range_nsplit(int64_t nq, int64_t max_cand) {
    int64_t want = (kRangeSplitTarget + nq - 1) / (nq > 0 ? nq : 1);
    if (want < 1) want = 1;
    // at least 4096 candidates per chunk so that the table fill is amortised
    int64_t most = (max_cand + 4095) / 4096;
    if (most < 1) most = 1;
    if (want > most) want = most;
    if (want > 65535) want = 65535;
    return (int)want;
}

struct RangeLayout {
    int nsplit;
    int chunk;
    int64_t rmask_words;
    size_t off_counts, off_cbase, off_d2, total;
};

RangeLayout range_layout(int64_t nq, int64_t max_cand) {
    RangeLayout L;
    L.nsplit = range_nsplit(nq, max_cand);
    int64_t chunk = (max_cand + L.nsplit - 1) / L.nsplit;
    chunk = (chunk + 63) / 64 * 64;
    if (chunk < 64) chunk = 64;
    L.chunk = (int)chunk;
    L.rmask_words = (int64_t)L.nsplit * (chunk / 32);
    size_t off = (size_t)nq * L.rmask_words * 4;
    off = (off + 255) & ~size_t(255);
    L.off_counts = off; off += (size_t)nq * L.nsplit * 4;
    off = (off + 255) & ~size_t(255);
    L.off_cbase = off; off += (size_t)nq * L.nsplit * 8;
    off = (off + 255) & ~size_t(255);
    // the exact distance of every result waits here, at its scan-order number, for the pass that
    // writes the CSR arrays (one binary32 per candidate slot; only result slots are touched)
    L.off_d2 = off; off += (size_t)nq * L.rmask_words * 32 * 4;
    L.total = (off + 255) & ~size_t(255);
    return L;
}

// The scratch area lives from the first use of the library on a GPU until the process ends.
// In host code the array's name is only a handle: its device address is asked for once per
// device (hipGetSymbolAddress with that device current) and kept here; host code passes that
// address, never the name, to kernels.
constexpr size_t kScratchBytes = TRIM_STATIC_SCRATCH_BYTES;
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices] = {};

int scratch_for_current_device(void **out) {
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return TRIM_INVALID_ARG;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p || (reinterpret_cast<uintptr_t>(p) & 255u)) return TRIM_HIP_ERROR;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return TRIM_OK;
}

// ---- the scan in separate passes (trim_mark.h) ----

// Table phases, block size and LDS layout of the finish pass: two workgroups of 512 threads per CU
// where they fit, else one of 1024.  few: most candidates' sums are not wanted (range searches, by the centroids' own tables), and a
// workgroup spends its time on the table and on getting ready; two per CU then pay for up to four phases (2,000 queries, 192 code
// bytes, 36 sums each: 188 -> 159 us; with every sum wanted, 120 code bytes: 555 -> 691).  Uneven variances and small radii leave more
// sums, but few enough too: whole searches, 1,000 queries x 100,000 x 960, before / with certain bits and this plan: 600 / 533 us, gamma 0
// and a small radius 501 / 470.
struct FinishPlan {
    int threads, P, Mp, vec;
    size_t lds;
    uint32_t off_q, off_segp, off_segd, off_bits, off_ring;
};
bool make_finish_plan(int d, int M, bool fs, int nseg, bool few, FinishPlan *pl) {
    const int row_bytes = fs ? (int)kByteRow<true> : (int)kByteRow<false>;
    const int ns = nseg > 0 ? nseg : 1;
    for (int i = few ? 0 : 4; i <= 3 + M / 4; ++i) {
        const int P = i < 4 ? i + 1 : i - 3;         // (the first four: two workgroups per CU or not at all)
        if (M % P || (M / P) % 4) continue;
        const int Mp = M / P;
        for (int threads = 512; threads <= (i < 4 ? 512 : 1024); threads *= 2) {
            size_t off = (size_t)Mp * row_bytes;
            pl->off_q = (uint32_t)off;    off += up16((size_t)d * 4);
            pl->off_segp = (uint32_t)off; off += up16((size_t)(ns + 1) * 4);
            pl->off_segd = (uint32_t)off; off += up16((size_t)ns * 4);
            pl->off_bits = (uint32_t)off; off += kFinishPiece / 8 + 64;
            pl->off_ring = (uint32_t)off; off += kFinishList * 2;
            if (off > (threads == 512 ? (size_t)81920 : kLdsBytes)) continue;
            pl->threads = threads; pl->P = P; pl->Mp = Mp; pl->lds = off;
            pl->vec = (M % 16 == 0 && Mp % 16 == 0) ? 4 : (M % 8 == 0 && Mp % 8 == 0) ? 2 : 1;
            return true;
        }
    }
    return false;
}
void fill_plan(FinishArgs &m, const FinishPlan &pl) {
    m.P = pl.P; m.Mp = pl.Mp;
    m.off_q = pl.off_q; m.off_segp = pl.off_segp; m.off_segd = pl.off_segd; m.off_bits = pl.off_bits; m.off_ring = pl.off_ring;
}
void fill_finish(FinishArgs &m, const FinishPlan &pl, const SearchArgs &a) {
    fill_plan(m, pl);
    m.codes = a.codes; m.dlx = a.dlx; m.codebooks = a.codebooks; m.n = a.n; m.d = a.d; m.M = a.M; m.dsub = a.dsub;
    m.queries = a.queries; m.nq = a.nq; m.order = a.order; m.lut = a.lut;
    m.list_offsets = a.list_offsets; m.probes = a.probes;
    m.nlist = a.nlist; m.nseg = a.nseg; m.max_cand = a.max_cand;
    m.two_gamma = a.two_gamma; m.n_scanned = a.n_scanned;
}

// Whether a search runs in passes.  They pay where rows are long (what the single kernel reads once per query and
// survivor), a list is scanned by a few queries at a time (its tiles hold 128 of them) and the single
// kernel has more queries than CUs.  How much depends on the data, which the host does not see: what the passes save are the rows and
// lookups of survivors, of which there are few where the vectors' groups lie far apart.  Measured, passes / single kernel
// (100,000 and 400,000 vectors, 20 of 316 and 40 of 632 lists, k = 10, gamma 0.3 and 0.6; queries 260 / 1000 / 3000):
//   unit vectors, groups of 4000:   512 values 0.59-0.77 / 0.37-0.63 / 0.38-0.55;  768: 0.57-0.71 / 0.38-0.55 / 0.36-0.47;  1536: 0.45-0.55 / 0.36-0.45 / 0.29-0.36
//   uneven variances, groups of 2000:   512: 0.99-1.73 / 0.80-1.31 / 0.68-1.00;  768: 0.87-1.74 / 0.73-1.17 / 0.61-0.88;  1536: 0.81-1.15 / 0.58-0.81 / 0.48-0.57
//   the same, no lists (60,000 vectors):   512: 1.10-1.13 / 0.79-0.87 / 0.75-0.80;  1024: 0.43-0.54 / 0.40-0.43 / 0.34-0.37
//   far apart, groups of 1000:   512: 1.46-2.18 / 1.33-1.76 / 1.05-1.53;  768: 1.33-2.44 / 1.18-1.96 / 0.93-1.54;  1536: 0.69-1.21 / 0.64-1.04 / 0.48-0.85
// The line is drawn for the first kind, which rows of 512 values and more (embeddings) usually are: of 69 searches of
// the first two kinds drawn over sizes, codes and gammas, kNN and range, 66 are faster in passes (0.17-0.98) and three
// slower (1.05-1.14).  A program whose data are of the last kind keeps the single kernel by giving no work space.  Below 512
// values: 256 values, 300 to 1200 queries: 1.4-1.8.
constexpr int64_t kManyQueries = 256;
constexpr int kLongRow = 512;
constexpr double kSharedValues = 8192.0;      // values per row times queries per list
constexpr size_t kKnnSlabBytes = size_t(8) << 30;
bool worth_passes(const trim_index_view *ix, int64_t nq, const trim_candidates *cand) {
    if (nq <= kManyQueries || ix->n <= 0 || ix->d < kLongRow || !filter_padded(ix->d / ix->M, is_fs(ix))) return false;
    const double share = cand ? (double)nq * cand->nprobe / cand->nlist : (double)nq;
    return share * ix->d >= kSharedValues;
}

// The passes count (query, list) pairs and tiles in 32 bits, and number the 16-byte pieces of the queries' 16-bit operands
// by as many.  mc: candidates per query.  A list that v queries scan has at most (mc / 256 + 1) (v / 128 + 1) tiles, v adding up to
// the pairs.
bool counts_fit(const trim_index_view *ix, int64_t rows, const trim_candidates *cand, int64_t mc) {
    const double pairs = (double)rows * (cand ? cand->nprobe : 1), lists = cand ? cand->nlist : 1;
    const double reach = (double)std::min(mc, ix->n);
    const double tiles = (reach / kMsrRows + 1) * (pairs / kFltQ + 1) + (double)ix->n / kMsrRows + lists;
    return pairs < 2147483648.0 && tiles < 2147483648.0 && (double)rows * (ix->d + 2 * kFltSlice) / 8 < 4294967296.0;
}

// What else a search in passes needs: room in the LDS for every one of them, and the centroids.
bool passes_fit(const trim_index_view *ix, const trim_candidates *cand, int k, bool few, FinishPlan *fp) {
    const int nseg = cand ? cand->nprobe : 0;
    return ix->codebooks && make_finish_plan(ix->d, code_bytes(ix), is_fs(ix), nseg, few, fp) &&
           replay_lds(ix->d, k, nseg) <= kLdsBytes && measure_lds(ix->d, 2, 4) <= kLdsBytes;
}

inline size_t up256(size_t x) { return (x + 255) & ~size_t(255); }

// Work space of the filter and measure passes for `rows` queries (offsets from `at`; 0 bytes: shape without a filter).
struct FilterLayout {
    int padded, kpad, kpad_rows;
    bool tables;              // distance tables beside (lut_tile_kernel)
    size_t off_start, off_cnt, off_tasks, off_inv, off_seg, off_mu, off_max, off_books, off_q16, off_q16r, off_qpar, off_bad, off_lut, end;
};
size_t table_bytes(const trim_index_view *ix) { return (size_t)ix->M * (is_fs(ix) ? kC4 : kC) * 4; }
size_t filter_bytes_per_query(const trim_index_view *ix, const trim_candidates *cand) {
    const int padded = filter_padded(ix->d / ix->M, is_fs(ix));
    return (size_t)(cand ? cand->nprobe : 0) * 16 + ((size_t)ix->M * padded + ix->d + 4 * kFltSlice) * 2 + 8 + 4 +
           (lut_tiled(ix->d / ix->M, is_fs(ix)) ? table_bytes(ix) : 0);
}
FilterLayout filter_layout(const trim_index_view *ix, int64_t rows, int64_t rows_all, const trim_candidates *cand, size_t at) {
    FilterLayout L{};
    L.padded = filter_padded(ix->d / ix->M, is_fs(ix));
    L.kpad = (ix->M * L.padded + 2 * kFltSlice - 1) / (2 * kFltSlice) * (2 * kFltSlice);     // (slices come in pairs)
    L.kpad_rows = (ix->d + 2 * kFltSlice - 1) / (2 * kFltSlice) * (2 * kFltSlice);
    size_t off = at;
    if (cand) {
        L.off_start = off; off += up256((size_t)(cand->nlist + 1) * 4);
        L.off_cnt = off;   off += up256((size_t)cand->nlist * 4);
        L.off_tasks = off; off += up256((size_t)(cand->nlist + 1) * 8);
        L.off_inv = off;   off += up256((size_t)rows * cand->nprobe * 8);
        L.off_seg = off;   off += up256((size_t)rows * cand->nprobe * 8);
    }
    L.off_mu = off;    off += up256((size_t)ix->d * 4);
    L.off_max = off;   off += 256;
    L.off_books = off; off += up256((size_t)L.kpad * (is_fs(ix) ? kC4 : kC) * 2);
    L.off_q16 = off;   off += up256((size_t)rows * L.kpad * 2);
    L.off_q16r = L.off_q16;
    if (ix->d / ix->M != L.padded) { L.off_q16r = off; off += up256((size_t)rows * L.kpad_rows * 2); }
    L.off_qpar = off;  off += up256((size_t)rows * 8);
    L.off_bad = off;   off += up256((size_t)rows_all * 4);
    // (tables of queries that are not taken in slabs: up to 2 GB of them)
    L.tables = lut_tiled(ix->d / ix->M, is_fs(ix)) && rows * table_bytes(ix) <= kKnnSlabBytes / 4;
    L.off_lut = off;   off += L.tables ? up256((size_t)rows * table_bytes(ix)) : 0;
    L.end = off;
    return L;
}
// Arguments of the passes that do not change from one to the next.
void fill_filter(FilterArgs &f, InvertArgs &v, const trim_index_view *ix, const SearchArgs &a, const FilterLayout &L, unsigned char *ws) {
    if (a.nseg > 0) {
        v.probes = a.probes; v.nq = a.nq; v.order = a.order; v.nseg = a.nseg; v.nlist = a.nlist;
        v.list_offsets = a.list_offsets; v.n = a.n; v.max_cand = a.max_cand;
        v.cnt = reinterpret_cast<int32_t *>(ws + L.off_cnt);
        v.start = reinterpret_cast<int32_t *>(ws + L.off_start);
        v.inv = reinterpret_cast<int2 *>(ws + L.off_inv);
        v.seg = reinterpret_cast<int32_t *>(ws + L.off_seg);
        v.tasks = reinterpret_cast<int32_t *>(ws + L.off_tasks);
        v.row_tasks = v.tasks + a.nlist + 1;
    }
    f.codes = a.codes; f.dlx = a.dlx; f.codebooks = a.codebooks; f.n = a.n; f.d = a.d; f.M = a.M; f.dsub = a.dsub;
    f.nsub = ix->M; f.ncent = is_fs(ix) ? kC4 : kC; f.queries = a.queries; f.nq = a.nq; f.order = a.order;
    f.list_offsets = a.nseg > 0 ? a.list_offsets : nullptr; f.nlist = a.nlist; f.nseg = a.nseg;
    f.inv_start = v.start; f.inv = v.inv; f.tasks = v.tasks; f.row_tasks = v.row_tasks;
    f.two_gamma = a.two_gamma; f.padded = L.padded; f.kpad = L.kpad; f.kpad_rows = L.kpad_rows; f.base = a.base;
    f.mu = reinterpret_cast<float *>(ws + L.off_mu);
    f.max_bits = reinterpret_cast<uint32_t *>(ws + L.off_max);
    f.books = reinterpret_cast<_Float16 *>(ws + L.off_books);
    f.q16 = reinterpret_cast<_Float16 *>(ws + L.off_q16);
    f.q16_rows = reinterpret_cast<_Float16 *>(ws + L.off_q16r);
    f.qpar = reinterpret_cast<float *>(ws + L.off_qpar);
}
// The inverted probe lists and the 16-bit operands of the queries [slot0, slot0 + nslots); z: what else is to be cleared.
int prepare_filter(FilterArgs &f, InvertArgs &v, int64_t slot0, int64_t nslots, ZeroAreas z, hipStream_t st) {
    int rc;
    f.slot0 = v.slot0 = slot0;
    f.nslots = v.nslots = nslots;
    if (v.cnt) z.add(v.cnt, (size_t)v.nlist);
    z.add(f.max_bits, 1);
    if ((rc = zero_areas(z, st))) return rc;
    if (v.cnt && (rc = launch_invert(v, st))) return rc;
    return launch_filter_operands(f, st);
}

// The tables of the finish pass, for the queries [slot0, slot0 + nslots): made here, or a caller's compared with the
// centroids (by_query: rows of the work space are at the queries' numbers).  z must have cleared the `bad` words.
int prepare_tables(FinishArgs &m, const trim_index_view *ix, const SearchArgs &a, const FilterLayout &L, unsigned char *ws, hipStream_t st) {
    LutArgs t{};
    t.queries = a.queries; t.nq = a.nq; t.d = a.d; t.codebooks = a.codebooks; t.nsub = ix->M; t.order = a.order;
    t.slot0 = m.slot0; t.nslots = m.nslots;
    if (a.lut) {
        t.lut = const_cast<float *>(a.lut);
        t.bad = reinterpret_cast<uint32_t *>(ws + L.off_bad);
        m.bad = t.bad;
        return launch_lut(t, a.dsub, is_fs(ix), true, st);
    }
    if (!L.tables) return TRIM_OK;
    t.lut = reinterpret_cast<float *>(ws + L.off_lut);
    t.by_slot = !m.by_query;
    m.lut = t.lut;
    m.lut_by_row = 1;
    return launch_lut(t, a.dsub, is_fs(ix), false, st);
}

struct KnnLayout {
    int64_t words, slab;      // bit words per query, queries per slab (0: one kernel)
    FilterLayout f;
    size_t off_possible, off_g, off_d2, total;   // totals at 0
};
KnnLayout knn_layout(const trim_index_view *ix, int64_t nq, const trim_candidates *cand, int k, FinishPlan *fp) {
    KnnLayout L{};
    const int64_t hard = (int64_t(1) << 31) - 1 - TRIM_MAX_BATCH - 2048;
    int64_t mc = cand ? cand->max_candidates : ix->n;
    if (mc <= 0 || mc > ix->n + (int64_t)(cand ? cand->nprobe : 0) * ix->n || !worth_passes(ix, nq, cand) || !passes_fit(ix, cand, k, false, fp)) return L;
    if (mc > hard) mc = hard;
    L.words = (mc + 31) / 32 + 1;
    const size_t per = (size_t)L.words * (4 + 32 * 8) + 4 + filter_bytes_per_query(ix, cand);
    L.slab = std::min<int64_t>((int64_t)(kKnnSlabBytes / per), std::min<int64_t>(nq, 1 << 20));
    if (L.slab < 64 || !counts_fit(ix, L.slab, cand, mc)) { L.slab = 0; return L; }
    size_t off = up256((size_t)L.slab * 4);
    L.off_possible = off; off += up256((size_t)L.slab * L.words * 4);
    L.off_g = off;        off += up256((size_t)L.slab * L.words * 32 * 4);
    L.off_d2 = off;       off += up256((size_t)L.slab * L.words * 32 * 4);
    L.f = filter_layout(ix, L.slab, nq, cand, off);
    L.total = L.f.end;
    return L;
}

int knn_in_passes(const trim_index_view *ix, const KnnLayout &L, const SearchArgs &a, const FinishPlan &pl, unsigned char *ws,
                  hipStream_t st) {
    FinishArgs m{};
    fill_finish(m, pl, a);
    m.totals = reinterpret_cast<int32_t *>(ws);
    m.possible = reinterpret_cast<uint32_t *>(ws + L.off_possible);
    m.g = reinterpret_cast<float *>(ws + L.off_g);
    m.words = L.words;
    m.tau_stride = a.k;
    InvertArgs v{};
    FilterArgs f{};
    fill_filter(f, v, ix, a, L.f, ws);
    f.tau_stride = a.k; f.tau_of = a.out_d2 + (a.k - 1);
    f.totals = m.totals; f.possible = m.possible; f.words = L.words;
    f.d2 = reinterpret_cast<float *>(ws + L.off_d2);
    ReplayArgs y{};
    y.base = a.base; y.queries = a.queries; y.d = a.d;
    y.ids = a.ids; y.n = a.n; y.nq = a.nq; y.list_offsets = a.list_offsets; y.probes = a.probes; y.nlist = a.nlist;
    y.nseg = a.nseg; y.max_cand = a.max_cand; y.k = a.k; y.batch = a.batch; y.order = a.order; y.totals = m.totals;
    y.possible = m.possible; y.g = m.g; y.d2 = f.d2; y.words = L.words; y.out_ids = a.out_ids; y.out_d2 = a.out_d2;
    y.n_exact = a.n_exact; y.mask = a.mask; y.mask_words = a.mask_words;
    m.seg = y.seg = v.seg;
    const int64_t most = a.max_cand;
    for (int64_t s0 = 0; s0 < a.nq; s0 += L.slab) {
        const int64_t ns = a.nq - s0 < L.slab ? a.nq - s0 : L.slab;
        m.slot0 = y.slot0 = s0;
        m.nslots = y.nslots = ns;
        int rc;
        ZeroAreas z;
        z.add(m.possible, (size_t)ns * L.words);
        if (a.lut && s0 == 0) z.add(ws + L.f.off_bad, (size_t)a.nq);
        if ((rc = prepare_filter(f, v, s0, ns, z, st))) return rc;
        if ((rc = prepare_tables(m, ix, a, L.f, ws, st))) return rc;
        // The seed and the first batch (no threshold yet), then everything else against the
        // threshold that they leave.  Where that is no threshold to speak of yet (short first batches;
        // candidates in no particular order), eight times as many candidates from pass to pass.
        int64_t lo = 0, hi = (int64_t)a.k + a.batch;
        int first = 0;                  // the first batch's end, while it is not measured yet
        for (;;) {
            if (hi > most) hi = most;
            m.lo = y.lo = f.lo = (int)lo;
            m.hi = y.hi = f.hi = (int)hi;
            m.tau_of = lo > 0 ? a.out_d2 + (a.k - 1) : nullptr;
            m.all = lo == 0;            // (all of the first pass's candidates are bounded; after that the filter goes first)
            if (lo > 0 && (rc = launch_filter(f, st))) return rc;
            if ((rc = launch_finish(m, pl.vec, is_fs(ix), pl.threads, pl.lds, (ns + kXcds - 1) / kXcds * kXcds, st))) return rc;
            // With lists, the first batch is measured with the pass after it: other queries have that pass's rows in their first batch, so that
            // most rows were read twice.  In passes of its own / with the next, us: 500,000 x 768 (unit vectors, 64 of 1024 lists), 2,500
            // queries, k = 10, batches of 1024, gamma 0.6: 2063 / 1818; 211,000 x 768, 300 queries, gamma 0.35: 608 / 506; 200,000 x 960, 4-bit
            // codes, 300: 603 / 494.
            // The picked threshold exceeds the first batch's a little, which lets more be measured where many bounds lie just there: 64
            // picks, the same with gamma 0.3 3458 / 3493; 1,600 over 211,000 x 768, gamma 0.27: 2011 / 1997.  (One pick per result, 6 to 10 % more:
            // 3458 / 5330.)  More results take more picks than that: k = 12 3538 / 3602; with 128 picks, k = 16 2106 / 2131, 100 2783 / 3042.
            // Fewer results take fewer picks (k = 1, 32 / 64: 2,931 over 68,440 x 768 1183 / 1198).  Picks are work per query, what they save is rows read: 16
            // vectors a query (665 queries over 20,232 x 1536, 30 a query, 502 / 475; 2,931 over 68,440 x 768, 23, 1332 / 1272; 3,255 over
            // 61,802, 4-bit codes, 19, 1419 / 1331; 100,000 x 1536, groups far apart, 50 a query 1113 / 1124, 25 1710 / 1770, 12 3000 / 3119; 25,664 x 960, 10,
            // 822 / 823; at gamma 0.24, where many bounds lie about the threshold, 3,548 over 188,000 x 768 3928 / 4004).  Longer batches have more to measure
            // than to share (with 128 picks, 4000 over 150,000 x 1536, 1,100 queries: 2586 / 2663).
            // After a shorter batch the next pass is short too, and one pick per result will do whatever the number of queries: batches of 512, 600 over 211,000 x
            // 768, gamma 0.27 1315 / 1207, 2,000 of 1536 over 100,000, gamma 0.25 2689 / 2585; of 256, k = 50, 400 over 100,000 x 512 424 / 396.
            // Without lists the passes have no rows in common: 500 x 100,000 x 960, k = 10: 755 / 806.
            const bool brief = hi < 1024;
            if (lo == 0 && hi < most && a.nseg > 0 && a.batch <= kPickBatch &&
                (brief ? a.k <= kPickMost || (a.k <= kPicks && a.batch >= kPickGroup * a.k) : a.k <= kPickMost && a.nq * kPickVectors <= a.n)) {
                y.picks = brief ? a.k : std::min(kPickLong, 32 + 4 * a.k);
                first = (int)hi;
                y.mid = first;
                if ((rc = launch_pick(y, st))) return rc;
            } else {
                y.mid = first;
                if (first > 0) y.lo = f.lo = 0;
                first = 0;
                if ((rc = launch_measure(f, st))) return rc;
                if ((rc = launch_replay(y, st))) return rc;
            }
            if (hi >= most) break;
            lo = hi;
            if (a.nseg == 0 || hi < 1024) {
                hi = (int64_t)a.k + (hi - a.k) * 8;
                if (hi > most / 2) hi = most;
            } else {
                hi = most;
            }
        }
    }
    return TRIM_OK;
}

// Probe selection in two kernels (distances, selection): up to 64 probes, and few enough queries for one
// workgroup per 8 of them to leave CUs idle.
bool probe_in_two(int64_t nq, int d, int nlist, int nprobe) {
    return nprobe <= 64 && nprobe > 1 && nq <= 4096 && (size_t)8 * d * 4 <= kLdsBytes / 2 && nlist >= 64 &&
           (size_t)nq * nlist <= size_t(1) << 26;
}

// Queries per workgroup of ivf_probe_kernel: 8 (one per wave for the selection), fewer if their key arrays do not fit half of the
// LDS (so that two workgroups share a CU).
int probe_queries(int d, int nlist, int *npow2, size_t *lds) {
    *npow2 = 1;
    while (*npow2 < nlist && *npow2 < 1 << 30) *npow2 <<= 1;
    int qt = 8;
    while (qt > 1 && (size_t)qt * ((size_t)*npow2 * 8 + (size_t)d * 4) > kLdsBytes / 2) qt >>= 1;
    *lds = (size_t)qt * ((size_t)*npow2 * 8 + (size_t)d * 4);
    return qt;
}

// The nearest list of many vectors: scored on the matrix cores.  Below 4096 vectors fewer than 16
// workgroups would do it, and below 64 lists a 256-wide tile is mostly padding.
bool nearest_pays(int64_t nq, int d, int nlist) { return nq >= 4096 && nlist >= 64 && d <= kAsgMaxD; }
// Bytes of work space for it, 256-byte aligned, or 0 where it goes without.
size_t nearest_bytes(int64_t nq, int d, int nlist) {
    return nq > 0 && d > 0 && d % 4 == 0 && nlist > 0 && d <= kAsrCols && nearest_pays(nq, d, nlist) ? ast_layout(d, nlist).total : 0;
}
// Of the training of coarse lists: the update's, then the assignment's.
size_t train_ivf_bytes(int64_t ns, int d, int nlist) {
    const size_t near = nearest_bytes(ns, d, nlist), sorted = update_layout(ns, d, nlist, 1).total;
    return near > 0 ? up256(sorted) + near : sorted;
}
template <int KS>
int launch_tiles(const float *x, int64_t n, int d, const float *cent, int nlist, int32_t *out, unsigned char *ws, hipStream_t st) {
    const AstLayout L = ast_layout(d, nlist);
    AstHead *head = reinterpret_cast<AstHead *>(ws);
    uint32_t *most = reinterpret_cast<uint32_t *>(ws + L.off_most);
    uint4 *ops = reinterpret_cast<uint4 *>(ws + L.off_ops);
    hipLaunchKernelGGL(assign_operands_kernel<KS>, dim3((unsigned)L.nst), dim3(512), 0, st, cent, nlist, d, head, most, ops);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(assign_tiles_kernel<KS>, dim3((unsigned)((n + kAstVecs - 1) / kAstVecs)), dim3(kAstThreads), 0, st, x, n, d, cent,
                       nlist, L.nst, head, most, ops, out);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}
int launch_nearest(const float *x, int64_t n, int d, const float *cent, int nlist, int32_t *out, unsigned char *ws, hipStream_t st) {
    if (ws) {
        if (const int rc = d <= kAsrCols / 2 ? launch_tiles<4>(x, n, d, cent, nlist, out, ws, st) : launch_tiles<8>(x, n, d, cent, nlist, out, ws, st))
            return rc;
    } else {
        const size_t lds = assign_lds(d);
        void (*assign)(const float *, int64_t, int, const float *, int, int32_t *) = assign_mfma_kernel;
        if (d <= kAsrCols) assign = d <= kAsrCols / 2 ? assign_rows_kernel<4> : assign_rows_kernel<8>;
        else HIP_TRY(allow_lds(reinterpret_cast<const void *>(assign_mfma_kernel), lds));
        hipLaunchKernelGGL(assign, dim3((unsigned)((n + kAsgTile - 1) / kAsgTile)), dim3(kAsgThreads), d <= kAsrCols ? 0 : lds, st, x, n, d,
                           cent, nlist, out);
        HIP_TRY(hipGetLastError());
    }
    // the marked vectors
    const size_t lds = (size_t)8 * d * 4;
    int span = kFixSpan;
    while (span > 64 && n / span < 512) span >>= 1;     // (two workgroups per CU, where there are so many vectors)
    const int64_t blocks = (n + span - 1) / span;
    const bool one = d <= kAsrCols || d > 1024 || blocks < 400;      // (see assign_fix_kernel)
    void (*fix)(const float *, int64_t, int, const float *, int, int, int32_t *) = one ? assign_fix_kernel<1024> : assign_fix_kernel<512>;
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(fix), lds));
    hipLaunchKernelGGL(fix, dim3((unsigned)blocks), dim3(one ? 1024 : 512), lds, st, x, n, d, cent, nlist, span, out);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

// trim_ivf_probe; ws: null, or where nearest_bytes bytes are, for one probe.
int ivf_probe(const float *queries, int64_t nq, int d, const float *centroids, int nlist, int nprobe, int32_t *probes_out, unsigned char *ws,
              hipStream_t st) {
    if (nq < 0 || d <= 0 || nlist <= 0 || nprobe <= 0) return TRIM_INVALID_ARG;
    if (nprobe > nlist || nprobe > TRIM_MAX_NPROBE) return TRIM_INVALID_ARG;
    if (d % 4) return TRIM_UNSUPPORTED_SHAPE;
    int npow2;
    size_t lds;
    const int qt = probe_queries(d, nlist, &npow2, &lds);
    if (lds > kLdsBytes) return TRIM_UNSUPPORTED_SHAPE;
    if (nq == 0) return TRIM_OK;
    if (!queries || !centroids || !probes_out || !aligned16(centroids)) return TRIM_INVALID_ARG;
    if (nq > 0x7fffffff) return TRIM_INVALID_ARG;
    if (nprobe == 1 && nearest_pays(nq, d, nlist) && aligned16(queries)) return launch_nearest(queries, nq, d, centroids, nlist, probes_out, ws, st);
    void (*fn)(const float *, int64_t, int, const float *, int, int, int, int32_t *) =
        qt == 8 ? ivf_probe_kernel<8> : qt == 4 ? ivf_probe_kernel<4> : qt == 2 ? ivf_probe_kernel<2> : ivf_probe_kernel<1>;
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(fn), lds));
    // a launch holds fewer than 2^32 threads: walk the queries in slabs
    const int64_t slab = (int64_t)qt * (1 << 22);
    for (int64_t q0 = 0; q0 < nq; q0 += slab) {
        const int64_t cnt = nq - q0 < slab ? nq - q0 : slab;
        hipLaunchKernelGGL(fn, dim3((unsigned)((cnt + qt - 1) / qt)), dim3(512), lds, st,
                           queries + (size_t)q0 * d, cnt, d, centroids, nlist, npow2, nprobe,
                           probes_out + (size_t)q0 * nprobe);
        HIP_TRY(hipGetLastError());
    }
    return TRIM_OK;
}

// Sizes that a probe selection takes, whatever its work space.
bool probe_takes(int64_t nq, int d, int nlist, int nprobe) {
    int npow2;
    size_t lds;
    probe_queries(d, nlist, &npow2, &lds);
    return nq <= 0x7fffffff && (lds <= kLdsBytes || probe_in_two(nq, d, nlist, nprobe));
}

// The work space of a probe selection through the matrix cores (trim_probe.h); total = 0: another one.
struct ProbeLayout {
    int32_t dpad, lpad;
    int64_t slab;              // queries at a time: 256 MB of scores and operands
    size_t off_c, off_q, off_cpar, off_cnm, off_qpar, off_left, off_t, total;
};
ProbeLayout probe_layout(int64_t nq, int d, int nlist, int nprobe) {
    ProbeLayout L{};
    if (!probe_ranked_pays(nq, d, nlist, nprobe) || nprobe < 2 || nprobe > 64 || nlist > 65536 || d % 4 || d > 4096 ||
        (int64_t)nlist * d > int64_t(1) << 27 || !probe_takes(nq, d, nlist, nprobe)) return L;
    L.dpad = (d + 15) / 16 * 16;
    L.lpad = (nlist + kPrbCols - 1) / kPrbCols * kPrbCols;
    L.slab = std::min<int64_t>((nq + 31) / 32 * 32, std::max<int64_t>(32, (int64_t(1) << 26) / (L.lpad + L.dpad / 2) / 32 * 32));
    size_t off = 0;
    L.off_c = off;    off += up256((size_t)L.lpad * L.dpad * 2);
    L.off_q = off;    off += up256((size_t)L.slab * L.dpad * 2);
    L.off_cpar = off; off += up256((size_t)L.lpad * 16);
    L.off_cnm = off;  off += up256((size_t)L.lpad * 8);
    L.off_qpar = off; off += up256((size_t)L.slab * 16);
    L.off_left = off; off += up256((size_t)kPrbLefts * (kPrbApart + (L.slab + kPrbLefts - 1) / kPrbLefts) * 4);
    L.off_t = off;    off += up256((size_t)L.slab * L.lpad * 4);
    L.total = off + 256;       // (the caller's memory need not be aligned)
    return L;
}

int launch_probe_ranked(const float *queries, int64_t nq, int d, const float *cent, int nlist, int nprobe, int32_t *out,
                        const ProbeLayout &L, unsigned char *ws, hipStream_t st) {
    ProbeArgs a{};
    a.cent = cent; a.d = d; a.nlist = nlist; a.nprobe = nprobe; a.dpad = L.dpad; a.lpad = L.lpad;
    a.c16 = reinterpret_cast<_Float16 *>(ws + L.off_c);
    a.q16 = reinterpret_cast<_Float16 *>(ws + L.off_q);
    a.cpar = reinterpret_cast<float4 *>(ws + L.off_cpar);
    a.cnm = reinterpret_cast<float2 *>(ws + L.off_cnm);
    a.qpar = reinterpret_cast<float4 *>(ws + L.off_qpar);
    a.left = reinterpret_cast<uint32_t *>(ws + L.off_left);
    a.left_pitch = (L.slab + kPrbLefts - 1) / kPrbLefts;
    a.t = reinterpret_cast<float *>(ws + L.off_t);
    void (*nearest)(ProbeArgs) = d <= 128 ? probe_nearest_kernel<true> : probe_nearest_kernel<false>;
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(probe_operands_kernel), (size_t)L.dpad * 4));
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(nearest), (size_t)d * 4));
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(probe_rest_kernel), (size_t)8 * d * 4));
    for (int64_t q0 = 0; q0 < nq; q0 += L.slab) {
        a.nq = std::min<int64_t>(L.slab, nq - q0);
        a.queries = queries + (size_t)q0 * d;
        a.out = out + (size_t)q0 * nprobe;
        a.list_groups = q0 == 0 ? L.lpad / kGrRows : 0;
        const unsigned qblocks = (unsigned)((a.nq + 31) / 32);
        hipLaunchKernelGGL(probe_operands_kernel, dim3((unsigned)a.list_groups + qblocks * (32 / kGrRows)), dim3(256), (size_t)L.dpad * 4, st, a);
        hipLaunchKernelGGL(probe_scores_kernel, dim3((unsigned)(L.lpad / kPrbCols), qblocks), dim3(256), 0, st, a);
        hipLaunchKernelGGL(nearest, dim3((unsigned)a.nq), dim3(kWave), (size_t)d * 4, st, a);
        hipLaunchKernelGGL(probe_rest_kernel, dim3(kPrbRestGrid), dim3(kProbeThreads), (size_t)8 * d * 4, st, a);
        hipLaunchKernelGGL(probe_rest_select_kernel, dim3((unsigned)std::min<int64_t>(a.nq, kPrbRestGrid)), dim3(kWave), 0, st, a);
        HIP_TRY(hipGetLastError());
    }
    return TRIM_OK;
}

// Few queries: bound_kernel and settle_kernel (see trim_few.h).  They pay while the single kernel, a workgroup per
// query, leaves CUs idle (up to 128 queries; 256 where it is slowed by results of more than one entry per lane and the
// rows are short), and while the lookups of all candidates (it abandons most of them early) cost less than that: up to 500,000
// per value of a row, since long rows are what its workgroups wait for; but with short rows no more than 105 million, and
// without lists, where each of its workgroups has a long scan to overlap its waits with, no more than 250 million.
// Measured, single kernel / these two, us (k = 10 and gamma = 0.4 where nothing is said):
//   1M x 128, 32 of 1024 lists, 1 / 64 / 96 queries                79 / 46   100 / 96   100 / 121
//   500,000 x 384, 64 of 1024 (M = 48), 64 / 96                   109 / 89   110 / 121
//   800,000 x 384, 44 of 894, gamma 0.5, 16 / 48 / 96              77 / 63    85 / 114   85 / 175
//   800,000 x 256, 44 of 894 (M = 64), gamma 0.5, 16 / 48          98 / 71   105 / 149
//   500,000 x 768, 64 of 1024, 64 / 96                            620 / 460  638 / 558
//   100,000 x 768, 15 of 316, k = 100, 128 / 160 / 256            422 / 408  432 / 490  505 / 627
//   30,000 x 128, 8 of 173, k = 100, 256 queries: 0.78 of the single kernel's time; x 384: 1.0; x 1536: 1.39
//   30,000 x 960, no lists, 64 / 80 / 128                         357 / 311  355 / 403  357 / 457
// What is left on the wrong side: 800,000 x 384 and 256 at gamma 0.5, 30 to 55 queries, up to 1.4 times the single kernel's time
// (it abandons nearly everything early there, which depends on the data), 30,000 x 768 and 1536 from 96 queries on, up to 1.14.
//
// Over rows of 512 values and more settle_kernel stops at the first batch, and what its threshold leaves is measured by many workgroups and
// then replayed (few_rows_kernel): two launches more, 4 to 5 us.  Without / with, us (k = 10, gamma 0.3 where nothing is said):
//   200,000 x 768 (unit vectors), 30 of 450 lists, 1 / 33 / 128 queries     195 / 68    373 / 190   658 / 524;  k = 100, 33: 695 / 252
//   500,000 x 768, 20 of 700, gamma 0.1, 1 / 16 / 33 queries                978 / 103   1548 / 311  1703 / 483
//   100,000 x 1536, 30 of 300, 1 / 33, gamma 0.1; gamma 0.5                 1850 / 136  2705 / 863;   283 / 87   615 / 363
//   200,000 x 960, no lists, 1 / 4 queries                                  251 / 164   389 / 220
//   60,000 x 768, 16 of 256 lists that separate the data, 1 / 33 queries    33 / 39     80 / 89     (hardly anyone is left: two launches more)
// With fewer values it costs more than it gives: 500,000 x 384, 64 of 1024, 1 / 67 queries 30.7 / 34.7  74.5 / 83.1.
// Without lists the lookups may be more then, about as a root of the vectors (one workgroup per query takes longer and longer), and with
// more than 64 results, which hold the single kernel up more.  Single kernel / this, us, x 960: 40,000 vectors, 48 / 67 queries 330 / 303
// 330 / 391; 100,000, 22 290 / 311; 200,000, 16 / 22 541 / 385  547 / 576; 500,000, 10 / 16 840 / 775  858 / 827; k = 100: 40,000, 67 / 90
// 521 / 545  527 / 681; 200,000, 40 1022 / 1750, k = 128, gamma 0.1, 22 / 26 1171 / 1177  1163 / 1340; 400,000 x 768, k = 200, 20 2872 / 3205;
// k = 300, 200,000, 40 3547 / 2683.  200,000 x 768, k = 10, 20 queries, unit vectors 9143 / 2004, groups far apart 1115 / 286.
// With lists they may not: the single kernel passes over most of them where they separate the data, whatever their number (400,000 x 768, 150 of 256
// lists, gamma 0.5, 33 / 128 queries 257 / 425  305 / 1357; 200,000 x 960, 4-bit codes, 64 of 256: 209 / 271  263 / 902), and only vectors that no list
// separates gain (500,000 x 768, unit vectors, 150 of 256: 1867 / 567  2000 / 1916).
constexpr int64_t kFewQueries = 128, kFewQueriesWide = 256;
constexpr double kFewLookups = 500000.0, kFewShortRows = 1.05e8, kFewNoLists = 2.5e8;
constexpr size_t kFewBytes = size_t(1) << 30;
constexpr int64_t kFewOnePass = 4;
double few_pass_lookups(int64_t n, int k) {
    const double root = std::sqrt((double)n);
    if (k <= kWave) return std::min(2600.0 * (double)n, 1.05e6 * root);
    return std::min(7000.0 * (double)n, k <= 2 * kWave ? 8.2e6 * std::cbrt((double)n) : (k <= 4 * kWave ? 1.2e6 : 2.6e6) * root);
}
struct FewLayout {
    int64_t stride;           // bounds per query (0: not this way)
    size_t off_g, off_least, off_d2, total;      // totals at 0
    bool measure_first;
    // passes over long rows (r_stride 0: none); a work space that holds only the `least` bytes goes without
    int64_t r_stride;
    size_t off_all, off_rd2, off_rid, off_n, least;
};
FewLayout few_layout(const trim_index_view *ix, int64_t nq, const trim_candidates *cand, int k, int batch) {
    FewLayout L{};
    const int64_t mc = cand ? std::min<int64_t>(cand->max_candidates, (int64_t)cand->nprobe * ix->n) : ix->n;
    if (nq <= 0 || nq > (k > kWave && ix->d < kLongRow ? kFewQueriesWide : kFewQueries) || mc <= 0 || k + batch > kSettleFirst || k < 1 || batch < 1) return L;
    const double lookups = (double)nq * scanned_per_query(ix, cand) * ix->M;
    const bool fits = nq == 1 || !(lookups > kFewLookups * ix->d || (ix->d < kLongRow && lookups > kFewShortRows) || (!cand && lookups > kFewNoLists));
    const bool passes = ix->d >= kLongRow && mc > (int64_t)k + batch;
    if (!fits && !(passes && !cand && lookups <= few_pass_lookups(ix->n, k))) return L;
    const int64_t stride = (mc + 15) / 16 * 16;
    const size_t g_bytes = (size_t)nq * stride * 4;
    if ((size_t)stride > kFewBytes || g_bytes > kFewBytes || mc > 0x40000000 || !few_fits(ix->d, code_bytes(ix), is_fs(ix), k, cand ? cand->nprobe : 0)) return L;
    L.stride = stride;
    // The seed and the first batch measured beside the bounds, survivors or not, while that is little to read.
    L.measure_first = (size_t)nq * (k + batch) * ix->d * 4 <= (size_t(128) << 20);
    L.off_g = up256((size_t)nq * 4);
    L.off_least = L.off_g + up256(g_bytes);
    L.off_d2 = L.off_least + up256((size_t)nq * ((stride + 63) / 64) * 4);
    L.total = L.off_d2 + (L.measure_first ? up256((size_t)nq * (k + batch) * 4) : 0);
    L.least = fits ? L.total : 0;
    if (passes) {
        L.r_stride = kWave * result_slots(k);
        L.off_all = L.total;
        L.off_rd2 = L.off_all + up256(g_bytes);
        L.off_rid = L.off_rd2 + up256((size_t)nq * L.r_stride * 4);
        L.off_n = L.off_rid + up256((size_t)nq * L.r_stride * 4);
        L.total = L.off_n + up256((size_t)nq * 4);
        if (!fits) L.least = L.total;
    }
    return L;
}
int knn_few(const trim_index_view *ix, const FewLayout &L, const SearchArgs &a, unsigned char *ws, size_t ws_bytes, hipStream_t st) {
    FewArgs f{};
    f.base = a.base; f.codes = a.codes; f.dlx = a.dlx; f.codebooks = a.codebooks; f.ids = a.ids; f.n = a.n;
    f.d = a.d; f.M = a.M; f.dsub = a.dsub; f.queries = a.queries; f.nq = a.nq; f.order = a.order; f.lut = a.lut;
    f.list_offsets = a.list_offsets; f.probes = a.probes; f.nlist = a.nlist; f.nseg = a.nseg;
    f.max_cand = (int32_t)std::min<int64_t>(a.max_cand, L.stride);
    f.two_gamma = a.two_gamma; f.k = a.k; f.batch = a.batch;
    f.totals = reinterpret_cast<int32_t *>(ws);
    f.g = reinterpret_cast<float *>(ws + L.off_g);
    f.stride = L.stride;
    f.least = reinterpret_cast<float *>(ws + L.off_least);
    f.d2 = L.measure_first ? reinterpret_cast<float *>(ws + L.off_d2) : nullptr;
    f.out_ids = a.out_ids; f.out_d2 = a.out_d2; f.n_scanned = a.n_scanned; f.n_exact = a.n_exact;
    f.mask = a.mask; f.mask_words = a.mask_words;
    int rc;
    if ((rc = launch_bound(f, is_fs(ix), st))) return rc;
    if (L.r_stride == 0 || ws_bytes < L.total) return launch_settle(f, st);
    f.d2_all = reinterpret_cast<float *>(ws + L.off_all);
    f.r_d2 = reinterpret_cast<float *>(ws + L.off_rd2);
    f.r_id = reinterpret_cast<int32_t *>(ws + L.off_rid);
    f.r_n = reinterpret_cast<int32_t *>(ws + L.off_n);
    f.r_stride = (int32_t)L.r_stride;
    if ((rc = launch_settle(f, st))) return rc;
    // (passes begin where batches do)  After a short first batch, or without lists, the next eight times as far against its threshold,
    // the rest against a better one.  With lists and up to 4 queries that saves less than two launches more: passes / one, us: 200,000 x 960, 4-bit codes, 20 of 450
    // lists, gamma 0.5, batches of 256, 1 / 4 queries 60 / 52  76 / 70; 200,000 x 768, unit vectors, gamma 0.3 87 / 74  119 / 103; 8 at gamma 0.27, where
    // many bounds lie about the threshold: 145 / 151, 16 180 / 208.
    const int64_t most = f.max_cand;
    for (int64_t lo = (int64_t)a.k + a.batch, hi; lo < most; lo = hi) {
        hi = most;
        if (a.nseg == 0 || (lo < 1024 && a.nq > kFewOnePass)) {
            hi = (int64_t)a.k + (lo - a.k) * 8;
            if (hi > most / 2) hi = most;
        }
        f.lo = (int32_t)lo;
        f.hi = (int32_t)hi;
        if ((rc = launch_few_rows(f, st))) return rc;
        if ((rc = launch_settle(f, st))) return rc;
    }
    return TRIM_OK;
}

int search_knn(const trim_index_view *index, const float *queries, int64_t nq, const float *lut, const trim_candidates *cand,
               int32_t k, float gamma, int32_t batch, const int32_t *query_order, int32_t *out_ids, float *out_d2,
               const trim_stats *stats, uint32_t *survivor_mask, int64_t mask_words, void *workspace, size_t workspace_bytes,
               void *stream) {
    int rc = check_index(index);
    if (rc) return rc;
    if ((rc = check_cand(cand))) return rc;
    if (nq < 0 || nq > TRIM_MAX_QUERIES || k < 1 || k > TRIM_MAX_K || batch < 1 || batch > TRIM_MAX_BATCH)
        return TRIM_INVALID_ARG;
    if (!(gamma >= 0.0f) || std::isinf(gamma)) return TRIM_INVALID_ARG;
    if (nq == 0) return TRIM_OK;
    if (!queries || !out_ids || !out_d2) return TRIM_INVALID_ARG;
    if (!lut && !index->codebooks) return TRIM_INVALID_ARG;
    if (lut && !aligned16(lut)) return TRIM_INVALID_ARG;
    if (survivor_mask && mask_words <= 0) return TRIM_INVALID_ARG;
    Plan pl;
    const int cap = batch > k ? batch : k;
    if (!make_plan(index->d, code_bytes(index), is_fs(index), cand ? cand->nprobe : 0, cap, batch, k, false, nq, scanned_per_query(index, cand), &pl))
        return TRIM_UNSUPPORTED_SHAPE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (survivor_mask && (rc = fill_u32(survivor_mask, (size_t)nq * mask_words, 0u, st))) return rc;
    SearchArgs a{};
    fill_common(a, index, queries, lut, cand, gamma, stats, survivor_mask, mask_words, pl);
    a.k = k; a.batch = batch; a.radius2 = 0.0f;
    a.out_ids = out_ids; a.out_d2 = out_d2;
    a.chunk = 0; a.nsplit = 1;
    a.nq = nq; a.order = query_order;
    if (workspace && !a.work && (reinterpret_cast<uintptr_t>(workspace) & 255u) == 0 && aligned16(queries)) {
        const FewLayout F = few_layout(index, nq, cand, k, batch);
        if (F.stride > 0 && workspace_bytes >= F.least) return knn_few(index, F, a, static_cast<unsigned char *>(workspace), workspace_bytes, st);
        FinishPlan fp;
        const KnnLayout L = knn_layout(index, nq, cand, k, &fp);
        if (L.slab > 0 && workspace_bytes >= L.total && (!lut || lut_tiled(a.dsub, is_fs(index))))
            return knn_in_passes(index, L, a, fp, static_cast<unsigned char *>(workspace), st);
    }
    const int64_t slots = (nq + kXcds - 1) / kXcds * kXcds;
    if (slots * pl.threads >= (int64_t(1) << 32)) return TRIM_INVALID_ARG;  // threads per launch
    return launch_search(false, is_fs(index), a, pl, dim3((unsigned)slots, 1), st);
}

// The pass that writes the CSR arrays from the marks, distances and offsets that a search left in its work space.
int range_fill(const SearchArgs &a, const RangeLayout &L, unsigned char *ws, int32_t *out_ids, float *out_d2, int64_t capacity,
               hipStream_t st) {
    RangeFillArgs f{};
    f.base = a.base; f.ids = a.ids; f.queries = a.queries;
    f.list_offsets = a.list_offsets; f.probes = a.probes; f.n = a.n; f.d = a.d;
    f.nlist = a.nlist; f.nseg = a.nseg; f.max_cand = a.max_cand; f.chunk = L.chunk;
    f.nsplit = L.nsplit; f.result_mask = reinterpret_cast<uint32_t *>(ws); f.rmask_words = L.rmask_words;
    f.result_d2 = reinterpret_cast<float *>(ws + L.off_d2);
    f.chunk_base = reinterpret_cast<int64_t *>(ws + L.off_cbase);
    f.out_ids = out_ids; f.out_d2 = out_d2; f.capacity = capacity;
    const int nsegs = a.nseg > 0 ? a.nseg : 1;
    size_t off = 0;
    f.off_q = (uint32_t)off;
    f.off_segp = (uint32_t)off; off += up16((size_t)(nsegs + 1) * 4);
    f.off_segd = (uint32_t)off; off += up16((size_t)nsegs * 4);
    f.off_list = (uint32_t)off; off += 2048 * 4;
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(range_fill_kernel), off));
    hipLaunchKernelGGL(range_fill_kernel, dim3((unsigned)a.nq, (unsigned)L.nsplit), dim3(256), off, st, f);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

// Scratch of a range search in passes: totals, then the filter's operands.  0: such a search runs as one kernel.
size_t range_scratch_bytes(const trim_index_view *ix, int64_t nq, const trim_candidates *cand, FinishPlan *fp) {
    const int64_t mc = cand && cand->max_candidates > 0 ? cand->max_candidates : ix->n;
    if (!worth_passes(ix, nq, cand) || !passes_fit(ix, cand, 1, true, fp) || !counts_fit(ix, nq, cand, mc)) return 0;
    // (behind the filter's: a bit per query and candidate, who passes for certain)
    return filter_layout(ix, nq, nq, cand, up256((size_t)nq * 4)).end + up256((size_t)nq * range_layout(nq, mc).rmask_words * 4);
}

// The range search behind all entry points: `workspace` is the caller's buffer or this
// device's copy of the static scratch area; scratch: see range_scratch_bytes (or null).
int range_search(const trim_index_view *index, const float *queries, int64_t nq,
                 const float *lut, const trim_candidates *cand, float radius, float gamma,
                 const int32_t *query_order, int64_t *out_offsets, int32_t *out_ids,
                 float *out_d2, int64_t capacity,
                 int64_t *required, const trim_stats *stats, uint32_t *survivor_mask,
                 int64_t mask_words, void *workspace, size_t workspace_bytes, void *scratch, size_t scratch_bytes, void *stream) {
    int rc = check_index(index);
    if (rc) return rc;
    if ((rc = check_cand(cand))) return rc;
    if (nq < 0 || nq > TRIM_MAX_QUERIES || capacity < 0) return TRIM_INVALID_ARG;
    if (!(gamma >= 0.0f) || std::isinf(gamma) || !(radius >= 0.0f)) return TRIM_INVALID_ARG;
    if (!out_offsets) return TRIM_INVALID_ARG;
    if (capacity > 0 && (!out_ids || !out_d2)) return TRIM_INVALID_ARG;
    if (lut && !aligned16(lut)) return TRIM_INVALID_ARG;
    if (!lut && !index->codebooks) return TRIM_INVALID_ARG;
    if (survivor_mask && mask_words <= 0) return TRIM_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (nq == 0) {
        if ((rc = fill_u32(reinterpret_cast<uint32_t *>(out_offsets), 2, 0u, st))) return rc;
        if (required && (rc = fill_u32(reinterpret_cast<uint32_t *>(required), 2, 0u, st))) return rc;
        return TRIM_OK;
    }
    if (!queries) return TRIM_INVALID_ARG;
    int64_t max_cand = cand ? cand->max_candidates : index->n;
    if (cand && max_cand <= 0) return TRIM_INVALID_ARG;  // needed to size the masks
    const RangeLayout L = range_layout(nq, max_cand);
    if (!workspace || workspace_bytes < L.total || (reinterpret_cast<uintptr_t>(workspace) & 255u))
        return TRIM_WORKSPACE;
    Plan pl;
    if (!make_plan(index->d, code_bytes(index), is_fs(index), cand ? cand->nprobe : 0, kRangeRound, kRangeRound, 1, true, nq, 0.0, &pl))
        return TRIM_UNSUPPORTED_SHAPE;

    unsigned char *ws = static_cast<unsigned char *>(workspace);
    uint32_t *rmask = reinterpret_cast<uint32_t *>(ws);
    int32_t *counts = reinterpret_cast<int32_t *>(ws + L.off_counts);
    int64_t *cbase = reinterpret_cast<int64_t *>(ws + L.off_cbase);
    float *rd2 = reinterpret_cast<float *>(ws + L.off_d2);

    ZeroAreas z;
    z.add(rmask, (size_t)nq * L.rmask_words);
    z.add(survivor_mask, (size_t)nq * mask_words);
    if (stats) {
        z.add(stats->n_exact, (size_t)nq);
        z.add(stats->work, (size_t)nq * kWorkCounters);
    }

    SearchArgs a{};
    fill_common(a, index, queries, lut, cand, gamma, stats, survivor_mask, mask_words, pl);
    a.k = 1; a.batch = kRangeRound;
    a.radius2 = radius * radius;
    a.chunk = L.chunk; a.nsplit = L.nsplit;
    a.result_mask = rmask; a.rmask_words = L.rmask_words; a.chunk_counts = counts;
    a.result_d2 = rd2;
    a.order = query_order;
    if (a.max_cand > max_cand) a.max_cand = (int32_t)max_cand;

    a.nq = nq;
    FinishPlan fpl, whole;
    const size_t want = range_scratch_bytes(index, nq, cand, &fpl);
    if (scratch && want > 0 && scratch_bytes >= want && !a.work && (reinterpret_cast<uintptr_t>(scratch) & 255u) == 0 &&
        aligned16(queries) && (!lut || lut_tiled(a.dsub, is_fs(index)))) {
        unsigned char *sc = static_cast<unsigned char *>(scratch);
        // (rows of the work space by query number; a query that the order does not name has no candidates)
        if (query_order) z.add(sc, (size_t)nq);
        z.add(counts, (size_t)nq * L.nsplit);
        InvertArgs v{};
        FilterArgs fa{};
        const FilterLayout FL = filter_layout(index, nq, nq, cand, up256((size_t)nq * 4));
        fill_filter(fa, v, index, a, FL, sc);
        fa.by_query = v.by_query = 1;
        fa.range = 1; fa.radius2 = a.radius2; fa.lo = 0; fa.hi = a.max_cand;
        fa.totals = reinterpret_cast<int32_t *>(sc); fa.possible = rmask; fa.words = L.rmask_words; fa.d2 = rd2;
        // (out of this range nobody passes for certain: see filter_kernel)
        const bool some = a.radius2 > kCertainLow && a.radius2 < kCertainHigh;
        make_finish_plan(index->d, code_bytes(index), is_fs(index), a.nseg, false, &whole);      // (it fits where the other one does)
        if (!some) fpl = whole;
        fa.certain = some ? reinterpret_cast<uint32_t *>(sc + FL.end) : nullptr;
        z.add(fa.certain, (size_t)nq * L.rmask_words);
        FinishArgs m{};
        fill_finish(m, fpl, a);
        m.certain = fa.certain;
        m.slot0 = 0; m.nslots = nq; m.by_query = 1; m.range = 1; m.radius2 = a.radius2; m.lo = 0; m.hi = a.max_cand;
        m.totals = reinterpret_cast<int32_t *>(sc); m.possible = rmask; m.words = L.rmask_words; m.g = rd2;
        m.n_exact = a.n_exact; m.mask = a.mask; m.mask_words = a.mask_words;
        ReplayArgs y{};
        y.base = a.base; y.queries = a.queries; y.d = a.d; y.n = a.n; y.nq = nq; y.list_offsets = a.list_offsets;
        y.probes = a.probes; y.nlist = a.nlist; y.nseg = a.nseg; y.max_cand = a.max_cand; y.order = query_order;
        y.totals = m.totals; y.bits = rmask; y.d2_out = rd2; y.words = L.rmask_words; y.radius2 = a.radius2;
        y.chunk = L.chunk; y.nchunk = L.nsplit; y.counts = counts;
        m.seg = y.seg = v.seg;
        if (a.lut) z.add(sc + FL.off_bad, (size_t)nq);
        if ((rc = prepare_filter(fa, v, 0, nq, z, st))) return rc;
        if ((rc = prepare_tables(m, index, a, FL, sc, st))) return rc;
        // candidates per query: the filter needs them before the finish pass writes them
        if ((rc = launch_totals(m, st))) return rc;
        if ((rc = launch_filter(fa, st))) return rc;
        // A caller's table that is not the centroids': every sum of that query is wanted, and the plan for few sums is the wrong one
        // (1,000 queries x 100,000 x 1536, all of them so: 2177 us by it, 1851 by a launch with the other; 2,000 x 200,000 x 768 in 192
        // subspaces 4504 / 3388).  The host does not see which: both launches, of which the second costs 2 to 9 us where there are none.
        const int64_t slots = (nq + kXcds - 1) / kXcds * kXcds;
        const bool both = m.bad && some && whole.P != fpl.P;
        m.only = both ? kFinishGood : 0;
        if ((rc = launch_finish(m, fpl.vec, is_fs(index), fpl.threads, fpl.lds, slots, st))) return rc;
        if (both) {
            fill_plan(m, whole);
            m.certain = nullptr;
            m.only = kFinishBad;
            if ((rc = launch_finish(m, whole.vec, is_fs(index), whole.threads, whole.lds, slots, st))) return rc;
        }
        if ((rc = launch_measure(fa, st))) return rc;
        if ((rc = launch_range_exact(y, nq, L.nsplit, st))) return rc;
    } else {
        // a query that the order does not name is not searched: its counts must read zero
        if (query_order) z.add(counts, (size_t)nq * L.nsplit);
        if ((rc = zero_areas(z, st))) return rc;
        const int64_t slots = (nq + kXcds - 1) / kXcds * kXcds;
        if (slots * pl.threads >= (int64_t(1) << 32)) return TRIM_INVALID_ARG;  // threads per launch
        if ((rc = launch_search(true, is_fs(index), a, pl, dim3((unsigned)slots, (unsigned)L.nsplit), st))) return rc;
    }
    hipLaunchKernelGGL(range_offsets_kernel, dim3(1), dim3(1024), 0, st, counts, nq, L.nsplit, cbase,
                       out_offsets, required);
    HIP_TRY(hipGetLastError());
    if (capacity > 0) return range_fill(a, L, ws, out_ids, out_d2, capacity, st);
    return TRIM_OK;
}

// The CSR arrays of a search that has been counted (trim_range_collect).
int range_collect(const trim_index_view *index, int64_t nq, const trim_candidates *cand, int32_t *out_ids, float *out_d2,
                  int64_t capacity, void *workspace, size_t workspace_bytes, void *stream) {
    int rc = check_index(index);
    if (rc) return rc;
    if ((rc = check_cand(cand))) return rc;
    if (nq < 0 || nq > TRIM_MAX_QUERIES || capacity < 0) return TRIM_INVALID_ARG;
    if (nq == 0 || capacity == 0) return TRIM_OK;
    if (!out_ids || !out_d2) return TRIM_INVALID_ARG;
    const int64_t max_cand = cand ? cand->max_candidates : index->n;
    if (cand && max_cand <= 0) return TRIM_INVALID_ARG;
    const RangeLayout L = range_layout(nq, max_cand);
    if (!workspace || workspace_bytes < L.total || (reinterpret_cast<uintptr_t>(workspace) & 255u)) return TRIM_WORKSPACE;
    SearchArgs a{};
    Plan pl{};
    fill_common(a, index, nullptr, nullptr, cand, 0.0f, nullptr, nullptr, 0, pl);
    a.nq = nq;
    if (a.max_cand > max_cand) a.max_cand = (int32_t)max_cand;
    return range_fill(a, L, static_cast<unsigned char *>(workspace), out_ids, out_d2, capacity, static_cast<hipStream_t>(stream));
}

// The work space of a gamma estimate through the matrix cores (trim_gamma.h): vectors in chunks whose keys take
// at most 400 MB.  total = 0: gamma_kernel computes every value: few pairs of long rows, whose operands cost more than they save
// (S Q < 100 d; 100 x 500 x 768: 47 against 42 us, 100 x 1000 x 768: 50 against 57, 100 x 500 x 384: 33 against 35).
struct GammaLayout {
    int32_t chunk, dpad, qpad;
    size_t off_l, off_u, off_q, off_vpar, off_qpar, off_keys, off_lists, total;
};
GammaLayout gamma_layout(int32_t d, int32_t S, int32_t Q) {
    GammaLayout L{};
    if (d <= 0 || S <= 0 || Q <= 0 || Q > 16384 || (int64_t)S * Q < 100 * (int64_t)d) return L;
    L.dpad = (d + 15) / 16 * 16;
    L.qpad = (Q + kGrQueries - 1) / kGrQueries * kGrQueries;
    if (gamma_rank_lds(d) + 1024 > kLdsBytes || (size_t)L.dpad * 4 + 8192 > kLdsBytes) return L;
    const int64_t most = std::max<int64_t>(32, (int64_t(1) << 26) / L.qpad / 32 * 32);
    L.chunk = (int32_t)std::min<int64_t>(most, ((int64_t)S + 31) / 32 * 32);
    size_t off = 0;
    L.off_l = off;    off += up256((size_t)L.chunk * L.dpad * 2);
    L.off_u = off;    off += up256((size_t)L.chunk * L.dpad * 2);
    L.off_q = off;    off += up256((size_t)L.qpad * L.dpad * 2);
    L.off_vpar = off; off += up256((size_t)L.chunk * 32);
    L.off_qpar = off; off += up256((size_t)L.qpad * 16);
    L.off_keys = off; off += up256((size_t)L.chunk * L.qpad * 2);
    L.off_lists = off; off += (size_t)L.chunk * L.qpad * 4;
    L.total = off;
    return L;
}

int launch_gamma_ranked(const GammaArgs &g, const GammaLayout &L, unsigned char *ws, hipStream_t st) {
    GammaRankArgs a{};
    a.g = g;
    a.dpad = L.dpad; a.qpad = L.qpad;
    a.l16 = reinterpret_cast<_Float16 *>(ws + L.off_l);
    a.u16 = reinterpret_cast<_Float16 *>(ws + L.off_u);
    a.q16 = reinterpret_cast<_Float16 *>(ws + L.off_q);
    a.vpar = reinterpret_cast<float *>(ws + L.off_vpar);
    a.qpar = reinterpret_cast<float4 *>(ws + L.off_qpar);
    a.keys = reinterpret_cast<uint16_t *>(ws + L.off_keys);
    a.lists = reinterpret_cast<uint32_t *>(ws + L.off_lists);
    const size_t lds_mu = (size_t)L.dpad * 4, lds_rank = gamma_rank_lds(g.d);
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(gamma_operands_kernel), lds_mu));
    const int threads = L.chunk <= 512 ? 512 : 256;
    void (*rank)(GammaRankArgs) = threads == 512 ? gamma_rank_kernel<512> : gamma_rank_kernel<256>;
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(rank), lds_rank));
    for (int64_t s0 = 0; s0 < g.S; s0 += L.chunk) {
        a.s0 = (int32_t)s0;
        a.ns = (int32_t)std::min<int64_t>(L.chunk, g.S - s0);
        a.vector_blocks = (a.ns + 31) / 32;
        const int groups = a.vector_blocks * (32 / kGrRows) + (s0 == 0 ? L.qpad / kGrRows : 0);
        hipLaunchKernelGGL(gamma_operands_kernel, dim3((unsigned)groups), dim3(256), lds_mu, st, a);
        HIP_TRY(hipGetLastError());
        hipLaunchKernelGGL(gamma_bins_kernel, dim3((unsigned)(L.qpad / kGrQueries), (unsigned)a.vector_blocks), dim3(256), 0, st, a);
        HIP_TRY(hipGetLastError());
        hipLaunchKernelGGL(rank, dim3((unsigned)a.ns), dim3(threads), lds_rank, st, a);
        HIP_TRY(hipGetLastError());
    }
    return TRIM_OK;
}

}  // namespace

extern "C" {

int trim_shape_supported(int32_t d, int32_t M) {
    Plan pl;
    if (d <= 0 || M <= 0 || d % M) return 0;
    return make_plan(d, M, false, 64, 2048, 2048, 10, true, 1, 0.0, &pl) ? 1 : 0;
}

int trim_fs_shape_supported(int32_t d, int32_t M) {
    Plan pl;
    if (d <= 0 || M <= 0 || M % 2 || d % M) return 0;
    return make_plan(d, M / 2, true, 64, 2048, 2048, 10, true, 1, 0.0, &pl) ? 1 : 0;
}

int trim_encode(const float *base, int64_t n, int32_t d, const float *codebooks, int32_t M,
                uint8_t *codes_out, float *dlx_out, void *stream) {
    if (n < 0 || d <= 0 || M <= 0) return TRIM_INVALID_ARG;
    if (d % M || M % 4) return TRIM_UNSUPPORTED_SHAPE;
    const int dsub = d / M;
    if ((size_t)kC * dsub * 4 > 64 * 1024) return TRIM_UNSUPPORTED_SHAPE;
    if (n == 0) return TRIM_OK;
    if (!base || !codebooks || !codes_out || !dlx_out) return TRIM_INVALID_ARG;
    if (reinterpret_cast<uintptr_t>(codes_out) & 3u) return TRIM_INVALID_ARG;
    return encode_codes(base, n, d, codebooks, M, codes_out, 0, dlx_out, static_cast<hipStream_t>(stream));
}

size_t trim_list_bounds_bytes(int32_t nlist, int32_t M) {
    if (nlist <= 0 || M <= 0) return 0;
    return (size_t)nlist * list_record_bytes(M);
}

int trim_pack_list_bounds(const trim_index_view *index, const int64_t *list_offsets, int32_t nlist,
                          void *out, void *stream) {
    const int rc = check_index(index);
    if (rc != TRIM_OK) return rc;
    if (nlist <= 0 || !list_offsets || !out || !aligned16(out)) return TRIM_INVALID_ARG;
    const int Mb = code_bytes(index);   // summaries are kept per code byte
    // 256 threads a list where the lists are many and short: 1024 are for the longest ones of a thousand (us, 1024 / 256 threads, vectors x
    // code bytes in lists: 200,000 x 32 in 16384 145 / 75, in 4096 44 / 29, in 2048 25 / 19, in 1024 17 / 17; 1,000,000 x 32 in 4096 52 / 40, in
    // 1024 33 / 51; 60,000 x 96 in 4096 67 / 55, in 1024 25 / 31; 30,000 x 32 in 1024 13 / 11, 20,000 x 192 in 1024 35 / 45).
    const bool narrow = (double)index->n * Mb < 2.5 * nlist * nlist;
    void (*fn)(const uint8_t *, const float *, int64_t, int, const int64_t *, uint8_t *) = narrow ? list_bounds_kernel<256> : list_bounds_kernel<1024>;
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(fn), (size_t)Mb * kBoundsPitch * 4));
    hipLaunchKernelGGL(fn, dim3((unsigned)nlist), dim3(narrow ? 256 : 1024), (size_t)Mb * kBoundsPitch * 4,
                       static_cast<hipStream_t>(stream), index->codes, index->dlx, index->n, Mb,
                       list_offsets, static_cast<uint8_t *>(out));
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

int trim_ceiling_stream_read(const void *buf, size_t bytes, int32_t blocks, uint32_t *sink,
                             void *stream) {
    if (!buf || !sink || bytes < 16 || (reinterpret_cast<uintptr_t>(buf) & 15u)) return TRIM_INVALID_ARG;
    if (blocks < 1 || blocks > TRIM_CEILING_MAX_BLOCKS) return TRIM_INVALID_ARG;
    hipLaunchKernelGGL(stream_read_kernel, dim3(blocks), dim3(512), 0,
                       static_cast<hipStream_t>(stream), static_cast<const uint4 *>(buf), bytes / 16,
                       sink);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

int trim_ceiling_lds_gather(int32_t blocks, int32_t iters, int32_t entry_floats, uint32_t seed,
                            float *sink, void *stream) {
    if (!sink || iters < 1 || iters > (1 << 20)) return TRIM_INVALID_ARG;
    if (blocks < 1 || blocks > TRIM_CEILING_MAX_BLOCKS) return TRIM_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    switch (entry_floats) {
        case 1:
            hipLaunchKernelGGL(lds_gather_kernel, dim3(blocks), dim3(512), 32 * kC * 4, st, iters, seed, sink);
            break;
        case 2:
            hipLaunchKernelGGL(lds_gather_wide_kernel<2>, dim3(blocks), dim3(512), 8 * kC * 8, st, iters, seed, sink);
            break;
        case 4:
            hipLaunchKernelGGL(lds_gather_wide_kernel<4>, dim3(blocks), dim3(512), 8 * kC * 16, st, iters, seed, sink);
            break;
        case 16:
            hipLaunchKernelGGL(lds_gather_fs_kernel, dim3(blocks), dim3(512), 64 * kC4 * 4, st, iters, seed, sink);
            break;
        default:
            return TRIM_INVALID_ARG;
    }
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

int trim_pack_scan_head(const uint8_t *codes, const float *dlx, int64_t n, int32_t M,
                        void *head_out, void *stream) {
    if (n < 0 || n >= (int64_t(1) << 31) || M <= 0) return TRIM_INVALID_ARG;
    if (M % 8) return TRIM_UNSUPPORTED_SHAPE;
    if (n == 0) return TRIM_OK;
    if (!codes || !dlx || !head_out) return TRIM_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(codes) & 7u) || (reinterpret_cast<uintptr_t>(head_out) & 3u))
        return TRIM_INVALID_ARG;
    size_t blocks = ((size_t)n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(pack_scan_head_kernel, dim3((unsigned)blocks), dim3(256), 0,
                       static_cast<hipStream_t>(stream), codes, dlx, n, M,
                       static_cast<uint32_t *>(head_out));
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

int trim_train_pq(const float *train, int64_t ns, int32_t d, int32_t M, int32_t iters,
                  const int32_t *init_rows, float *codebooks_out, uint8_t *codes_ws, float *dlx_ws,
                  void *stream) {
    return trim_train_pq_ws(train, ns, d, M, iters, init_rows, codebooks_out, codes_ws, dlx_ws, nullptr, 0, stream);
}

size_t trim_train_pq_workspace_bytes(int64_t ns, int32_t d, int32_t M) {
    if (ns <= 0 || d <= 0 || M <= 0 || d % M) return 0;
    const UpdateLayout L = update_layout(ns, d / M, kC, M);
    return L.total > 0 ? L.total + 256 : 0;
}

int trim_train_pq_ws(const float *train, int64_t ns, int32_t d, int32_t M, int32_t iters,
                     const int32_t *init_rows, float *codebooks_out, uint8_t *codes_ws, float *dlx_ws,
                     void *workspace, size_t workspace_bytes, void *stream) {
    if (ns <= 0 || d <= 0 || M <= 0 || iters < 0) return TRIM_INVALID_ARG;
    if (d % M || M % 4 || M > 65535) return TRIM_UNSUPPORTED_SHAPE;
    if (!train || !init_rows || !codebooks_out || !codes_ws || !dlx_ws) return TRIM_INVALID_ARG;
    const int dsub = d / M;
    if (iters > 0 && (size_t)kC * dsub * 4 > 64 * 1024) return TRIM_UNSUPPORTED_SHAPE;
    if (iters > 0 && (reinterpret_cast<uintptr_t>(codes_ws) & 3u)) return TRIM_INVALID_ARG;
    const UpdateLayout L = update_layout(ns, dsub, kC, M);
    unsigned char *ws = update_space(workspace, workspace_bytes, L.total);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int per = kC * dsub;  // centroid coordinates per subspace
    hipLaunchKernelGGL(kmeans_init_kernel, dim3((per + 255) / 256, M), dim3(256), 0, st, train, ns, (int64_t)d, dsub,
                       init_rows, kC, codebooks_out);
    HIP_TRY(hipGetLastError());
    if (const int rc = iters > 0 ? kmeans_columns(train, ns, d, dsub, M, L, ws, st) : TRIM_OK) return rc;
    for (int it = 0; it < iters; ++it) {
        // The codes and landmark distances that the caller sees are the last iteration's; before that the codes are laid out for
        // the update, subspace by subspace (a workgroup reads 64 KB of 2 MB; row by row every one brings all of it in).
        const bool last = it + 1 == iters;
        int rc = encode_codes(train, ns, d, codebooks_out, M, codes_ws, last ? 0 : ns, last ? dlx_ws : nullptr, st);
        if (rc) return rc;
        if ((rc = kmeans_update<1>(train, ns, d, dsub, codes_ws, last ? M : 1, last ? 1 : ns, kC, M, codebooks_out, ws, st))) return rc;
    }
    return TRIM_OK;
}

int trim_train_ivf(const float *train, int64_t ns, int32_t d, int32_t nlist, int32_t iters,
                   const int32_t *init_rows, float *centroids_out, int32_t *assign_ws, void *stream) {
    return trim_train_ivf_ws(train, ns, d, nlist, iters, init_rows, centroids_out, assign_ws, nullptr, 0, stream);
}

size_t trim_train_ivf_workspace_bytes(int64_t ns, int32_t d, int32_t nlist) {
    const size_t need = train_ivf_bytes(ns, d, nlist);
    return need > 0 ? need + 256 : 0;
}

int trim_train_ivf_ws(const float *train, int64_t ns, int32_t d, int32_t nlist, int32_t iters,
                      const int32_t *init_rows, float *centroids_out, int32_t *assign_ws, void *workspace, size_t workspace_bytes,
                      void *stream) {
    if (ns <= 0 || d <= 0 || nlist <= 0 || iters < 0) return TRIM_INVALID_ARG;
    if (d % 4) return TRIM_UNSUPPORTED_SHAPE;
    if (!train || !init_rows || !centroids_out || !assign_ws) return TRIM_INVALID_ARG;
    if ((int64_t)nlist * d > 0x7fffffff) return TRIM_UNSUPPORTED_SHAPE;
    const UpdateLayout L = update_layout(ns, d, nlist, 1);
    unsigned char *ws = update_space(workspace, workspace_bytes, train_ivf_bytes(ns, d, nlist));
    unsigned char *sorted = L.total > 0 ? ws : nullptr, *near = ws && nearest_bytes(ns, d, nlist) > 0 ? ws + up256(L.total) : nullptr;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int per = nlist * d;
    hipLaunchKernelGGL(kmeans_init_kernel, dim3((per + 255) / 256), dim3(256), 0, st, train, ns, (int64_t)d, d, init_rows,
                       nlist, centroids_out);
    HIP_TRY(hipGetLastError());
    for (int it = 0; it < iters; ++it) {
        int rc = ivf_probe(train, ns, d, centroids_out, nlist, 1, assign_ws, near, st);
        if (rc) return rc;
        if ((rc = kmeans_update<4>(train, ns, d, d, assign_ws, 1, 0, nlist, 1, centroids_out, sorted, st))) return rc;
    }
    return TRIM_OK;
}

int trim_estimate_gamma(const trim_index_view *index, const int32_t *sample_rows, int32_t S,
                        const float *sample_queries, int32_t Q, float p, float *gamma_x_out,
                        float *gamma_out, void *stream) {
    return trim_estimate_gamma_ws(index, sample_rows, S, sample_queries, Q, p, gamma_x_out, gamma_out, nullptr, 0, stream);
}

size_t trim_estimate_gamma_workspace_bytes(int32_t d, int32_t S, int32_t Q) {
    return gamma_layout(d, S, Q).total;
}

int trim_estimate_gamma_ws(const trim_index_view *index, const int32_t *sample_rows, int32_t S,
                           const float *sample_queries, int32_t Q, float p, float *gamma_x_out,
                           float *gamma_out, void *workspace, size_t workspace_bytes, void *stream) {
    if (!index || index->n <= 0 || index->d <= 0 || index->M <= 0) return TRIM_INVALID_ARG;
    if (index->code_bits == 4) return TRIM_UNSUPPORTED_SHAPE;   // 8-bit landmark codes only
    if (index->d % 4 || index->d % index->M) return TRIM_UNSUPPORTED_SHAPE;
    if (S <= 0 || Q <= 0 || !(p >= 0.0f && p <= 1.0f)) return TRIM_INVALID_ARG;
    if (Q > 16384) return TRIM_UNSUPPORTED_SHAPE;
    if (!index->base || !index->codes || !index->codebooks || !sample_rows || !sample_queries || !gamma_out)
        return TRIM_INVALID_ARG;
    if (!aligned16(sample_queries)) return TRIM_INVALID_ARG;
    const int per = S > 1 && gamma_lds(2, index->d, Q) + 1024 <= kLdsBytes ? 2 : 1;
    const size_t lds = gamma_lds(per, index->d, Q);
    if (lds + 1024 > kLdsBytes) return TRIM_UNSUPPORTED_SHAPE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    GammaArgs a{};
    a.base = index->base; a.codes = index->codes; a.codebooks = index->codebooks;
    a.rows = sample_rows; a.queries = sample_queries; a.n = index->n; a.d = index->d; a.M = index->M;
    a.S = S; a.Q = Q;
    long m = (long)std::ceil((double)p * (double)Q);
    if (m < 1) m = 1;
    if (m > Q) m = Q;
    a.rank = (int32_t)(Q - m);
    a.gamma_x = gamma_x_out; a.gamma_bits = reinterpret_cast<uint32_t *>(gamma_out);
    const GammaLayout L = gamma_layout(index->d, S, Q);
    if (workspace && L.total > 0 && workspace_bytes >= L.total && (reinterpret_cast<uintptr_t>(workspace) & 255u) == 0)
        return launch_gamma_ranked(a, L, static_cast<unsigned char *>(workspace), st);
    int rc = fill_u32(reinterpret_cast<uint32_t *>(gamma_out), 1, 0x7f800000u, st);  // +inf
    if (rc) return rc;
    void (*fn)(GammaArgs) = per == 2 ? gamma_kernel<2> : gamma_kernel<1>;
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(fn), lds));
    hipLaunchKernelGGL(fn, dim3((unsigned)((S + per - 1) / per)), dim3(kGammaThreads), lds, st, a);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

int trim_estimate_gamma_normal(const trim_index_view *index, const int32_t *sample_rows, int32_t S,
                               const float *normals, int32_t Q, float p, int32_t grid, double *work,
                               float *gamma_x_out, float *gamma_out, void *stream) {
    if (!index || index->n <= 0 || index->d <= 0 || index->M <= 0) return TRIM_INVALID_ARG;
    if (index->code_bits == 4) return TRIM_UNSUPPORTED_SHAPE;   // 8-bit landmark codes only
    if (index->d % index->M || index->d < 3) return TRIM_UNSUPPORTED_SHAPE;
    if (S <= 0 || Q <= 0 || grid < 2 || !(p >= 0.0f && p <= 1.0f)) return TRIM_INVALID_ARG;
    if (Q > 16384 || grid > (1 << 24)) return TRIM_UNSUPPORTED_SHAPE;
    if (!index->base || !index->codes || !index->codebooks || !sample_rows || !normals || !work || !gamma_out)
        return TRIM_INVALID_ARG;
    if (reinterpret_cast<uintptr_t>(work) & 7u) return TRIM_INVALID_ARG;
    int npow2 = 1;
    while (npow2 < Q) npow2 <<= 1;
    const size_t lds = (size_t)npow2 * 8;
    hipStream_t st = static_cast<hipStream_t>(stream);
    int rc = fill_u32(reinterpret_cast<uint32_t *>(gamma_out), 1, 0x7f800000u, st);  // +inf
    if (rc) return rc;
    hipLaunchKernelGGL(normal_triples_kernel, dim3((unsigned)((Q + 255) / 256)), dim3(256), 0, st, normals,
                       (int64_t)Q, index->d, work);
    HIP_TRY(hipGetLastError());
    GammaNormalArgs a{};
    a.base = index->base; a.codes = index->codes; a.codebooks = index->codebooks; a.rows = sample_rows;
    a.triples = work; a.n = index->n; a.d = index->d; a.M = index->M; a.Q = Q; a.npow2 = npow2;
    a.grid = grid; a.one_minus_p = 1.0 - (double)p;
    a.gamma_x = gamma_x_out; a.gamma_bits = reinterpret_cast<uint32_t *>(gamma_out);
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(gamma_normal_kernel), lds));
    hipLaunchKernelGGL(gamma_normal_kernel, dim3((unsigned)S), dim3(256), lds, st, a);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

size_t trim_codes_tiled_bytes(int64_t n, int32_t M) {
    if (n <= 0 || M <= 0) return 0;
    return (size_t)((n + 63) / 64) * 64 * (size_t)M;
}

int trim_pack_codes_tiled(const uint8_t *codes, int64_t n, int32_t M, void *tiled_out, void *stream) {
    if (n < 0 || n >= (int64_t(1) << 31) || M <= 0) return TRIM_INVALID_ARG;
    if (M % 16) return TRIM_UNSUPPORTED_SHAPE;
    if (n == 0) return TRIM_OK;
    if (!codes || !tiled_out || !aligned16(codes) || !aligned16(tiled_out)) return TRIM_INVALID_ARG;
    const size_t total = trim_codes_tiled_bytes(n, M) / 16;
    size_t blocks = (total + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(pack_codes_tiled_kernel, dim3((unsigned)blocks), dim3(256), 0,
                       static_cast<hipStream_t>(stream), codes, n, M, static_cast<uint4 *>(tiled_out));
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

int trim_fs_encode(const float *base, int64_t n, int32_t d, const float *codebooks, int32_t M,
                   uint8_t *codes_out, float *dlx_out, void *stream) {
    if (n < 0 || d <= 0 || M <= 0) return TRIM_INVALID_ARG;
    if (d % M || M % 2) return TRIM_UNSUPPORTED_SHAPE;
    const int dsub = d / M;
    if ((size_t)2 * kC4 * dsub * 4 > 64 * 1024) return TRIM_UNSUPPORTED_SHAPE;
    if (n == 0) return TRIM_OK;
    if (!base || !codebooks || !codes_out || !dlx_out) return TRIM_INVALID_ARG;
    return launch_encode_fs<true>(base, n, d, codebooks, M, codes_out, 0, dlx_out, static_cast<hipStream_t>(stream));
}

int trim_fs_train_pq(const float *train, int64_t ns, int32_t d, int32_t M, int32_t iters,
                     const int32_t *init_rows, float *codebooks_out, uint8_t *assign_ws, void *stream) {
    return trim_fs_train_pq_ws(train, ns, d, M, iters, init_rows, codebooks_out, assign_ws, nullptr, 0, stream);
}

size_t trim_fs_train_pq_workspace_bytes(int64_t ns, int32_t d, int32_t M) {
    if (ns <= 0 || d <= 0 || M <= 0 || d % M) return 0;
    const UpdateLayout L = update_layout(ns, d / M, kC4, M);
    return L.total > 0 ? L.total + 256 : 0;
}

int trim_fs_train_pq_ws(const float *train, int64_t ns, int32_t d, int32_t M, int32_t iters,
                        const int32_t *init_rows, float *codebooks_out, uint8_t *assign_ws, void *workspace, size_t workspace_bytes,
                        void *stream) {
    if (ns <= 0 || d <= 0 || M <= 0 || iters < 0) return TRIM_INVALID_ARG;
    if (d % M || M % 2 || M > 65535) return TRIM_UNSUPPORTED_SHAPE;
    if (!train || !init_rows || !codebooks_out || !assign_ws) return TRIM_INVALID_ARG;
    const int dsub = d / M;
    if ((size_t)2 * kC4 * dsub * 4 > 64 * 1024) return TRIM_UNSUPPORTED_SHAPE;
    const UpdateLayout L = update_layout(ns, dsub, kC4, M);
    unsigned char *ws = update_space(workspace, workspace_bytes, L.total);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int per = kC4 * dsub;  // centroid coordinates per subspace
    hipLaunchKernelGGL(kmeans_init_kernel, dim3((per + 255) / 256, M), dim3(256), 0, st, train, ns, (int64_t)d, dsub,
                       init_rows, kC4, codebooks_out);
    HIP_TRY(hipGetLastError());
    if (const int rc = iters > 0 ? kmeans_columns(train, ns, d, dsub, M, L, ws, st) : TRIM_OK) return rc;
    for (int it = 0; it < iters; ++it) {
        const bool last = it + 1 == iters;      // (see trim_train_pq)
        if (const int rc = launch_encode_fs<false>(train, ns, d, codebooks_out, M, assign_ws, last ? 0 : ns, nullptr, st)) return rc;
        if (const int rc = kmeans_update<1>(train, ns, d, dsub, assign_ws, last ? M : 1, last ? 1 : ns, kC4, M, codebooks_out, ws, st))
            return rc;
    }
    return TRIM_OK;
}

int trim_fs_build_lut(const float *queries, int64_t nq, int32_t d, const float *codebooks, int32_t M,
                      float *lut_out, void *stream) {
    if (nq < 0 || d <= 0 || M <= 0) return TRIM_INVALID_ARG;
    if (d % M || M % 2) return TRIM_UNSUPPORTED_SHAPE;
    if (nq == 0) return TRIM_OK;
    if (!queries || !codebooks || !lut_out) return TRIM_INVALID_ARG;
    if (lut_tiled(d / M, true) && M % 8 == 0 && aligned16(lut_out)) {
        LutArgs a{};
        a.queries = queries; a.nq = a.nslots = nq; a.d = d; a.codebooks = codebooks; a.nsub = M; a.lut = lut_out;
        return launch_lut(a, d / M, true, false, static_cast<hipStream_t>(stream));
    }
    const int bper = 64;   // code bytes per block: 2048 entries
    for (int64_t q0 = 0; q0 < nq; q0 += 65535) {
        const int64_t cnt = nq - q0 < 65535 ? nq - q0 : 65535;
        hipLaunchKernelGGL(lut_fs_kernel, dim3((M / 2 + bper - 1) / bper, (unsigned)cnt), dim3(256),
                           (size_t)d * 4, static_cast<hipStream_t>(stream), queries + (size_t)q0 * d, d,
                           codebooks, M, d / M, bper, lut_out + (size_t)q0 * M * kC4);
        HIP_TRY(hipGetLastError());
    }
    return TRIM_OK;
}

int trim_build_lut(const float *queries, int64_t nq, int32_t d, const float *codebooks, int32_t M,
                   float *lut_out, int32_t mfma, void *stream) {
    if (nq < 0 || d <= 0 || M <= 0) return TRIM_INVALID_ARG;
    if (d % M) return TRIM_UNSUPPORTED_SHAPE;
    const int dsub = d / M;
    if (mfma && dsub != 4 && dsub != 8) return TRIM_UNSUPPORTED_SHAPE;
    if (nq == 0) return TRIM_OK;
    if (!queries || !codebooks || !lut_out) return TRIM_INVALID_ARG;
    if (!aligned16(codebooks) || nq > 0x7fffffff) return TRIM_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (mfma) {
        const dim3 grid((unsigned)((nq + 15) / 16), (unsigned)((M + 3) / 4));
        if (grid.y > 65535) return TRIM_UNSUPPORTED_SHAPE;
        if (dsub == 4)
            hipLaunchKernelGGL(lut_mfma_kernel<4>, grid, dim3(256), 0, st, queries, nq, d, codebooks, M, lut_out);
        else
            hipLaunchKernelGGL(lut_mfma_kernel<8>, grid, dim3(256), 0, st, queries, nq, d, codebooks, M, lut_out);
        HIP_TRY(hipGetLastError());
        return TRIM_OK;
    }
    if (lut_tiled(dsub, false) && aligned16(lut_out)) {
        LutArgs a{};
        a.queries = queries; a.nq = a.nslots = nq; a.d = d; a.codebooks = codebooks; a.nsub = M; a.lut = lut_out;
        return launch_lut(a, dsub, false, false, st);
    }
    const int jper = 8;
    // grid.y is limited to 65535: walk the queries in slabs
    for (int64_t q0 = 0; q0 < nq; q0 += 65535) {
        const int64_t cnt = nq - q0 < 65535 ? nq - q0 : 65535;
        hipLaunchKernelGGL(lut_kernel, dim3((M + jper - 1) / jper, (unsigned)cnt), dim3(256),
                           (size_t)d * 4, st, queries + (size_t)q0 * d, d, codebooks, M, dsub, jper,
                           lut_out + (size_t)q0 * M * kC);
        HIP_TRY(hipGetLastError());
    }
    return TRIM_OK;
}

int trim_search_knn(const trim_index_view *index, const float *queries, int64_t nq,
                    const float *lut, const trim_candidates *cand, int32_t k, float gamma,
                    int32_t batch, const int32_t *query_order,
                    int32_t *out_ids, float *out_d2,
                    const trim_stats *stats, uint32_t *survivor_mask, int64_t mask_words,
                    void *stream) {
    return search_knn(index, queries, nq, lut, cand, k, gamma, batch, query_order, out_ids, out_d2, stats, survivor_mask,
                      mask_words, nullptr, 0, stream);
}

size_t trim_knn_workspace_bytes(const trim_index_view *index, int64_t nq, const trim_candidates *cand, int32_t k, int32_t batch) {
    if (check_index(index) || check_cand(cand) || nq <= 0 || k < 1 || batch < 1) return 0;
    const FewLayout F = few_layout(index, nq, cand, k, batch);
    FinishPlan fp;
    return F.stride > 0 ? F.total : knn_layout(index, nq, cand, k, &fp).total;
}

int trim_search_knn_ws(const trim_index_view *index, const float *queries, int64_t nq,
                       const float *lut, const trim_candidates *cand, int32_t k, float gamma,
                       int32_t batch, const int32_t *query_order,
                       int32_t *out_ids, float *out_d2,
                       const trim_stats *stats, uint32_t *survivor_mask, int64_t mask_words,
                       void *workspace, size_t workspace_bytes, void *stream) {
    return search_knn(index, queries, nq, lut, cand, k, gamma, batch, query_order, out_ids, out_d2, stats, survivor_mask,
                      mask_words, workspace, workspace_bytes, stream);
}

size_t trim_range_workspace_bytes(int64_t nq, int64_t max_candidates) {
    if (nq <= 0 || max_candidates < 0) return 256;
    return range_layout(nq, max_candidates).total;
}

int trim_search_range(const trim_index_view *index, const float *queries, int64_t nq,
                      const float *lut, const trim_candidates *cand, float radius, float gamma,
                      const int32_t *query_order, int64_t *out_offsets, int32_t *out_ids,
                      float *out_d2, int64_t capacity,
                      int64_t *required, const trim_stats *stats, uint32_t *survivor_mask,
                      int64_t mask_words, void *workspace, size_t workspace_bytes, void *stream) {
    return range_search(index, queries, nq, lut, cand, radius, gamma, query_order, out_offsets, out_ids, out_d2,
                        capacity, required, stats, survivor_mask, mask_words, workspace,
                        workspace_bytes, nullptr, 0, stream);
}

int trim_search_range_static(const trim_index_view *index, const float *queries, int64_t nq,
                             const float *lut, const trim_candidates *cand, float radius, float gamma,
                             const int32_t *query_order, int64_t *out_offsets, int32_t *out_ids,
                             float *out_d2, int64_t capacity,
                             int64_t *required, const trim_stats *stats, uint32_t *survivor_mask,
                             int64_t mask_words, void *stream) {
    // refuse what does not fit before anything else: no device call has been made yet
    if (nq > 0 && index) {
        const int64_t max_cand = cand ? cand->max_candidates : index->n;
        if (max_cand >= 0 && nq <= TRIM_MAX_QUERIES && range_layout(nq, max_cand).total > kScratchBytes)
            return TRIM_WORKSPACE;
    }
    void *ws = nullptr;
    const int rc = scratch_for_current_device(&ws);
    if (rc) return rc;
    return range_search(index, queries, nq, lut, cand, radius, gamma, query_order, out_offsets, out_ids, out_d2,
                        capacity, required, stats, survivor_mask, mask_words, ws, kScratchBytes, nullptr, 0, stream);
}

size_t trim_range_scratch_bytes(const trim_index_view *index, int64_t nq, const trim_candidates *cand) {
    if (check_index(index) || check_cand(cand) || nq <= 0) return 0;
    FinishPlan fp;
    return range_scratch_bytes(index, nq, cand, &fp);
}

int trim_search_range_ws(const trim_index_view *index, const float *queries, int64_t nq,
                         const float *lut, const trim_candidates *cand, float radius, float gamma,
                         const int32_t *query_order, int64_t *out_offsets, int32_t *out_ids,
                         float *out_d2, int64_t capacity,
                         int64_t *required, const trim_stats *stats, uint32_t *survivor_mask,
                         int64_t mask_words, void *workspace, size_t workspace_bytes, void *scratch,
                         size_t scratch_bytes, void *stream) {
    return range_search(index, queries, nq, lut, cand, radius, gamma, query_order, out_offsets, out_ids, out_d2,
                        capacity, required, stats, survivor_mask, mask_words, workspace,
                        workspace_bytes, scratch, scratch_bytes, stream);
}

int trim_range_collect(const trim_index_view *index, int64_t nq, const trim_candidates *cand, int32_t *out_ids, float *out_d2,
                       int64_t capacity, void *workspace, size_t workspace_bytes, void *stream) {
    return range_collect(index, nq, cand, out_ids, out_d2, capacity, workspace, workspace_bytes, stream);
}

size_t trim_static_scratch_bytes(void) { return kScratchBytes; }

size_t trim_ivf_nearest_workspace_bytes(int64_t nq, int32_t d, int32_t nlist) {
    const size_t need = nearest_bytes(nq, d, nlist);
    return need > 0 ? need + 256 : 0;
}

size_t trim_ivf_probe_workspace_bytes(int64_t nq, int32_t d, int32_t nlist, int32_t nprobe) {
    if (nq <= 0 || d <= 0 || nlist <= 0 || nprobe <= 0) return 0;
    const ProbeLayout L = probe_layout(nq, d, nlist, nprobe);
    return L.total > 0 ? L.total : probe_in_two(nq, d, nlist, nprobe) ? (size_t)nq * nlist * 4 : 0;
}

int trim_ivf_probe_ws(const float *queries, int64_t nq, int32_t d, const float *centroids, int32_t nlist, int32_t nprobe,
                      int32_t *probes_out, void *workspace, size_t workspace_bytes, void *stream) {
    if (nprobe == 1)
        return ivf_probe(queries, nq, d, centroids, nlist, 1, probes_out, update_space(workspace, workspace_bytes, nearest_bytes(nq, d, nlist)),
                         static_cast<hipStream_t>(stream));
    const ProbeLayout L = nq > 0 && d > 0 && nlist > 0 ? probe_layout(nq, d, nlist, nprobe) : ProbeLayout{};
    if (L.total > 0 && workspace && workspace_bytes >= L.total && queries && centroids && probes_out && aligned16(centroids) &&
        aligned16(queries))
        return launch_probe_ranked(queries, nq, d, centroids, nlist, nprobe, probes_out, L,
                                   reinterpret_cast<unsigned char *>((reinterpret_cast<uintptr_t>(workspace) + 255) & ~uintptr_t(255)),
                                   static_cast<hipStream_t>(stream));
    if (nq <= 0 || d <= 0 || nlist <= 0 || nprobe <= 0 || nprobe > nlist || d % 4 || !queries || !centroids || !probes_out ||
        !aligned16(centroids) || !workspace || (reinterpret_cast<uintptr_t>(workspace) & 3u) ||
        !probe_in_two(nq, d, nlist, nprobe) || workspace_bytes < (size_t)nq * nlist * 4)
        return trim_ivf_probe(queries, nq, d, centroids, nlist, nprobe, probes_out, stream);
    hipStream_t st = static_cast<hipStream_t>(stream);
    uint32_t *dist = static_cast<uint32_t *>(workspace);
    const int qt = nq >= 8 ? 8 : nq >= 4 ? 4 : nq >= 2 ? 2 : 1, rows = kProbeThreads / 32 * (qt == 8 ? 4 : 8);
    void (*fn)(const float *, int64_t, int, const float *, int, uint32_t *) =
        qt == 8 ? probe_distance_kernel<8> : qt == 4 ? probe_distance_kernel<4> : qt == 2 ? probe_distance_kernel<2> : probe_distance_kernel<1>;
    const size_t lds = (size_t)qt * d * 4;
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(fn), lds));
    hipLaunchKernelGGL(fn, dim3((unsigned)((nlist + rows - 1) / rows), (unsigned)((nq + qt - 1) / qt)), dim3(kProbeThreads), lds, st,
                       queries, nq, d, centroids, nlist, dist);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(probe_select_kernel, dim3((unsigned)nq), dim3(kWave), 0, st, dist, nlist, nprobe, probes_out);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

int trim_ivf_probe(const float *queries, int64_t nq, int32_t d, const float *centroids,
                   int32_t nlist, int32_t nprobe, int32_t *probes_out, void *stream) {
    return ivf_probe(queries, nq, d, centroids, nlist, nprobe, probes_out, nullptr, static_cast<hipStream_t>(stream));
}

int trim_query_order(const int32_t *probes, int64_t nq, int32_t nprobe, int32_t nlist,
                     int32_t *order_out, void *stream) {
    if (nq < 0 || nq > 0x7fffffff - 8 || nprobe <= 0 || nlist <= 0) return TRIM_INVALID_ARG;
    if (nq == 0) return TRIM_OK;
    if (!probes || !order_out) return TRIM_INVALID_ARG;
    const int nbucket = nlist < 32768 ? nlist : 32768;
    const size_t lds = (size_t)nbucket * 4;
    hipStream_t st = static_cast<hipStream_t>(stream);
    HIP_TRY(allow_lds(reinterpret_cast<const void *>(query_order_kernel), lds));
    hipLaunchKernelGGL(query_order_kernel, dim3(1), dim3(1024), lds, st, probes, nq, nprobe, nbucket,
                       order_out);
    HIP_TRY(hipGetLastError());
    return TRIM_OK;
}

const char *trim_strerror(int status) {
    switch (status) {
        case TRIM_OK: return "ok";
        case TRIM_INVALID_ARG: return "invalid argument";
        case TRIM_UNSUPPORTED_SHAPE: return "unsupported shape (d, M) for this build";
        case TRIM_WORKSPACE: return "workspace missing, misaligned or too small (trim_search_range_static: the search needs more than TRIM_STATIC_SCRATCH_BYTES)";
        case TRIM_HIP_ERROR: return "HIP call failed (see trim_last_hip_error)";
        case TRIM_INTERNAL: return "the library was built wrongly (a search kernel carries static LDS)";
        default: return "unknown status";
    }
}

int trim_last_hip_error(void) { return trim::g_last_hip_error; }

const char *trim_version(void) { return "0.1"; }

}  // extern "C"
