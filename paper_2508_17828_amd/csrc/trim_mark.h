// The scan in separate passes (Section 4.2), for launches whose exact distances are better computed
// apart from the bounds:
//
//   filter  holds a stretch of every query's candidates against ONE threshold, on the matrix cores, list by
//           list for all the queries that scan the list, and marks who may pass: a bit per candidate
//   finish  the bounds of the marked candidates, by the rule; who does not pass is unmarked
//   measure a lower bound of the distance of everyone still marked, on the matrix cores: a raw row is read once for
//           all the queries that want it, and few exact distances are left to take
//   pick    (kNN) a threshold from the bounds of the first batch, so that it is measured with what comes after it
//   replay  (kNN) walks a query's marked candidates in scan order, batch by batch, with the threshold
//           rule of Section 4.2, and merges the survivors into R
//   range_exact  (range) the exact distances of those that the lower bound leaves
//
// search_kernel does all of it inside one workgroup per query, so every survivor's row is read by
// that query alone.  With long rows this is what bounds the search: on 2,500 queries over 500,000 x 768
// every query refines the 3,940 rows of its own mixture component, 30 GB of the same few rows over
// and over, and the distance table leaves one workgroup per CU, whose lookups wait while its rows
// are fetched.  Thresholds only fall, so the candidates marked against the threshold at the start
// of a stretch contain every survivor of it; the replay decides which they are, exactly as in search_kernel.
#pragma once

#include "trim_passes.h"
#include "trim_steps.h"

namespace trim {

// ---- filter: who can pass, on the matrix cores ----
// With long codes the table lookups of the bounds are what a search costs, and early abandon saves
// little of them where no part of a code decides (unit vectors: half of the subspaces have to be summed
// before far candidates are out).  But Gamma(l,q)^2 = |q|^2 + |l|^2 - 2 q.l is a contraction, and
// queries that probe the same list share its landmarks: list by list, 512 landmarks x 128 queries
// per workgroup and tile, by v_mfma_f32_32x32x16_f16.  A landmark's operand is its centroids, so it is never built:
// a lane gathers 16 bytes of the (16-bit) centroids of its code byte from LDS and that is the operand.
//
// The filter only decides who is looked at again: whoever may pass is marked, and finish_kernel takes
// the marked candidates' table sums by the rule.  Soundness: with q', l' the rounded operands (relative
// to the centroids' means mu, scaled by a power of two), |q - l| >= |q' - l'| - |q - q'| - |l - l'|;
// the two distances moved by rounding are added to the line that bounds sqrt(s) (see abandon_line),
//     r = alpha + beta b + moved(q) + moved(l),    out if s' > r |r|,
// moved(q) measured, moved(l) <= (2^-11 + 2^-22) |l'| and what 16-bit subnormals lose; the binary32
// accumulation of s' errs by at most (4 d + 64) 2^-24 of |q'|^2 + |l'|^2, taken off.
// A query out of the 16-bit range after scaling has alpha = inf: all its candidates are marked.
//
// In a range search the threshold is the same for all queries, and next to all who may pass do (2,000 queries x 250,000 x 1536: all but
// a per cent).  So the larger root of g(a, b) = tau is kept per row, and who lies below
// it by more than what rounding moved passes for certain (CERTAIN): no table sums are taken of those (filter 621 -> 677 us, finish 512 -> 187).  tau is taken
// (nsub + dsub + 64) 2^-23 (a + b)^2 lower for it: the rule's table sums err by (nsub + dsub + 2) 2^-24 of
// s, i.e. 2 (a + b)^2 times half of that in g, its own chain by 2^-21 (a + b)^2.
__global__ __launch_bounds__(256) void filter_means_kernel(const FilterArgs a) {
    const int j = blockIdx.x, c = threadIdx.x, wave = c >> 6;
    __shared__ float part[4];
    float most = 0.0f;
    for (int t = 0; t < a.dsub; ++t) {
        const float v = c < a.ncent ? a.codebooks[((size_t)j * a.ncent + c) * a.dsub + t] : 0.0f;
        float sum = v;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
        if ((c & 63) == 0) part[wave] = sum;
        sync_block();
        const float mu = (part[0] + part[1] + part[2] + part[3]) / (float)a.ncent;
        sync_block();
        if (c == 0) a.mu[j * a.dsub + t] = mu;
        if (c < a.ncent) most = __builtin_fmaxf(most, __builtin_fabsf(v - mu));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) most = __builtin_fmaxf(most, __shfl_xor(most, off));
    if ((c & 63) == 0) atomicMax(a.max_bits, __float_as_uint(most));
}
// The power of two that brings the largest centered centroid value to 2^9 .. 2^10.  From 1e18 on its square leaves the
// binary32 range and the measured distances could not be scaled back; below, a square above the range only makes them 0.
__device__ __forceinline__ float filter_scale(uint32_t max_bits) {
    const float m = __uint_as_float(max_bits);
    if (!(m > 1e-30f && m < 1e18f)) return 0.0f;           // (no scale: everything is marked)
    const int k = 9 - ((int)(max_bits >> 23) - 127);
    return __uint_as_float((uint32_t)(k + 127) << 23);
}
// grid.x: the padded subspaces first (one thread per centroid), then one workgroup per query row
__global__ __launch_bounds__(256) void filter_operands_kernel(const FilterArgs a) {
    const float sc = filter_scale(*a.max_bits);
    const int nb = a.kpad / a.padded;
    if ((int)blockIdx.x < nb) {
        const int j = blockIdx.x, c = threadIdx.x;
        if (c >= a.ncent) return;
        _Float16 *out = a.books + ((size_t)j * a.ncent + c) * a.padded;
        for (int t = 0; t < a.padded; ++t) {
            float v = 0.0f;
            if (j < a.nsub && t < a.dsub) v = (a.codebooks[((size_t)j * a.ncent + c) * a.dsub + t] - a.mu[j * a.dsub + t]) * sc;
            out[t] = (_Float16)v;
        }
        return;
    }
    const int64_t slot = blockIdx.x - nb;
    const int64_t q = a.order ? a.order[a.slot0 + slot] : a.slot0 + slot;
    if (q < 0 || q >= a.nq) return;
    const int64_t row = a.by_query ? q : slot;
    if (a.q16_rows != a.q16)               // the same values without the padding between sub-vectors, for the raw rows
        for (int k = threadIdx.x; k < a.kpad_rows; k += 256) {
            float v = 0.0f;
            if (k < a.d) v = (a.queries[(size_t)q * a.d + k] - a.mu[k]) * sc;
            if (!(__builtin_fabsf(v) <= 16384.0f)) v = 0.0f;
            a.q16_rows[(size_t)row * a.kpad_rows + k] = (_Float16)(-2.0f * (float)(_Float16)v);
        }
    __shared__ float part[3][4];
    float n2 = 0.0f, moved = 0.0f, most = 0.0f;
    for (int k = threadIdx.x; k < a.kpad; k += 256) {
        const int j = k / a.padded, t = k - j * a.padded;
        float v = 0.0f;
        if (j < a.nsub && t < a.dsub) v = (a.queries[(size_t)q * a.d + j * a.dsub + t] - a.mu[j * a.dsub + t]) * sc;
        const float av = __builtin_fabsf(v);
        most = av <= 16384.0f ? __builtin_fmaxf(most, av) : __builtin_inff();
        if (!(av <= 16384.0f)) v = 0.0f;
        const _Float16 h = (_Float16)v;
        const float f = (float)h, e = v - f;
        n2 = __builtin_fmaf(f, f, n2);
        moved = __builtin_fmaf(e, e, moved);
        a.q16[(size_t)row * a.kpad + k] = (_Float16)(-2.0f * f);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        n2 += __shfl_xor(n2, off);
        moved += __shfl_xor(moved, off);
        most = __builtin_fmaxf(most, __shfl_xor(most, off));
    }
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { part[0][wave] = n2; part[1][wave] = moved; part[2][wave] = most; }
    sync_block();
    if (threadIdx.x == 0) {
        n2 = part[0][0] + part[0][1] + part[0][2] + part[0][3];
        moved = part[1][0] + part[1][1] + part[1][2] + part[1][3];
        most = __builtin_fmaxf(__builtin_fmaxf(part[2][0], part[2][1]), __builtin_fmaxf(part[2][2], part[2][3]));
        float m = sqrt_rn(moved) * 1.001f + sqrt_rn(n2) * (1.0f / 4194304.0f) + sqrt_rn((float)a.d) * (1.0f / 16384.0f);
        if (!(most < __builtin_inff()) || sc == 0.0f) m = __builtin_inff();
        a.qpar[2 * row] = n2;
        a.qpar[2 * row + 1] = m;
    }
}

// Candidates per query (what the filter cuts its tiles at), one wave per query.
__global__ __launch_bounds__(256) void totals_kernel(const FinishArgs a) {
    const int lane = threadIdx.x & 63;
    const int64_t slot = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (slot >= a.nslots) return;
    const int64_t q = a.order ? a.order[a.slot0 + slot] : a.slot0 + slot;
    const int64_t row = a.by_query ? q : slot;
    if (q < 0 || q >= a.nq) {
        if (!a.by_query && lane == 0) a.totals[row] = 0;
        return;
    }
    int64_t sum = 0;
    if (a.nseg == 0) sum = lane == 0 ? a.n : 0;
    for (int p = lane; p < a.nseg; p += kWave) {
        const int32_t l = a.probes[(size_t)q * a.nseg + p];
        if (l >= 0 && l < a.nlist) {
            int64_t s = a.list_offsets[l], e = a.list_offsets[l + 1];
            s = s < 0 ? 0 : (s > a.n ? a.n : s);
            e = e < s ? s : (e > a.n ? a.n : e);
            sum += e - s;
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor((long long)sum, off);
    if (lane == 0) a.totals[row] = (int)(sum < a.max_cand ? sum : a.max_cand);
}

// The list whose tiles hold tile `task` (start: prefix of the lists' tiles, start[0] = 0), by one wave, 64 lists at a
// look: 2 dependent loads for 1024 lists instead of 10.
__device__ __forceinline__ int list_of_task(const int32_t *start, int nlist, int task) {
    const int lane = threadIdx.x & 63;
    int lo = 0, len = nlist;
    while (len > 1) {
        const int step = (len + 63) >> 6, at = lo + lane * step;
        const int cnt = __popcll(__ballot(at < nlist && at < lo + len && start[at < nlist ? at : 0] <= task));
        lo += (cnt - 1) * step;
        len = step;
    }
    return lo;
}

// PAD: values per sub-vector after padding; FS: two 4-bit codes per byte; AL: code words (4 bytes) that may be loaded together.
// Persistent: workgroups take tiles until there are no more.  512 landmarks x 128 queries per tile, eight waves of
// 64 x 128.  A slice is 32 values: 16 KB of centroids and 8 KB of queries go through the LDS, four buffers: a slice is staged two
// slices ahead, loaded into registers three ahead, and its first step's operands are read before the barrier that opens it.
// 2,500 queries x 500,000 x 768: 455 -> 415 us; 2,000 x 250,000 x 1536 (range): 682 -> 588; 500 x 300,000 x 960, no lists: 471 ->
// 437.  Taken out of copies one at a time, the gathers' bank conflicts cost 8 % of what is left, staging 5 to 8, the norms 4, barriers
// 10; half the products are 76 us of the last: the products themselves, at the clock they leave, and a tile's ends (18,000
// of 60,000 clocks at 24 slices: finding it, its queries' lines, marking) are most of it.  Six buffers and a barrier
// every two slices: 416, 571, 442.  Those are sub-vectors of 8 values; 2,000 x 200,000 x 768 with sub-vectors of 4: 190 -> 182, of 16:
// 179 -> 156, 4-bit codes: 188 -> 174 (range searches, with the certain bits and without: 220 / 186, 192 / 174, 194 / 185, for a finish
// pass of 149 / 477, 26 / 105, 63 / 322).  What instances spill (2 to 18 registers, most with sub-vectors of 4) they spill outside of the loop
// over slices, whose assembly has no scratch instruction.
template <int PAD, bool FS, int AL, bool CERTAIN>
__global__ __launch_bounds__(kFltThreads, 1) void filter_kernel(const FilterArgs a) {
    typedef _Float16 h8 __attribute__((ext_vector_type(8)));
    typedef _Float16 h4 __attribute__((ext_vector_type(4)));
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    typedef float v16f __attribute__((ext_vector_type(16)));
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    constexpr int kCent = FS ? kC4 : kC;
    constexpr int kSubs = kFltSlice / PAD;                        // subspaces per slice
    constexpr int kBytes = FS ? kSubs / 2 : kSubs;                // code bytes per slice
    constexpr int kBookBytes = kFltSlice * kCent * 2;             // 16 KB (FS: 1 KB)
    constexpr int kBookV = kBookBytes / 16, kBooks = kBookV > kFltThreads ? kBookV / kFltThreads : 1;
    constexpr int CH = kBytes >= 2 ? kBytes / 2 : 1;              // code words of two slices
    constexpr int kAl = AL < CH ? AL : CH;
    constexpr int kQStride = kFltQ + 4;                           // (bank spread)
    __shared__ __align__(16) unsigned char s_book[4 * kBookBytes];
    __shared__ __align__(16) h8 s_q[4 * 4 * kQStride];            // [8 values][query]
    __shared__ __align__(16) float s_b[kFltRows], s_nl[kFltRows], s_ml[kFltRows], s_hi[CERTAIN ? kFltRows : 4];
    __shared__ float s_al[kFltQ], s_be[kFltQ], s_nq[kFltQ], s_mq[CERTAIN ? kFltQ : 1];
    __shared__ uint32_t s_room;
    __shared__ int s_row[kFltQ], s_c0[kFltQ], s_end[kFltQ];
    __shared__ float s_b0[kFltThreads / kWave];
    const float sc = filter_scale(*a.max_bits);
    const int nslice = a.kpad / kFltSlice;
    const int64_t rows_all = a.n < a.hi ? a.n : a.hi, qall = a.by_query ? a.nq : a.nslots;
    const int total_tasks = a.list_offsets ? a.tasks[a.nlist]
                            : (int)((rows_all + kFltRows - 1) / kFltRows * ((qall + kFltQ - 1) / kFltQ));
    for (int task = blockIdx.x; task < total_tasks; task += gridDim.x) {
        // (opaque: addresses that depend on the thread are made per tile; kept over the tiles they would not fit the
        // registers, and a reload inside the slices waits for everything that is on its way)
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63, wave = tid >> 6, col = lane & 31, half = lane >> 5;
        // which list, rows, queries
        int64_t ls = 0, le = a.n;
        int i0 = 0, i1 = (int)qall, t = task;
        if (a.list_offsets) {
            const int x = list_of_task(a.tasks, a.nlist, task);
            ls = a.list_offsets[x];
            le = a.list_offsets[x + 1];
            ls = ls < 0 ? 0 : (ls > a.n ? a.n : ls);
            le = le < ls ? ls : (le > a.n ? a.n : le);
            i0 = a.inv_start[x];
            i1 = a.inv_start[x + 1];
            t -= a.tasks[x];
        }
        const int nqt = (i1 - i0 + kFltQ - 1) / kFltQ;
        const int rt = t / nqt, qt = t - rt * nqt;
        const int64_t r0 = ls + (int64_t)rt * kFltRows;
        const int nrows = le - r0 < kFltRows ? (int)(le - r0) : kFltRows;
        const int q0 = i0 + qt * kFltQ, nqs = i1 - q0 < kFltQ ? i1 - q0 : kFltQ;
        sync_block();     // the previous tile is done with
        if constexpr (CERTAIN) {
            if (tid == 0) s_room = 0x7f800000u;
            sync_block();
        }
        // the queries' rows of the workspace; landmark distances of the rows, their mean (the tangent point)
        int row = 0, c0q = 0, endq = 0;
        if (tid < kFltQ) {
            row = q0 + (tid < nqs ? tid : 0);
            int64_t c = 0;
            if (a.list_offsets) { const int2 v = a.inv[row]; row = v.x; c = v.y; }
            c += r0 - ls;
            s_row[tid] = row;
            endq = a.totals[row];
            endq = endq < a.hi ? endq : a.hi;
            c0q = c < endq ? (int)c : endq;
            if (tid >= nqs || c >= endq || c + nrows <= a.lo) endq = c0q;      // nothing of this query in these rows
        }
        {
            float b = 0.0f;
            if (tid < nrows) b = a.dlx[r0 + tid];
            const float bs = b * sc;
            s_b[tid] = bs < 1e30f ? bs : __builtin_nanf("");       // (marked: the line would fall to -inf there)
            if constexpr (CERTAIN) {
                // the larger root; the smaller one has to lie well below zero (it does while the radius exceeds the landmark
                // distances by anything), s_room: by how much
                const float c1 = 1.0f - 0.5f * a.two_gamma, tau = a.radius2, under = b * b * (1.0f - c1 * c1);
                float hi = -__builtin_inff(), room = __builtin_inff();
                if (tau > kCertainLow && tau < kCertainHigh) {
                    const float end = __builtin_fabsf(c1 * b) + sqrt_rn(__builtin_fmaxf(tau - under, 0.0f)) + __builtin_fabsf(b);
                    const float root2 = tau - end * end * ((float)(a.nsub + a.dsub + 64) * (1.0f / 8388608.0f)) - under;
                    if (root2 > 0.0f) {
                        const float root = sqrt_rn(root2);
                        hi = (c1 * b + root) * sc * 0.999999f;
                        room = __builtin_fmaxf((root - c1 * b) * sc * 0.999999f, 0.0f);
                    }
                }
                s_hi[tid] = hi;
                uint32_t least = tid < nrows && hi > -__builtin_inff() ? __float_as_uint(room) : 0x7f800000u;
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) least = min(least, (uint32_t)__shfl_xor((int)least, off));
                if (lane == 0) atomicMin(&s_room, least);
            }
            float sum = b;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
            if (lane == 0) s_b0[wave] = sum;
        }
        if (!__syncthreads_or(c0q < endq)) continue;
        // staging: a slice of the centroids (contiguous) and of the queries (four threads each)
        const u4 *book_src = reinterpret_cast<const u4 *>(a.books);
        const int sq = tid >> 2, sp = tid & 3;
        const u4 *q_src = reinterpret_cast<const u4 *>(a.q16 + (size_t)s_row[sq] * a.kpad) + sp;
        struct Ahead { u4 bk[kBooks], qv; };
        auto load = [&](int sl, Ahead &r) {
            sl = sl < nslice ? sl : nslice - 1;             // (past the end: loaded and staged, never used)
#pragma unroll
            for (int i = 0; i < kBooks; ++i)
                if (kBookV >= kFltThreads || tid < kBookV) r.bk[i] = book_src[(size_t)sl * kBookV + i * kFltThreads + tid];
            r.qv = q_src[(size_t)sl * (kFltSlice / 8)];
        };
        auto stage = [&](int sl, const Ahead &r) {
            u4 *bd = reinterpret_cast<u4 *>(s_book + (sl & 3) * kBookBytes);
#pragma unroll
            for (int i = 0; i < kBooks; ++i)
                if (kBookV >= kFltThreads || tid < kBookV) bd[i * kFltThreads + tid] = r.bk[i];
            reinterpret_cast<u4 *>(s_q + (sl & 3) * (4 * kQStride))[sp * kQStride + sq] = r.qv;
        };
        // the code words of this lane's two rows, those of two slices at a time
        const uint8_t *codes = a.codes + (size_t)r0 * a.M;
        uint32_t code[2];
        uint32_t cw[2][CH];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int r = wave * 64 + u * 32 + col;
            code[u] = (uint32_t)((r < nrows ? r : 0) * a.M);
        }
        auto load_code = [&](int sl, uint32_t (&w)[2][CH]) {       // (past the code: padding subspaces, all centroids zero, any code)
            const int at = sl * kBytes & ~3;
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int v = 0; v < CH; v += kAl) {
                    uint32_t x[kAl];
                    load_codes<kAl>(x, codes + (code[u] + (uint32_t)(at + 4 * v < a.M ? at + 4 * v : 0)));
#pragma unroll
                    for (int e = 0; e < kAl; ++e) w[u][v + e] = x[e];
                }
        };
        Ahead ahead, first[2];
        load(0, first[0]);
        load_code(0, cw);
        load(1, first[1]);
        load(2, ahead);
        // (while these are under way) the lines that bound the queries' table sums
        if (tid < kFltQ) {
            float al = -1.0f, be = 0.0f, nq = 0.0f, mq = 0.0f;
            if (c0q < endq) {
                const int64_t q = a.by_query ? row : a.order ? a.order[a.slot0 + row] : a.slot0 + row;
                const float tau = a.range ? a.radius2 : a.tau_of ? a.tau_of[(size_t)q * a.tau_stride] : __builtin_inff();
                float b0 = 0.0f;
#pragma unroll
                for (int w = 0; w < kFltThreads / kWave; ++w) b0 += s_b0[w];
                const AbandonLine line = abandon_line(tau, a.two_gamma, b0 / (float)nrows);
                nq = a.qpar[2 * (size_t)row];
                mq = a.qpar[2 * (size_t)row + 1];
                al = line.alpha * sc + mq;
                be = line.beta;
                if (!(al == al)) al = __builtin_inff();
            }
            s_al[tid] = al; s_be[tid] = be; s_nq[tid] = nq;
            if constexpr (CERTAIN) s_mq[tid] = mq;
            s_c0[tid] = c0q; s_end[tid] = endq;
        }
        v16f acc[2][4];
        float nl[2] = {0.0f, 0.0f};
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[u][v][i] = 0.0f;
        const bool busy = __builtin_amdgcn_readfirstlane(wave) * 64 < nrows;
        const int nv = (nqs + 31) >> 5;               // query tiles of this one in use
        stage(0, first[0]);
        stage(1, first[1]);
        sync_block();
        // (the number of query tiles is fixed inside: a branch around each leaves its operands' latency open four times a step)
        auto slices = [&](auto tiles) {
            constexpr int NV = decltype(tiles)::value;
            struct Operands { h8 lm[2], qf[NV]; };
            auto operands = [&](int sl, auto odd, auto step, const uint32_t (&w)[2][CH], Operands &o) {
                constexpr int j = decltype(odd)::value, ks = decltype(step)::value;
                const unsigned char *bb = s_book + (sl & 3) * kBookBytes;
                const h8 *qq = s_q + (sl & 3) * (4 * kQStride) + (ks * 2 + half) * kQStride + col;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if constexpr (FS) {                       // four sub-vectors of two values
                        const uint32_t word = w[u][2 * j + ks] >> (16 * half);
                        h2 p[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            p[e] = *reinterpret_cast<const h2 *>(bb + (((ks * 8 + half * 4 + e) * kCent + ((word >> (4 * e)) & 15u)) << 2));
                        o.lm[u] = h8{p[0][0], p[0][1], p[1][0], p[1][1], p[2][0], p[2][1], p[3][0], p[3][1]};
                    } else if constexpr (PAD == 4) {          // two
                        const uint32_t word = w[u][2 * j + ks] >> (16 * half);
                        const h4 p0 = *reinterpret_cast<const h4 *>(bb + (((ks * 4 + half * 2) * kCent + (word & 255u)) << 3));
                        const h4 p1 = *reinterpret_cast<const h4 *>(bb + (((ks * 4 + half * 2 + 1) * kCent + ((word >> 8) & 255u)) << 3));
                        o.lm[u] = h8{p0[0], p0[1], p0[2], p0[3], p1[0], p1[1], p1[2], p1[3]};
                    } else {                                  // one, or a part of one
                        constexpr int kParts = PAD >= 8 ? PAD / 8 : 1;       // operands per sub-vector
                        const int op = ks * 2 + half, sub = op / kParts, part = op % kParts;
                        const int at = PAD == 8 ? 0 : PAD == 16 ? 16 * j : 8 * (sl & 3);
                        const uint32_t c = (w[u][PAD == 8 ? j : 0] >> (8 * sub + at)) & 255u;
                        o.lm[u] = *reinterpret_cast<const h8 *>(bb + (sub * kCent + c) * (PAD * 2) + part * 16);
                    }
                }
#pragma unroll
                for (int v = 0; v < NV; ++v) o.qf[v] = qq[v * 32];
            };
            auto multiply = [&](const Operands &o) {
#pragma unroll
                for (int v = 0; v < NV; ++v)
#pragma unroll
                    for (int u = 0; u < 2; ++u) acc[u][v] = __builtin_amdgcn_mfma_f32_32x32x16_f16(o.lm[u], o.qf[v], acc[u][v], 0, 0, 0);
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const h2 p = {o.lm[u][2 * e], o.lm[u][2 * e + 1]};
                        nl[u] = __builtin_amdgcn_fdot2(p, p, nl[u], false);
                    }
            };
            // per slice: its second step's operands under way, the first step's products, slice sl + 2 to the LDS, the next slice's
            // first operands under way, the second step's products
            auto slice = [&](int sl, auto odd, const uint32_t (&w)[2][CH], const uint32_t (&next)[2][CH], Operands &o) {
                constexpr int j = decltype(odd)::value;
                Operands p;
                __builtin_amdgcn_sched_barrier(0);
                operands(sl, odd, std::integral_constant<int, 1>{}, w, p);
                multiply(o);
                stage(sl + 2, ahead);
                load(sl + 3, ahead);
                if constexpr (NV >= 3 && !FS && PAD >= 8) {
#pragma unroll
                    for (int i = 0; i < 2 + NV; ++i) {
                        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    }
                    __builtin_amdgcn_sched_group_barrier(0x8, NV - 2, 0);
                    __builtin_amdgcn_sched_group_barrier(0x200, kBooks + 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x20, kBooks + 1, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                operands(sl + 1, std::integral_constant<int, 1 - j>{}, std::integral_constant<int, 0>{}, next, o);
                multiply(p);
                if constexpr (NV >= 3 && !FS && PAD >= 8) {
#pragma unroll
                    for (int i = 0; i < 2 + NV; ++i) {
                        __builtin_amdgcn_sched_group_barrier(0x8, 1, 1);
                        __builtin_amdgcn_sched_group_barrier(0x100, 1, 1);
                    }
                    __builtin_amdgcn_sched_group_barrier(0x8, NV - 2, 1);
                }
                __builtin_amdgcn_sched_barrier(0);
                sync_block();
            };
            Operands o;
            operands(0, std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{}, cw, o);
#pragma unroll 1
            for (int sl = 0; sl < nslice; sl += 2) {      // (an even number)
                uint32_t cn[2][CH];
                load_code(sl + 2, cn);
                slice(sl, std::integral_constant<int, 0>{}, cw, cw, o);
                slice(sl + 1, std::integral_constant<int, 1>{}, cw, cn, o);
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int v = 0; v < CH; ++v) cw[u][v] = cn[u][v];
            }
        };
        if (!busy) {
#pragma unroll 1
            for (int sl = 0; sl < nslice; ++sl) {
                stage(sl + 2, ahead);
                load(sl + 3, ahead);
                sync_block();
            }
        } else switch (nv) {
            case 1: slices(std::integral_constant<int, 1>{}); break;
            case 2: slices(std::integral_constant<int, 2>{}); break;
            case 3: slices(std::integral_constant<int, 3>{}); break;
            default: slices(std::integral_constant<int, 4>{}); break;
        }
        constexpr float kUlp = 1.0f / 16777216.0f;
        const float keep = 1.0f - (4.0f * a.d + 64.0f) * kUlp;
        const float over = 2.5f * (4.0f * a.d + 64.0f) * kUlp;       // (of the norms, kept low: what a score may be too low by)
        if (busy) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {                         // (this wave's rows only: no barrier needed)
                const float n2 = nl[u] + __shfl_xor(nl[u], 32);
                const int r = wave * 64 + u * 32 + col;
                if (half == 0) {
                    s_nl[r] = n2 * keep;
                    s_ml[r] = sqrt_rn(n2) * (1.0f / 2048.0f + 1.0f / 4194304.0f) * 1.001f + sqrt_rn((float)a.d) * (1.0f / 16384.0f);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                float rb[16], rn[16], rm[16], rh[16] = {}, widest = 0.0f;      // (rh: the larger root less what moved the landmark)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int r = wave * 64 + u * 32 + 8 * i + 4 * half;
                    const float4 x = *reinterpret_cast<const float4 *>(s_b + r), y = *reinterpret_cast<const float4 *>(s_nl + r),
                                 z = *reinterpret_cast<const float4 *>(s_ml + r);
                    rb[4 * i] = x.x; rb[4 * i + 1] = x.y; rb[4 * i + 2] = x.z; rb[4 * i + 3] = x.w;
                    rn[4 * i] = y.x; rn[4 * i + 1] = y.y; rn[4 * i + 2] = y.z; rn[4 * i + 3] = y.w;
                    rm[4 * i] = z.x; rm[4 * i + 1] = z.y; rm[4 * i + 2] = z.z; rm[4 * i + 3] = z.w;
                    if constexpr (CERTAIN) {
                        const float4 h = *reinterpret_cast<const float4 *>(s_hi + r);
                        rh[4 * i] = h.x - z.x * 1.00001f; rh[4 * i + 1] = h.y - z.y * 1.00001f;
                        rh[4 * i + 2] = h.z - z.z * 1.00001f; rh[4 * i + 3] = h.w - z.w * 1.00001f;
                        widest = __builtin_fmaxf(__builtin_fmaxf(widest, __builtin_fmaxf(z.x, z.y)), __builtin_fmaxf(z.z, z.w));
                    }
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    if (v >= nv) break;
                    __builtin_amdgcn_sched_barrier(0);
                    const int qi = v * 32 + col;
                    const float al = s_al[qi], be = s_be[qi], nq = s_nq[qi] * keep;
                    uint32_t m = 0, in = 0;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const float r = __builtin_fmaf(be, rb[i], al) + rm[i];
                        const float s = acc[u][v][i] + (nq + rn[i]);
                        if (!(s > r * __builtin_fabsf(r))) m |= 1u << (8 * (i >> 2) + (i & 3));
                    }
                    if constexpr (CERTAIN) {
                        const float mq = s_mq[qi] * 1.00001f;
#pragma unroll
                        for (int i = 15; i >= 0; --i) {
                            // (below zero: within.  A NaN counts as 1.)
                            const float h = rh[i] - mq, base = nq + rn[i];
                            const float past = __builtin_fmaf(-h, __builtin_fabsf(h), __builtin_fmaf(base, over, acc[u][v][i] + base));
                            in = __builtin_amdgcn_alignbit(in, __float_as_uint(__builtin_fminf(past, 1.0f)), 31);
                        }
                        in = (in & 0xfu) | (in & 0xf0u) << 4 | (in & 0xf00u) << 8 | (in & 0xf000u) << 12;
                        if (!((widest + mq) * 1.01f < __uint_as_float(s_room))) in = 0;
                    }
                    // rows of the tile that exist, candidates of this pass
                    const int c0 = s_c0[qi] + wave * 64 + u * 32, end = s_end[qi];
                    auto put = [&](uint32_t bits, uint32_t *to) {
                        bits <<= 4 * half;
                        bits |= (uint32_t)__shfl_xor((int)bits, 32);
                        if (c0 + 32 > end) bits &= c0 < end ? (1u << (end - c0)) - 1u : 0u;
                        if (c0 < a.lo) bits &= a.lo - c0 < 32 ? ~0u << (a.lo - c0) : 0u;
                        const int left = nrows - (wave * 64 + u * 32);
                        if (left < 32) bits &= left > 0 ? (1u << left) - 1u : 0u;
                        const int shf = c0 & 31;
                        const uint32_t part = half == 0 ? bits << shf : (shf ? bits >> (32 - shf) : 0u);
                        if (part) atomicOr(&to[(size_t)s_row[qi] * a.words + (c0 >> 5) + half], part);
                    };
                    put(m, a.possible);
                    if constexpr (CERTAIN) put(in, a.certain);
                }
            }
        }
    }
}

// ---- measure: lower bounds of the exact distances of the marked candidates ----
// The filter's contraction over the raw rows (16-bit, relative to mu, scaled; converted while they are staged), list by
// list, 256 rows at a time against the queries that have a candidate marked among them (up to 64 WQ together):
//     d2 >= ((|q' - x'| - moved(q) - moved(x)) / scale)^2   less the exact rule's own roundings.
// Only where that does not exceed the threshold is the exact distance taken (replay_kernel,
// range_exact_kernel).  A row is read once for all its queries, and the contraction takes the place of 2 d
// vector operations per survivor: of 3,940 survivors per query (2,500 queries x 500,000 x 768) some forty
// can still matter.  WR waves of 64 rows by WQ waves of 64 queries; NS slices of 32 values are on their way in registers while one is
// used; WAVES: per SIMD.  Lists are cut at kMsrRows rows: WR = 4 there.
//   <2, 4, 1, 4>  two workgroups per CU, bound by reading the rows (4.2 TB/s): 2,500 queries x 500,000 x 768, 440 -> 405 us
//   <4, 4, 2, 4>  256 queries at a time, rows are read half as often: 500 queries x 300,000 x 960 906 -> 547 us
//   <8, 2, 1, 4>  512 queries, half as many rows: the same bytes through the LDS, rows read once: there 555 -> 404 us (NS = 2 spills: 426;
//                 waves of 64 x 128 at two per SIMD: 474).  Bound by the chain of barriers over slices, one workgroup per CU
//   <2, 2, 4, 2>  too few tiles for the chip: bound by a tile's own chain; half as long a tile, rows asked for further ahead: 52 -> 35 us
// Queries go to workgroups in blocks of 512, so that a list that many want is not one workgroup's tail.
template <int WQ, int WR, int NS, int WAVES>
__global__ __launch_bounds__(64 * WQ * WR, WAVES) void measure_kernel(const FilterArgs a) {
    typedef _Float16 h8 __attribute__((ext_vector_type(8)));
    typedef _Float16 h4 __attribute__((ext_vector_type(4)));
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    typedef float v16f __attribute__((ext_vector_type(16)));
    typedef float f4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    constexpr int kMsrThreads = 64 * WQ * WR, kMsrQ = 64 * WQ, kRows = 64 * WR;
    constexpr int kApart = kMsrThreads / 8, kPer = kRows / kApart;        // rows staged by a thread
    constexpr int kQApart = kMsrThreads / 4, kQPer = kMsrQ / kQApart;     // queries staged by a thread
    constexpr int kStep = NS > 2 ? NS : 2;                        // slices a turn of the loop
    constexpr int kXRows = kRows + 2;                          // rows per 8 columns (two spare: bank spread)
    constexpr int kQStride = kMsrQ + 4;                           // (bank spread)
    __shared__ __align__(16) unsigned char s_x[2][4 * kXRows * 16];
    __shared__ __align__(16) h8 s_q[2][4 * kQStride];             // [8 columns][query]
    __shared__ __align__(16) float s_nx[kRows], s_mx[kRows];
    __shared__ float s_mq[2 * kMsrQ], s_nq[2 * kMsrQ];
    __shared__ int s_row[2 * kMsrQ], s_c0[2 * kMsrQ], s_end[2 * kMsrQ];
    __shared__ int s_n;
    extern __shared__ __align__(16) float s_mu[];                 // [d]
    const float sc = filter_scale(*a.max_bits);
    const int nslice = a.kpad_rows / kFltSlice;
    const int64_t rows_all = a.n < a.hi ? a.n : a.hi, qall = a.by_query ? a.nq : a.nslots;
    constexpr float kUlp = 1.0f / 16777216.0f;
    const float keep = 1.0f - (4.0f * a.d + 64.0f) * kUlp;
    const float back = sc > 0.0f ? (1.0f - (a.d / 32 + 16.0f) * 2.0f * kUlp) / (sc * sc) : 0.0f;
    const float lost = sqrt_rn((float)a.d) * (1.0f / 16384.0f);
    for (int t = threadIdx.x; t < a.d; t += kMsrThreads) s_mu[t] = a.mu[t];      // (barriers follow)
    const int total_tasks = a.list_offsets ? a.row_tasks[a.nlist]
                            : (int)((rows_all + kRows - 1) / kRows * ((qall + a.msr_block - 1) / a.msr_block));
    for (int task = blockIdx.x; task < total_tasks; task += gridDim.x) {
        int tid = threadIdx.x;            // (opaque: see filter_kernel)
        asm volatile("" : "+v"(tid));
        int64_t ls = 0, r0, le = a.n;
        int qb, q1;
        if (a.list_offsets) {
            const int x = list_of_task(a.row_tasks, a.nlist, task);
            ls = a.list_offsets[x];
            le = a.list_offsets[x + 1];
            ls = ls < 0 ? 0 : (ls > a.n ? a.n : ls);
            le = le < ls ? ls : (le > a.n ? a.n : le);
            qb = a.inv_start[x];
            q1 = a.inv_start[x + 1];
            const int nqb = (q1 - qb + a.msr_block - 1) / a.msr_block, t = task - a.row_tasks[x], rt = t / nqb;
            qb += (t - rt * nqb) * a.msr_block;
            q1 = qb + a.msr_block < q1 ? qb + a.msr_block : q1;
            r0 = ls + (int64_t)rt * kRows;
        } else {
            const int nqb = (int)((qall + a.msr_block - 1) / a.msr_block);
            const int rt = task / nqb;
            qb = (task - rt * nqb) * a.msr_block;
            q1 = qb + a.msr_block < (int)qall ? qb + a.msr_block : (int)qall;
            r0 = (int64_t)rt * kRows;
        }
        const int nrows = le - r0 < kRows ? (int)(le - r0) : kRows;
        int have = 0;                     // queries waiting in the arrays (the same for all threads)
        sync_block();                  // (the previous tile is done with)
        while (qb < q1 || have > 0) {
            // gather queries with a mark in these rows until there are 64 WQ, or no more
            while (qb < q1 && have < kMsrQ) {
                if (tid == 0) s_n = have;
                sync_block();
                if (tid < kMsrQ && qb + tid < q1) {
                    int row = qb + tid;
                    int64_t c = 0;
                    if (a.list_offsets) { const int2 v = a.inv[qb + tid]; row = v.x; c = v.y; }
                    c += r0 - ls;
                    int end = a.totals[row];
                    end = end < a.hi ? end : a.hi;
                    if (c < end && c + nrows > a.lo) {
                        const uint32_t *bits = a.possible + (size_t)row * a.words;
                        const int64_t c1 = c + nrows < end ? c + nrows : end, c2 = c > a.lo ? c : a.lo;
                        const int w0 = (int)(c2 >> 5), w1 = (int)((c1 - 1) >> 5);
                        uint32_t any = 0;
                        for (int w = w0; w <= w1; ++w) {
                            uint32_t b = bits[w];
                            if (w == w0) b &= ~0u << (c2 & 31);
                            if (w == w1 && (c1 & 31)) b &= (1u << (c1 & 31)) - 1u;
                            any |= b;
                        }
                        if (any) {
                            const int at = atomicAdd(&s_n, 1);
                            s_row[at] = row; s_c0[at] = (int)c; s_end[at] = end;
                            s_nq[at] = a.qpar[2 * (size_t)row];
                            s_mq[at] = a.qpar[2 * (size_t)row + 1];
                        }
                    }
                }
                qb += kMsrQ;
                sync_block();
                have = s_n;
                sync_block();
            }
            if (have == 0) break;
            asm volatile("" : "+v"(tid));
            const int lane = tid & 63, wave = (tid >> 6) % WR, wq = (tid >> 6) / WR, col = lane & 31, half = lane >> 5;
            const int nqs = have < kMsrQ ? have : kMsrQ, nq32 = (nqs + 31) >> 5;
            const int nv = nq32 - 2 * wq < 2 ? nq32 - 2 * wq : 2;        // query tiles of this wave
            // staging: eight threads per row (a whole cache line together), kPer rows each, kApart apart; four per query, kQPer each
            const int xr = tid >> 3, xc = tid & 7, sq = tid >> 2, sp = tid & 3;
            float nx[kPer] = {};
            const u4 *q_src = reinterpret_cast<const u4 *>(a.q16_rows);
            uint32_t q_at[kQPer];              // (16 bytes)
#pragma unroll
            for (int i = 0; i < kQPer; ++i) {
                const int w = sq + kQApart * i;
                q_at[i] = (uint32_t)s_row[w < nqs ? w : 0] * (uint32_t)(a.kpad_rows / 8) + sp;
            }
            const unsigned char *x_src = reinterpret_cast<const unsigned char *>(a.base + (size_t)r0 * a.d);
            struct Ahead { f4 x[kPer]; u4 q[kQPer]; };
            auto load = [&](int sl, Ahead &r) {
                sl = sl < nslice ? sl : nslice - 1;
                const int k = sl * kFltSlice + 4 * xc;
                const bool in = k < a.d;
#pragma unroll
                for (int i = 0; i < kPer; ++i) {
                    const int w = xr + kApart * i;
                    r.x[i] = *reinterpret_cast<const f4 *>(x_src + (uint32_t)((w < nrows ? w : 0) * a.d + (in ? k : 0)) * 4u);
                }
#pragma unroll
                for (int i = 0; i < kQPer; ++i) r.q[i] = q_src[q_at[i] + (uint32_t)sl * (kFltSlice / 8)];
            };
            auto stage = [&](int sl, const Ahead &r) {
                const bool in = sl * kFltSlice + 4 * xc < a.d;     // (nothing past the end)
                f4 mu = {0.0f, 0.0f, 0.0f, 0.0f};
                if (in) mu = *reinterpret_cast<const f4 *>(s_mu + sl * kFltSlice + 4 * xc);
#pragma unroll
                for (int i = 0; i < kPer; ++i) {
                    h4 h = {0, 0, 0, 0};
                    if (in) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) h[e] = (_Float16)__builtin_fmaf(r.x[i][e], sc, -(mu[e] * sc));
                        nx[i] = __builtin_amdgcn_fdot2(h2{h[0], h[1]}, h2{h[0], h[1]}, nx[i], false);
                        nx[i] = __builtin_amdgcn_fdot2(h2{h[2], h[3]}, h2{h[2], h[3]}, nx[i], false);
                    }
                    *reinterpret_cast<h4 *>(s_x[sl & 1] + ((xc >> 1) * kXRows + xr + kApart * i) * 16 + (xc & 1) * 8) = h;
                }
#pragma unroll
                for (int i = 0; i < kQPer; ++i) reinterpret_cast<u4 *>(s_q[sl & 1])[sp * kQStride + sq + kQApart * i] = r.q[i];
            };
            v16f acc[2][2];
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int v = 0; v < 2; ++v)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[u][v][i] = 0.0f;
            const bool busy = wave * 64 < nrows && nv > 0;
            Ahead ahead[NS];
#pragma unroll
            for (int i = 0; i < NS; ++i) load(i, ahead[i]);
            stage(0, ahead[0]);
            load(NS, ahead[0]);
            sync_block();
            auto slice = [&](int sl, Ahead &r) {     // r: slice sl + 1
                stage(sl + 1, r);
                load(sl + 1 + NS, r);
                if (busy) {
                    const unsigned char *bb = s_x[sl & 1];
                    const h8 *qq = s_q[sl & 1];
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks) {
                        __builtin_amdgcn_sched_barrier(0);     // (registers: one step's operands at a time)
                        h8 xf[2];
#pragma unroll
                        for (int u = 0; u < 2; ++u)
                            xf[u] = *reinterpret_cast<const h8 *>(bb + ((ks * 2 + half) * kXRows + wave * 64 + u * 32 + col) * 16);
#pragma unroll
                        for (int v = 0; v < 2; ++v)
                            if (v < nv) {
                                const h8 qf = qq[(ks * 2 + half) * kQStride + wq * 64 + v * 32 + col];
#pragma unroll
                                for (int u = 0; u < 2; ++u) acc[u][v] = __builtin_amdgcn_mfma_f32_32x32x16_f16(xf[u], qf, acc[u][v], 0, 0, 0);
                            }
                    }
                }
                sync_block();
            };
#pragma unroll 1
            for (int sl = 0; sl < nslice; sl += kStep) {
#pragma unroll
                for (int u = 0; u < kStep; ++u) {
                    if (u >= 2 && sl + u >= nslice) break;         // (an even number of slices)
                    slice(sl + u, ahead[(u + 1) % NS]);
                }
            }
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                float v = nx[i];
                v += __shfl_xor(v, 1);
                v += __shfl_xor(v, 2);
                v += __shfl_xor(v, 4);
                if (xc == 0) {
                    s_nx[xr + kApart * i] = v * keep;
                    s_mx[xr + kApart * i] = sqrt_rn(v) * (1.0f / 2048.0f + 1.0f / 4194304.0f) * 1.001f + lost;
                }
            }
            sync_block();
            if (busy) {
#pragma unroll
                for (int v = 0; v < 2; ++v) {
                    if (v >= nv) break;
                    __builtin_amdgcn_sched_barrier(0);
                    const int qi = wq * 64 + v * 32 + col;
                    const bool real = qi < nqs;
                    const float mq = real ? s_mq[qi] : 0.0f, nq = real ? s_nq[qi] * keep : 0.0f;
                    const int cq = real ? s_c0[qi] : 0, end = real ? s_end[qi] : 0;
                    const size_t at = (size_t)(real ? s_row[qi] : 0) * a.words;
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const int c0 = cq + wave * 64 + u * 32;
                        uint32_t m = 0;
                        if (c0 < end) {
                            m = a.possible[at + (c0 >> 5)] >> (c0 & 31);
                            if (c0 & 31) m |= a.possible[at + (c0 >> 5) + 1] << (32 - (c0 & 31));
                            if (c0 + 32 > end) m &= (1u << (end - c0)) - 1u;
                            if (c0 < a.lo) m &= a.lo - c0 < 32 ? ~0u << (a.lo - c0) : 0u;
                            const int left = nrows - (wave * 64 + u * 32);
                            if (left < 32) m &= left > 0 ? (1u << left) - 1u : 0u;
                        }
                        if (!__any(m != 0)) continue;
                        float *out = a.d2 + at * 32 + c0;
#pragma unroll
                        for (int i = 0; i < 16; ++i) {
                            const int r = 8 * (i >> 2) + 4 * half + (i & 3);
                            if ((m >> r) & 1u) {
                                const float s = acc[u][v][i] + (nq + s_nx[wave * 64 + u * 32 + r]);
                                float dist = __builtin_amdgcn_sqrtf(__builtin_fmaxf(s, 0.0f)) * (1.0f - 8.0f * kUlp) - (mq + s_mx[wave * 64 + u * 32 + r]);
                                // (out of the 16-bit range: nothing is known)
                                dist = dist < 1e18f && s < 1e36f ? __builtin_fmaxf(dist, 0.0f) : 0.0f;
                                out[r] = dist * dist * back;
                            }
                        }
                    }
                }
            }
            sync_block();
            // who did not fit comes to the front
            const int rest = have - nqs;
            int r_row = 0, r_c0 = 0, r_end = 0;
            float r_nq = 0.0f, r_mq = 0.0f;
            if (tid < rest) {
                r_row = s_row[nqs + tid]; r_c0 = s_c0[nqs + tid]; r_end = s_end[nqs + tid];
                r_nq = s_nq[nqs + tid]; r_mq = s_mq[nqs + tid];
            }
            sync_block();
            if (tid < rest) { s_row[tid] = r_row; s_c0[tid] = r_c0; s_end[tid] = r_end; s_nq[tid] = r_nq; s_mq[tid] = r_mq; }
            have = rest;
            sync_block();
        }
    }
}

// ---- distance tables of many queries ----
// 256 entries per workgroup (a subspace; 16 of them with 4-bit codes), four centroids per lane kept in registers, and
// one wave per query and step: a query's 256 entries are one 1 KB store.  The kernel before it built a query's
// rows from the centroids' memory (1.5 MB per query of 1536 values): 175 us for 2000 x 192 rows, 393 MB; now 97 us (4.1 TB/s).
// Bound by writing.  VERIFY: lut is a caller's, bad[query] is set unless its entries are the
// centroids' distances bit for bit.  by_slot: a query's table is at its place in the order, else at its number.
template <int DSUB, bool FS, bool VERIFY>
__global__ __launch_bounds__(256) void lut_tile_kernel(const LutArgs a) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int entries = a.nsub * (FS ? kC4 : kC), e = blockIdx.x * 256 + 4 * lane;
    const bool on = e < entries;
    const int sj = FS ? (on ? e >> 4 : 0) : (int)blockIdx.x;
    float c[4][DSUB];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int t = 0; t < DSUB; ++t) c[u][t] = a.codebooks[(size_t)(on ? e + u : u) * DSUB + t];
    const int64_t s0 = (int64_t)blockIdx.y * kLutQueries + wave;
#pragma unroll 2
    for (int i = 0; i < kLutQueries; i += 4) {
        const int64_t slot = s0 + i;
        if (slot >= a.nslots) break;
        const int64_t q = a.order ? a.order[a.slot0 + slot] : a.slot0 + slot;
        if (q < 0 || q >= a.nq) continue;
        const float *x = a.queries + (size_t)q * a.d + sj * DSUB;
        float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int t = 0; t < DSUB; ++t) {
            const float xt = x[t];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float v = xt - c[u][t];
                acc[u] = __builtin_fmaf(v, v, acc[u]);
            }
        }
        if (!on) continue;
        float4 *out = reinterpret_cast<float4 *>(a.lut + (size_t)(a.by_slot ? slot : q) * entries + e);
        if constexpr (VERIFY) {
            const float4 v = *out;
            if (__float_as_uint(v.x) != __float_as_uint(acc[0]) || __float_as_uint(v.y) != __float_as_uint(acc[1]) ||
                __float_as_uint(v.z) != __float_as_uint(acc[2]) || __float_as_uint(v.w) != __float_as_uint(acc[3]))
                a.bad[q] = 1;
        } else {
            *out = make_float4(acc[0], acc[1], acc[2], acc[3]);
        }
    }
}

// ---- finish: the bounds of the marked candidates, by the rule ----
// One workgroup per query: its table in the LDS (rows of one phase at a time), its marked candidates
// (or, all: every candidate of the pass) listed a few thousand at a time, one per thread; who does not
// pass is unmarked.  PICK: only the queries that a.only names.
template <int VEC, bool FS, bool PICK>
__global__ __launch_bounds__(1024)
__attribute__((amdgpu_waves_per_eu(4)))
void finish_kernel(const FinishArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    float *tab = reinterpret_cast<float *>(smem);
    float *q_lds = reinterpret_cast<float *>(smem + a.off_q);
    int *segp = reinterpret_cast<int *>(smem + a.off_segp);
    int *segd = reinterpret_cast<int *>(smem + a.off_segd);
    uint32_t *bits = reinterpret_cast<uint32_t *>(smem + a.off_bits);   // [kFinishPiece / 32], then the waves' counts
    int *part = reinterpret_cast<int *>(bits + kFinishPiece / 32);      // [16]
    uint16_t *list = reinterpret_cast<uint16_t *>(smem + a.off_ring);   // [kFinishList]
    const int tid = threadIdx.x, T = blockDim.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int64_t per_xcd = (a.nslots + kXcds - 1) / kXcds;
    const int64_t slot = (int64_t)(blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
    if (slot >= a.nslots) return;
    const int64_t q = a.order ? a.order[a.slot0 + slot] : a.slot0 + slot;
    if (q < 0 || q >= a.nq) {
        if (!a.by_query && a.totals && a.lo == 0 && tid == 0) a.totals[slot] = 0;
        return;
    }
    if (PICK && (a.bad[q] != 0) != (a.only == kFinishBad)) return;
    const int64_t row = a.by_query ? q : slot;
    const int nseg = a.nseg > 0 ? a.nseg : 1;
    // the first rows of the table are on their way while the rest is made ready
    typedef float f4 __attribute__((ext_vector_type(4)));
    constexpr int kPre = 8;
    f4 pre[kPre] = {};
    const f4 *lut = a.lut ? reinterpret_cast<const f4 *>(a.lut + (size_t)(a.lut_by_row ? row : q) * a.M * kByteEntries<FS>) : nullptr;
    const bool ahead = lut && !a.certain;      // (few table sums: few queries need a table at all)
    const int n_pre = a.Mp * (kByteEntries<FS> / 4);
    if (ahead) {
#pragma unroll
        for (int i = 0; i < kPre; ++i) pre[i] = lut[tid + i * T < n_pre ? tid + i * T : 0];
    }
    for (int t = tid; t < a.d; t += T) q_lds[t] = a.queries[(size_t)q * a.d + t];
    segment_table_ready(a.seg, a.nseg, a.n, a.max_cand, row, segp, segd);
    const int total = segp[nseg];
    if (a.lo == 0 && tid == 0) {
        a.totals[row] = total;
        if (a.n_scanned) a.n_scanned[q] = total;
    }
    const int lo = a.lo < total ? a.lo : total, hi = a.hi < total ? a.hi : total;
    if (lo >= hi) return;
    const float tau = a.range ? a.radius2 : a.tau_of ? a.tau_of[(size_t)q * a.tau_stride] : __builtin_inff();
    auto fill = [&](int j0, int nj) {
        if (lut) {
            const f4 *src = lut + (size_t)j0 * (kByteEntries<FS> / 4);
            f4 *dst = reinterpret_cast<f4 *>(tab);
            const int all = nj * (kByteEntries<FS> / 4);
            for (int e = tid; e < all; e += kPre * T) {
                f4 v[kPre];
#pragma unroll
                for (int i = 0; i < kPre; ++i) v[i] = src[e + i * T < all ? e + i * T : e];
#pragma unroll
                for (int i = 0; i < kPre; ++i)
                    if (e + i * T < all) dst[e + i * T] = v[i];
            }
        } else {
            build_table_rows<FS>(tab, q_lds, a.codebooks, a.dsub, j0, nj);
        }
    };
    uint32_t *row_bits = a.possible + (size_t)row * a.words;
    float *row_g = a.g + (size_t)row * a.words * 32;
    int n_marked = 0, in_place = -1;            // the phase whose rows are in place
    if (ahead) {
        f4 *dst = reinterpret_cast<f4 *>(tab);
#pragma unroll
        for (int i = 0; i < kPre; ++i)
            if (tid + i * T < n_pre) dst[tid + i * T] = pre[i];
        for (int e = tid + kPre * T; e < n_pre; e += T) dst[e] = lut[e];
        in_place = 0;                            // (barriers follow)
    }
    // The filter went by the centroids.  A caller's table may hold something else: unless its entries are the
    // centroids' distances bit for bit (lut_tile_kernel), every candidate of the query counts as marked.
    const bool all_marked = a.all != 0 || (a.bad != nullptr && a.bad[q] != 0);
    const uint32_t *row_in = a.certain && !all_marked ? a.certain + (size_t)row * a.words : nullptr;
    for (int p0 = lo & ~31; p0 < hi; p0 += kFinishPiece) {
        const int S = hi - p0 < kFinishPiece ? hi - p0 : kFinishPiece;
        const int nwords = (S + 31) >> 5;
        // (one word per thread and step; T >= 512)
        int all = 0;
        bool some = false;
        for (int w = tid; w < kFinishPiece / 32; w += T) {
            uint32_t b = 0;
            if (w < nwords) {
                b = all_marked ? ~0u : row_bits[(p0 >> 5) + w];
                if (p0 + w * 32 < lo) b &= ~0u << (lo - p0 - w * 32);
                if (p0 + w * 32 + 32 > hi) b &= (1u << (hi - p0 - w * 32)) - 1u;
            }
            bits[w] = b;
            if (row_in && w < nwords) b &= ~row_in[(p0 >> 5) + w];
            some = some || b != 0;
        }
        if (row_in) {           // (nobody's sum wanted in this piece: no table either)
            const bool here = __any(some);
            if (lane == 0) part[wave] = here ? 1 : 0;
            sync_block();
            some = false;
            for (int v = 0; v < T / kWave; ++v) some = some || part[v] != 0;
        } else {
            some = true;
        }
        sync_block();
        for (int ph = 0; some && ph < a.P; ++ph) {
            const bool last = ph == a.P - 1;
            if (in_place != ph) { fill(ph * a.Mp, a.Mp); in_place = ph; sync_block(); }
            for (int w0 = 0; w0 < nwords; w0 += T) {
                uint32_t b = w0 + tid < nwords ? bits[w0 + tid] : 0u;
                if (row_in && w0 + tid < nwords) b &= ~row_in[(p0 >> 5) + w0 + tid];      // (these keep their mark)
                const int cnt = __popc(b);
                int incl = cnt;
#pragma unroll
                for (int off = 1; off < kWave; off <<= 1) {
                    const int v = __shfl_up(incl, off);
                    if (lane >= off) incl += v;
                }
                if (lane == kWave - 1) part[wave] = incl;
                sync_block();
                int before = incl - cnt;
                all = 0;
                for (int v = 0; v < T / kWave; ++v) {
                    const int x = part[v];
                    if (v < wave) before += x;
                    all += x;
                }
                for (int e0 = 0; e0 < all; e0 += kFinishList) {
                    const int np = all - e0 < kFinishList ? all - e0 : kFinishList;
                    uint32_t rem = b;
                    int at = before - e0;
                    while (rem) {
                        if (at >= 0 && at < np) list[at] = (uint16_t)((w0 + tid) * 32 + (__ffs((int)rem) - 1));
                        rem &= rem - 1;
                        ++at;
                    }
                    sync_block();
                    for (int i = tid; i < np; i += T) {
                        const int cl = list[i];
                        const int pos = segment_position(p0 + cl, segp, segd, nseg);
                        const uint8_t *code = a.codes + (size_t)pos * a.M + ph * a.Mp;
                        const float b1 = last ? a.dlx[pos] : 0.0f;
                        float sum = ph > 0 ? row_g[p0 + cl] : 0.0f;
                        constexpr int kAhead = 6;
                        for (int j = 0; j < a.Mp; j += kAhead * 4 * VEC) {
                            uint32_t w[kAhead][VEC];
#pragma unroll
                            for (int c = 0; c < kAhead; ++c)
                                if (j + c * 4 * VEC < a.Mp) load_codes<VEC>(w[c], code + j + c * 4 * VEC);
#pragma unroll
                            for (int c = 0; c < kAhead; ++c)
                                if (j + c * 4 * VEC < a.Mp)
                                    sum = gather_add<VEC, false, FS>(sum, (j + c * 4 * VEC) * kByteRow<FS>, w[c], __builtin_inff());
                        }
                        float keep = sum;
                        if (last) {
                            keep = plb_from_s(sum, b1, a.two_gamma);
                            // (the seed is measured whatever its bounds, also where they are no numbers)
                            if (!a.all && !(keep <= tau)) atomicAnd(&bits[cl >> 5], ~(1u << (cl & 31)));
                        }
                        row_g[p0 + cl] = keep;
                    }
                    sync_block();
                }
                sync_block();     // part[] is read (where nothing is marked no barrier has come since)
            }
        }
        for (int w = tid; w < nwords; w += T) {
            const uint32_t b = bits[w];
            if (a.range) {
                n_marked += __popc(b);
                if (a.mask && b) {
                    const int64_t wi = (p0 >> 5) + w;
                    if (wi < a.mask_words) atomicOr(&a.mask[(size_t)q * a.mask_words + wi], b);
                }
            }
            // (the marks of the pass before stay: they may not be read yet)
            const uint32_t before = p0 + w * 32 < lo ? row_bits[(p0 >> 5) + w] & ((1u << (lo - p0 - w * 32)) - 1u) : 0u;
            row_bits[(p0 >> 5) + w] = b | before;
        }
        sync_block();
    }
    if (a.range && a.n_exact) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) n_marked += __shfl_xor(n_marked, off);
        if (lane == 0 && n_marked) atomicAdd(&a.n_exact[q], n_marked);
    }
}

// ---- which queries scan a list ----

// kInvPer (query, probe) pairs per workgroup, counted in the LDS first where the lists have room there (kInvLists): with one atomic
// operation in memory per pair, 160,000 of them on 1024 counters took 35 us, now 7.
constexpr int kInvPer = 2048, kInvLists = 16384;
__global__ __launch_bounds__(1024) void invert_count_kernel(const InvertArgs a) {
    extern __shared__ __align__(16) int32_t s_cnt[];      // [nlist], or nothing
    const bool lds = a.nlist <= kInvLists;
    if (lds) {
        for (int l = threadIdx.x; l < a.nlist; l += blockDim.x) s_cnt[l] = 0;
        sync_block();
    }
    for (int64_t i = (int64_t)blockIdx.x * kInvPer + threadIdx.x; i < ((int64_t)blockIdx.x + 1) * kInvPer && i < a.nslots * a.nseg; i += blockDim.x) {
        const int64_t slot = i / a.nseg, q = a.query(slot);
        if (q < 0) continue;
        const int32_t l = a.probes[(size_t)q * a.nseg + (i - slot * a.nseg)];
        if (l >= 0 && l < a.nlist) atomicAdd(lds ? &s_cnt[l] : &a.cnt[l], 1);
    }
    if (!lds) return;
    sync_block();
    for (int l = threadIdx.x; l < a.nlist; l += blockDim.x)
        if (s_cnt[l]) atomicAdd(&a.cnt[l], s_cnt[l]);
}
// cnt [nlist] -> start [nlist + 1], and cnt becomes the running slots.  Single workgroup.
__global__ __launch_bounds__(1024) void invert_scan_kernel(const InvertArgs a) {
    int32_t *cnt = a.cnt, *start = a.start;
    const int nlist = a.nlist;
    __shared__ int part[16], tpart[16], rpart[16];
    __shared__ int carry, tcarry, rcarry;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) carry = tcarry = rcarry = 0;
    sync_block();
    for (int l0 = 0; l0 < nlist; l0 += 1024) {
        const int l = l0 + tid, v = l < nlist ? cnt[l] : 0;
        int t = 0, rt = 0;
        if (l < nlist && v > 0) {        // tiles of the filter: rows x queries
            int64_t s = a.list_offsets[l], e = a.list_offsets[l + 1];
            s = s < 0 ? 0 : (s > a.n ? a.n : s);
            e = e < s ? s : (e > a.n ? a.n : e);
            const int64_t len = e - s < a.max_cand ? e - s : a.max_cand;       // (no query comes further; see counts_fit)
            t = (int)((len + kFltRows - 1) / kFltRows) * ((v + kFltQ - 1) / kFltQ);
            rt = (int)((len + kMsrRows - 1) / kMsrRows) * ((v + kMsrBlock - 1) / kMsrBlock);     // (measure)
        }
        int incl = v, tincl = t, rincl = rt;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int o = __shfl_up(incl, off), to = __shfl_up(tincl, off), ro = __shfl_up(rincl, off);
            if (lane >= off) { incl += o; tincl += to; rincl += ro; }
        }
        if (lane == 63) { part[wave] = incl; tpart[wave] = tincl; rpart[wave] = rincl; }
        sync_block();
        int before = carry, tbefore = tcarry, rbefore = rcarry;
        for (int w = 0; w < wave; ++w) { before += part[w]; tbefore += tpart[w]; rbefore += rpart[w]; }
        if (l < nlist) {
            start[l] = before + incl - v;
            cnt[l] = before + incl - v;
            a.tasks[l] = tbefore + tincl - t;
            a.row_tasks[l] = rbefore + rincl - rt;
        }
        sync_block();
        if (tid == 1023) { carry = before + incl; tcarry = tbefore + tincl; rcarry = rbefore + rincl; }
        sync_block();
    }
    if (tid == 0) {
        start[nlist] = carry;
        a.tasks[nlist] = tcarry;
        a.row_tasks[nlist] = rcarry;
    }
}
// One wave per query, kInvQueries queries per workgroup.  A workgroup takes its places of every list at once: its pairs are numbered in
// the LDS, then the lists' counters are moved on by their numbers.
constexpr int kInvQueries = 32;
__global__ __launch_bounds__(1024) void invert_place_kernel(const InvertArgs a) {
    extern __shared__ __align__(16) int32_t s_cnt[];      // [nlist]: pairs so far, then the first place; or nothing
    const bool lds = a.nlist <= kInvLists;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nseg = a.nseg;
    constexpr int kWaves = 1024 / kWave;
    if (lds) {
        for (int l = threadIdx.x; l < a.nlist; l += 1024) s_cnt[l] = 0;
        sync_block();
    }
    // twice over the pairs: numbers and segment tables, then places
    for (int round = lds ? 0 : 1; round < 2; ++round) {
        for (int qi = wave; qi < kInvQueries; qi += kWaves) {
            const int64_t slot = (int64_t)blockIdx.x * kInvQueries + qi;
            if (slot >= a.nslots) continue;
            const int64_t q = a.query(slot);
            if (q < 0) continue;
            const int64_t row = a.by_query ? q : slot;
            int64_t carry = 0;
            for (int p0 = 0; p0 < nseg; p0 += kWave) {
                const int p = p0 + lane;
                int32_t l = p < nseg ? a.probes[(size_t)q * nseg + p] : -1;
                if (round == 0) {
                    if (l >= 0 && l < a.nlist) atomicAdd(&s_cnt[l], 1);
                    continue;
                }
                int64_t len = 0, first = 0;
                if (l >= 0 && l < a.nlist) {
                    int64_t s = a.list_offsets[l], e = a.list_offsets[l + 1];
                    s = s < 0 ? 0 : (s > a.n ? a.n : s);
                    e = e < s ? s : (e > a.n ? a.n : e);
                    len = e - s;
                    first = s;
                } else {
                    l = -1;
                }
                int64_t incl = len;
#pragma unroll
                for (int off = 1; off < kWave; off <<= 1) {
                    const int64_t v = __shfl_up((long long)incl, off);
                    if (lane >= off) incl += v;
                }
                const int64_t c0 = carry + incl - len, c1 = carry + incl;
                // (beyond 2^31 candidates nothing is scanned: such a list is placed out of reach)
                if (l >= 0) a.inv[atomicAdd(lds ? &s_cnt[l] : &a.cnt[l], 1)] = make_int2((int)row, c0 < 0x7fffffff ? (int)c0 : 0x7fffffff);
                if (p < nseg) {
                    const int64_t before = c0 < a.max_cand ? c0 : a.max_cand;
                    a.seg[(size_t)row * 2 * nseg + p] = (int)(c1 < a.max_cand ? c1 : a.max_cand);
                    a.seg[((size_t)row * 2 + 1) * nseg + p] = (int)(first - before);
                }
                carry += __shfl((long long)incl, kWave - 1);
            }
        }
        if (round == 0) {
            sync_block();
            for (int l = threadIdx.x; l < a.nlist; l += 1024)
                if (s_cnt[l]) s_cnt[l] = atomicAdd(&a.cnt[l], s_cnt[l]);
            sync_block();
        }
    }
}

// ---- a threshold for the rest before the first batch is measured (kNN) ----
// The a.picks vectors of the first batch with the least bounds have their exact distances taken, and of the larger of the
// two, over the picks, the k-th least is no less than the k-th distance tau that the first batch will leave.  (Either all of these k survive the
// seed's threshold and are in the running, or the bound of one exceeds that threshold, which is no less than tau.)  Any choice of picks will do
// for that: which of the same bin of the histogram are taken is left to chance.
// What is marked against it contains what tau would mark, so that the rows of the first batch and of the next pass are measured
// together and read once.  64 picks, k = 10: a bound of the rest lies below it for 0.372 of them where tau has 0.317 (unit vectors of 768 values,
// gamma 0.27, first batches of 1024; 10 picks 0.79, 128 0.337, 64 and 128 groups' least 0.405 and 0.365), and elsewhere as often as below tau.
// Bound by the rows, which neighbouring queries share: 2,500 queries over 500,000 x 768, 118 more of them cost 90 us.
// One workgroup per query.  A candidate whose bound is no number never passes a threshold and is left out, like an infinite one; a pick whose
// distance is no number counts as infinite, and so does what is missing where there are fewer.
__global__ __launch_bounds__(kReplayThreads) void pick_kernel(const ReplayArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    int *segp = reinterpret_cast<int *>(smem + a.off_segp), *segd = reinterpret_cast<int *>(smem + a.off_segd);
    float *q_lds = reinterpret_cast<float *>(smem + a.off_q);
    __shared__ int hist[256], s_at[kPicks], s_n, s_bin;
    __shared__ uint32_t s_low, s_high;
    __shared__ float s_bound[kPicks], s_val[kPicks];
    const int tid = threadIdx.x, half = tid >> 5, lane32 = tid & 31;
    const int64_t per_xcd = gridDim.x / kXcds, row = (int64_t)(blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
    if (row >= a.nslots) return;
    const int64_t q = a.order ? a.order[a.slot0 + row] : a.slot0 + row;
    if (q < 0 || q >= a.nq) return;
    const int picks = a.picks;
    const int total = a.totals[row], end = total < a.mid ? total : a.mid;
    constexpr int kHeld = kPickBatch / kReplayThreads;
    static_assert(kPickBatch % kReplayThreads == 0 && kPicks <= kReplayThreads, "the first batch in registers");
    uint32_t key[kHeld];                 // (bounds are not negative: they order as their bits)
    const float *g = a.g + (size_t)row * a.words * 32;
#pragma unroll
    for (int u = 0; u < kHeld; ++u) {
        const int i = a.k + u * kReplayThreads + tid;
        const float v = i < end ? g[i] : __builtin_inff();
        key[u] = v < __builtin_inff() ? __float_as_uint(v) : ~0u;
    }
    for (int t = tid; t < a.d; t += kReplayThreads) q_lds[t] = a.queries[(size_t)q * a.d + t];
    if (tid < 256) hist[tid] = 0;
    if (tid < kPicks) s_val[tid] = __builtin_inff();
    if (tid == 0) { s_low = ~0u; s_high = 0; s_n = 0; }
    segment_table_ready(a.seg, a.nseg, a.n, a.max_cand, row, segp, segd);
    uint32_t low = ~0u, high = 0;
#pragma unroll
    for (int u = 0; u < kHeld; ++u)
        if (key[u] != ~0u) { low = min(low, key[u]); high = max(high, key[u]); }
    wave_max(&s_high, high);
    if (low != ~0u) atomicMin(&s_low, low);
    sync_block();
    const uint32_t base = s_low, width = s_high > base ? s_high - base : 1u;
    const int shift = max(0, 24 - (int)__clz(width));       // 256 bins
#pragma unroll
    for (int u = 0; u < kHeld; ++u)
        if (key[u] != ~0u) atomicAdd(&hist[(key[u] - base) >> shift], 1);
    sync_block();
    if (tid < kWave) {                   // the bin that the last pick is in
        int c[4], sum = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) { c[e] = hist[4 * tid + e]; sum += c[e]; }
        int incl = sum;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int v = __shfl_up(incl, off);
            if (tid >= off) incl += v;
        }
        int run = incl - sum;
        if (tid == kWave - 1 && incl < picks) s_bin = 255;          // (all of them)
        if (run < picks && incl >= picks) {
            int b = 4 * tid;
#pragma unroll
            for (int e = 0; e < 4; ++e) { run += c[e]; if (run < picks) ++b; }
            s_bin = b;
        }
    }
    sync_block();
    const int bin = s_bin;
#pragma unroll
    for (int turn = 0; turn < 2; ++turn) {
#pragma unroll
        for (int u = 0; u < kHeld; ++u) {
            if (key[u] == ~0u) continue;
            const int mine = (int)((key[u] - base) >> shift);
            if (turn == 0 ? mine >= bin : mine != bin) continue;
            const int at = atomicAdd(&s_n, 1);
            if (at < picks) { s_at[at] = a.k + u * kReplayThreads + tid; s_bound[at] = __uint_as_float(key[u]); }
        }
        sync_block();
    }
    const int n = min(s_n, picks);
    for (int j = half; j < n; j += kReplayThreads / 32 * 2) {
        const int j1 = j + kReplayThreads / 32;
        float d2[2];
        exact_d2_half_x2_deep<4>(a.base + (size_t)segment_position(s_at[j], segp, segd, a.nseg) * a.d,
                                 a.base + (size_t)segment_position(s_at[j1 < n ? j1 : j], segp, segd, a.nseg) * a.d, q_lds, a.d, lane32, d2);
        if (lane32 == 0) {
            s_val[j] = d2[0] <= __builtin_inff() ? __builtin_fmaxf(d2[0], s_bound[j]) : __builtin_inff();
            if (j1 < n) s_val[j1] = d2[1] <= __builtin_inff() ? __builtin_fmaxf(d2[1], s_bound[j1]) : __builtin_inff();
        }
    }
    sync_block();
    if (tid < picks) {
        const float v = s_val[tid];
        int before = 0;
        for (int j = 0; j < picks; ++j) before += s_val[j] < v || (s_val[j] == v && j < tid);
        if (before == a.k - 1) a.out_d2[(size_t)q * a.k + a.k - 1] = v;
    }
}

// ---- replay (kNN) ----
// One workgroup per query.  The entries of a stretch are listed in scan order; the exact distance is taken
// here of those whose lower bound (a.d2) does not exceed the threshold at the start, the first wave
// goes through the batch rule with these, and all threads count the others by the thresholds it leaves.  (When the first
// wave went through all of them, the other seven waited: 2,500 queries x 500,000 x 768 472 -> 365 us, 500 x 300,000 x 960, k = 100,
// 963 -> 575.  Of a later pass's 340,000 clocks there, 144,000 were the first wave's, some 200 insertions one after the
// other, 80,000 the rows, 31,000 the bounds read.  A batch's entries inserted together, and that wave first on its SIMD: 537 -> 510 us.)
// The first pass (seed and first batch, lo == 0) is done by all threads: the seed's distances give the
// batch its threshold; of its survivors the k with the least lower bounds are measured, the largest of those
// distances bounds the k-th, so that only bounds up to it need measuring; a sort gives R.
template <int E>
__global__ __launch_bounds__(kReplayThreads) void replay_kernel(const ReplayArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    int *segp = reinterpret_cast<int *>(smem + a.off_segp), *segd = reinterpret_cast<int *>(smem + a.off_segd);
    int32_t *s_cl = reinterpret_cast<int32_t *>(smem + a.off_cl), *s_id = reinterpret_cast<int32_t *>(smem + a.off_id);
    float *s_g = reinterpret_cast<float *>(smem + a.off_g), *s_d2 = reinterpret_cast<float *>(smem + a.off_d2);
    float *rd2 = reinterpret_cast<float *>(smem + a.off_rd2);
    int32_t *rid = reinterpret_cast<int32_t *>(smem + a.off_rid);
    float *q_lds = reinterpret_cast<float *>(smem + a.off_q);
    unsigned long long *s_key = reinterpret_cast<unsigned long long *>(smem + a.off_key);   // [kReplayCap]
    uint16_t *s_todo = reinterpret_cast<uint16_t *>(smem + a.off_todo);                     // [kReplayCap]
    __shared__ int part[kReplayThreads / kWave];
    __shared__ int s_ntodo, s_count;
    __shared__ uint32_t s_most, s_bit[kReplayCap / 32];
    __shared__ TauSteps s_steps;
    static_assert(kReplayCap / 32 == kWave, "a word of the measured ones per lane");
    __shared__ float s_tau;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t row = blockIdx.x;       // one workgroup per place in the order
    const int64_t q = a.order ? a.order[a.slot0 + row] : a.slot0 + row;
    if (q < 0 || q >= a.nq) return;
    const int total = a.totals[row];
    const int lo = a.lo < total ? a.lo : total, hi = a.hi < total ? a.hi : total;
    if (a.lo > 0 && lo >= hi) return;        // nothing of this query in this pass: R stays as it is
    for (int t = tid; t < a.d; t += kReplayThreads) q_lds[t] = a.queries[(size_t)q * a.d + t];
    segment_table_ready(a.seg, a.nseg, a.n, a.max_cand, row, segp, segd);
    for (int i = tid; i < kWave * E; i += kReplayThreads) {
        const bool have = a.lo > 0 && i < a.k;
        const int32_t id = have ? a.out_ids[(size_t)q * a.k + i] : -1;
        rd2[i] = have ? a.out_d2[(size_t)q * a.k + i] : __builtin_inff();
        rid[i] = id < 0 ? kEmptyId : id;
    }
    sync_block();
    ResultRegs<E> R;
    int frozen_b = -2, survivors = 0;          // (survivors: this thread's)
    float tau_f = 0.0f;
    if (wave == 0) {
        R.load(rd2, rid, a.k, lane);
        if (lane == 0) s_tau = R.t_d2;
    }
    const uint32_t *bits = a.possible + (size_t)row * a.words;
    const float *row_g = a.g + (size_t)row * a.words * 32, *row_d2 = a.d2 + (size_t)row * a.words * 32;
    uint32_t *mask_row = a.mask ? a.mask + (size_t)q * a.mask_words : nullptr;
    // the exact distances of the entries s_todo[0 .. n), by half waves, two rows each; s_id: positions before, ids after
    auto measure = [&](int n) {
        const int half = tid >> 5, lane32 = tid & 31;
        constexpr int kHalves = kReplayThreads / 32;
        for (int i = half; i < n; i += 2 * kHalves) {
            const int e0 = s_todo[i], e1 = s_todo[i + kHalves < n ? i + kHalves : i];
            const int p0 = segment_position(s_cl[e0], segp, segd, a.nseg), p1 = segment_position(s_cl[e1], segp, segd, a.nseg);
            const int32_t id0 = a.ids ? a.ids[p0] : p0, id1 = a.ids ? a.ids[p1] : p1;
            float d2[2];
            exact_d2_half_x2_deep<4>(a.base + (size_t)p0 * a.d, a.base + (size_t)p1 * a.d, q_lds, a.d, lane32, d2);
            if (lane32 == 0) {
                s_d2[e0] = d2[0]; s_id[e0] = id0;
                s_d2[e1] = d2[1]; s_id[e1] = id1;
            }
        }
        sync_block();
    };
    // (with the first batch, the pass after it: see pick_kernel)
    const int mid = a.mid > lo && a.mid < hi ? a.mid : hi;
    for (int turn = 0; turn < 2; ++turn) {
        const int part_lo = turn ? mid : lo, part_hi = turn ? hi : mid;
        const int w_end = part_lo < part_hi ? (part_hi + 31) >> 5 : 0;
        for (int w0 = part_lo >> 5; w0 < w_end; w0 += kReplayThreads) {
            const int w = w0 + tid;
            uint32_t b = w < w_end ? bits[w] : 0u;
            if (w == part_lo >> 5) b &= ~0u << (part_lo & 31);
            if (w == part_hi >> 5) b &= (1u << (part_hi & 31)) - 1u;
            const int cnt = __popc(b);
            int incl = cnt;
#pragma unroll
            for (int off = 1; off < kWave; off <<= 1) {
                const int v = __shfl_up(incl, off);
                if (lane >= off) incl += v;
            }
            if (lane == 63) part[wave] = incl;
            sync_block();
            int before = incl - cnt, all = 0;
            for (int v = 0; v < kReplayThreads / kWave; ++v) {
                const int p = part[v];
                if (v < wave) before += p;
                all += p;
            }
            for (int e0 = 0; e0 < all; e0 += kReplayCap) {
                const int np = all - e0 < kReplayCap ? all - e0 : kReplayCap;
                uint32_t rem = b;
                int at = before - e0;
                while (rem) {
                    const int c = w * 32 + (__ffs((int)rem) - 1);
                    rem &= rem - 1;
                    if (at >= 0 && at < np) s_cl[at] = c;
                    ++at;
                }
                if (tid == 0) s_ntodo = 0;
                if (tid < kReplayCap / 32) s_bit[tid] = 0;
                sync_block();
                const float tau = s_tau;
                // the seed and the first batch, whole (the candidates of this pass are all marked)
                if (part_lo == 0 && part_hi <= (int64_t)a.k + a.batch && all == np && np == part_hi) {
                    const int ns = np < a.k ? np : a.k;
                    for (int i = tid; i < np; i += kReplayThreads) {
                        const int c = s_cl[i];
                        s_g[i] = row_g[c];
                        s_d2[i] = row_d2[c];
                        if (i < ns) s_todo[i] = (uint16_t)i;
                    }
                    if (tid == 0) { s_most = 0; s_count = 0; }
                    sync_block();
                    measure(ns);
                    uint32_t most = 0;
                    for (int i = tid; i < ns; i += kReplayThreads) most = max(most, __float_as_uint(s_d2[i]));
                    wave_max(&s_most, most);
                    sync_block();
                    // (a distance that is no number is never in R: then R is not full yet)
                    const float tau1 = ns == a.k && s_most <= 0x7f800000u ? __uint_as_float(s_most) : __builtin_inff();
                    int mine = 0;
                    for (int i = tid; i < np; i += kReplayThreads) {
                        const bool on = i < ns || s_g[i] <= tau1;
                        if (on) {
                            ++mine;
                            if (mask_row && (i >> 5) < a.mask_words) atomicOr(&mask_row[i >> 5], 1u << (i & 31));
                            // who could enter R at all, by lower bound (seeds: measured already)
                            if (i >= ns && s_d2[i] <= tau1)
                                s_key[atomicAdd(&s_ntodo, 1)] = ((unsigned long long)__float_as_uint(s_d2[i]) << 32) | (uint32_t)i;
                        }
                    }
                    wave_add(&s_count, mine);
                    sync_block();
                    int nc = s_ntodo;
                    if (tid == 0) survivors += s_count;
                    int size = 1;
                    while (size < nc) size <<= 1;
                    for (int i = nc + tid; i < size; i += kReplayThreads) s_key[i] = ~0ull;
                    sync_block();
                    sort_keys(s_key, size);
                    const int first = nc < a.k ? nc : a.k;
                    for (int i = tid; i < first; i += kReplayThreads) s_todo[i] = (uint16_t)s_key[i];
                    if (tid == 0) s_most = 0;
                    sync_block();
                    measure(first);
                    most = 0;
                    for (int i = tid; i < first; i += kReplayThreads) most = max(most, __float_as_uint(s_d2[s_todo[i]]));
                    wave_max(&s_most, most);
                    if (tid == 0) s_ntodo = 0;
                    sync_block();
                    // (a distance that is no number bounds nothing)
                    const float cut = first == a.k && s_most <= 0x7f800000u ? __uint_as_float(s_most) : __builtin_inff();
                    int more = 0;                         // bounds are ascending: a prefix
                    for (int i = first + tid; i < nc; i += kReplayThreads) {
                        const bool need = __uint_as_float((uint32_t)(s_key[i] >> 32)) <= cut;
                        if (need) { s_todo[i - first] = (uint16_t)s_key[i]; ++more; }
                    }
                    wave_add(&s_ntodo, more);
                    sync_block();
                    const int n2 = s_ntodo;
                    measure(n2);
                    nc = first + n2;
                    // R: the k least of the seed and the measured ones, by (distance, id)
                    for (int i = tid; i < nc; i += kReplayThreads) {
                        const int e = (int)(uint32_t)s_key[i];
                        s_key[i] = ((unsigned long long)__float_as_uint(s_d2[e]) << 32) | ((uint32_t)s_id[e] ^ 0x80000000u);   // (ids order as signed)
                    }
                    size = 1;
                    while (size < nc + ns) size <<= 1;
                    for (int i = tid; i < ns; i += kReplayThreads)
                        s_key[nc + i] = ((unsigned long long)__float_as_uint(s_d2[i]) << 32) | ((uint32_t)s_id[i] ^ 0x80000000u);
                    for (int i = nc + ns + tid; i < size; i += kReplayThreads) s_key[i] = ~0ull;
                    sync_block();
                    sort_keys(s_key, size);
                    const int have = nc + ns < a.k ? nc + ns : a.k;
                    for (int i = tid; i < kWave * E; i += kReplayThreads) {
                        const bool in = i < have && (uint32_t)(s_key[i] >> 32) <= 0x7f800000u;      // (what is no number sorts last)
                        rd2[i] = in ? __uint_as_float((uint32_t)(s_key[i] >> 32)) : __builtin_inff();
                        rid[i] = in ? (int32_t)((uint32_t)s_key[i] ^ 0x80000000u) : kEmptyId;
                    }
                    sync_block();
                    if (wave == 0) {
                        R.load(rd2, rid, a.k, lane);
                        if (lane == 0) s_tau = R.t_d2;
                    }
                    continue;
                }
                for (int i = tid; i < np; i += kReplayThreads) {
                    const int c = s_cl[i];
                    const float d2 = row_d2[c], g = row_g[c];
                    s_g[i] = g;
                    // (its bound is held against the threshold of its own batch, later)
                    if (d2 <= tau) {
                        s_todo[atomicAdd(&s_ntodo, 1)] = (uint16_t)i;
                        atomicOr(&s_bit[i >> 5], 1u << (i & 31));
                    }
                }
                sync_block();
                const int nt = s_ntodo;
                measure(nt);
                if (wave == 0) {
                    __builtin_amdgcn_s_setprio(3);       // (the workgroup waits for this wave)
                    // the measured ones in scan order
                    uint32_t word = s_bit[lane];
                    const int ones = __popc(word);
                    int place = ones;
#pragma unroll
                    for (int off = 1; off < kWave; off <<= 1) {
                        const int v = __shfl_up(place, off);
                        if (lane >= off) place += v;
                    }
                    place -= ones;
                    while (word) {
                        s_todo[place++] = (uint16_t)(lane * 32 + (__ffs((int)word) - 1));
                        word &= word - 1;
                    }
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    replay_measured<E>(R, frozen_b, tau_f, s_cl, s_g, s_d2, s_id, s_todo, nt, a.batch, &s_steps, s_key);
                    if (lane == 0) s_tau = R.t_d2;
                    __builtin_amdgcn_s_setprio(0);
                }
                sync_block();
                const TauSteps steps = s_steps;
                for (int i = tid; i < np; i += kReplayThreads) {
                    const int c = s_cl[i], b4 = c < a.k ? -1 : (c - a.k) / a.batch;
                    if (b4 < 0 || s_g[i] <= threshold_of(b4, steps, s_key)) {
                        ++survivors;
                        if (mask_row && (c >> 5) < a.mask_words) atomicOr(&mask_row[c >> 5], 1u << (c & 31));
                    }
                }
                sync_block();
            }
            sync_block();
        }
    }
    if (a.n_exact) {
        if (tid == 0) s_count = 0;
        sync_block();
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) survivors += __shfl_xor(survivors, off);
        if (lane == 0 && survivors) atomicAdd(&s_count, survivors);
        sync_block();
        if (tid == 0) a.n_exact[q] = s_count + (a.lo > 0 ? a.n_exact[q] : 0);
    }
    if (wave == 0) R.store(rd2, rid);
    sync_block();
    for (int i = tid; i < a.k; i += kReplayThreads) {
        const int32_t id = rid[i];
        a.out_ids[(size_t)q * a.k + i] = id == kEmptyId ? -1 : id;
        a.out_d2[(size_t)q * a.k + i] = rd2[i];
    }
}

// ---- exact distances of a range search's marked candidates (a.d2: their lower bounds) ----
// One workgroup per (query, chunk): those whose bound does not exceed the radius are listed and measured by half waves;
// results keep their mark and leave their distance, the others are unmarked.
__global__ __launch_bounds__(kReplayThreads) void range_exact_kernel(const ReplayArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    int *segp = reinterpret_cast<int *>(smem + a.off_segp), *segd = reinterpret_cast<int *>(smem + a.off_segd);
    int32_t *s_cl = reinterpret_cast<int32_t *>(smem + a.off_cl);     // [kReplayCap]
    float *q_lds = reinterpret_cast<float *>(smem + a.off_q);
    uint32_t *s_word = reinterpret_cast<uint32_t *>(smem + a.off_key);  // [kReplayThreads] words in work
    __shared__ int part[kReplayThreads / kWave];
    __shared__ int s_n;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t q = a.order ? a.order[blockIdx.x] : (int64_t)blockIdx.x;
    if (q < 0 || q >= a.nq) return;
    const int total = a.totals[q];
    const int lo = (int)blockIdx.y * a.chunk, hi = lo + a.chunk < total ? lo + a.chunk : total;
    if (lo >= hi) return;
    for (int t = tid; t < a.d; t += kReplayThreads) q_lds[t] = a.queries[(size_t)q * a.d + t];
    segment_table_ready(a.seg, a.nseg, a.n, a.max_cand, q, segp, segd);
    uint32_t *bits = a.bits + (size_t)q * a.words;
    float *row_d2 = a.d2_out + (size_t)q * a.words * 32;
    const int half = tid >> 5, lane32 = tid & 31;
    int results = 0;
    const int w_end = (hi + 31) >> 5;
    for (int w0 = lo >> 5; w0 < w_end; w0 += kReplayThreads) {
        const int w = w0 + tid;
        uint32_t b = w < w_end ? bits[w] : 0u, out = b;
        const int cnt = __popc(b);
        int incl = cnt;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int v = __shfl_up(incl, off);
            if (lane >= off) incl += v;
        }
        if (lane == 63) part[wave] = incl;
        s_word[tid] = b;
        sync_block();
        int before = incl - cnt, all = 0;
        for (int v = 0; v < kReplayThreads / kWave; ++v) {
            const int p = part[v];
            if (v < wave) before += p;
            all += p;
        }
        for (int e0 = 0; e0 < all; e0 += kReplayCap) {
            const int np = all - e0 < kReplayCap ? all - e0 : kReplayCap;
            uint32_t rem = b;
            int at = before - e0;
            while (rem) {
                if (at >= 0 && at < np) s_cl[at] = w * 32 + (__ffs((int)rem) - 1);
                rem &= rem - 1;
                ++at;
            }
            if (tid == 0) s_n = 0;
            sync_block();
            // bounds beyond the radius leave at once; the others are listed in place of the candidates
            int keep[kReplayCap / kReplayThreads];
#pragma unroll
            for (int v = 0; v < kReplayCap / kReplayThreads; ++v) {
                const int i = tid + v * kReplayThreads;
                keep[v] = -1;
                if (i < np) {
                    const int c = s_cl[i];
                    if (row_d2[c] <= a.radius2) keep[v] = c;
                    else atomicAnd(&s_word[(c >> 5) - w0], ~(1u << (c & 31)));
                }
            }
            sync_block();
#pragma unroll
            for (int v = 0; v < kReplayCap / kReplayThreads; ++v)
                if (keep[v] >= 0) s_cl[atomicAdd(&s_n, 1)] = keep[v];
            sync_block();
            const int n = s_n;
            constexpr int kHalves = kReplayThreads / 32;
            for (int i = half; i < n; i += 2 * kHalves) {
                const int c0 = s_cl[i], c1 = s_cl[i + kHalves < n ? i + kHalves : i];
                const int p0 = segment_position(c0, segp, segd, a.nseg), p1 = segment_position(c1, segp, segd, a.nseg);
                float d2[2];
                exact_d2_half_x2_deep<4>(a.base + (size_t)p0 * a.d, a.base + (size_t)p1 * a.d, q_lds, a.d, lane32, d2);
                if (lane32 == 0) {
#pragma unroll
                    for (int v = 0; v < 2; ++v) {           // (the last one twice where their number is odd)
                        const int c = v == 0 ? c0 : c1;
                        if (d2[v] <= a.radius2) row_d2[c] = d2[v];
                        else atomicAnd(&s_word[(c >> 5) - w0], ~(1u << (c & 31)));
                    }
                }
            }
            sync_block();
        }
        out = s_word[tid];
        if (w < w_end) {
            if (out != b) bits[w] = out;
            results += __popc(out);
        }
        sync_block();
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) results += __shfl_xor(results, off);
    if (lane == 0 && results) atomicAdd(&a.counts[(size_t)q * a.nchunk + blockIdx.y], results);
}

}  // namespace trim
