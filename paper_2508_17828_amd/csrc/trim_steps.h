// Device functions that the kernels of trim_mark.h and trim_few.h share.
#pragma once

#include "trim_search.h"

namespace trim {

// The segment table of a query (see SearchArgs): segp[0..nseg] prefix of the lengths, cut at max_cand,
// segd[p] = storage position of the segment's first candidate less its scan-order number.  All
// threads of the workgroup; ends with a barrier.  Sums saturate at max_cand < 2^31, so 32 bits do.
__device__ __forceinline__ void segment_table(const int64_t *list_offsets, const int32_t *probes, int nlist, int nseg,
                                              int64_t n, int max_cand, int64_t q, int *segp, int *segd) {
    const int ns = nseg > 0 ? nseg : 1;
    for (int p = threadIdx.x; p < ns; p += blockDim.x) {
        int64_t s = 0, e = n;
        if (nseg > 0) {
            const int32_t l = probes[(size_t)q * nseg + p];
            if (l >= 0 && l < nlist) {
                s = list_offsets[l];
                e = list_offsets[l + 1];
                s = s < 0 ? 0 : (s > n ? n : s);
                e = e < s ? s : (e > n ? n : e);
            } else {
                s = e = 0;
            }
        }
        segd[p] = (int)s;
        segp[p + 1] = (int)(e - s);
    }
    sync_block();
    if (threadIdx.x < kWave) segment_prefix(segp, segd, ns, (uint32_t)max_cand);
    sync_block();
}

// The same where it has been made already (invert_place_kernel): one look at memory instead of three, one after the other.
__device__ __forceinline__ void segment_table_ready(const int32_t *seg, int nseg, int64_t n, int max_cand, int64_t row, int *segp, int *segd) {
    if (seg) {
        for (int p = threadIdx.x; p < nseg; p += blockDim.x) {
            segp[p + 1] = seg[(size_t)row * 2 * nseg + p];
            segd[p] = seg[((size_t)row * 2 + 1) * nseg + p];
        }
    } else if (threadIdx.x == 0) {
        segp[1] = (int)(n < max_cand ? n : max_cand);
        segd[0] = 0;
    }
    if (threadIdx.x == 0) segp[0] = 0;
    sync_block();
}

// Into a word of the LDS, one atomic a wave: lanes with a value each, the compiler would let take their turns (64 of them, some
// 10,000 clocks where 16 waves do).  All lanes take part.
__device__ __forceinline__ void wave_add(int *to, int v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & (kWave - 1)) == 0 && v) atomicAdd(to, v);
}
__device__ __forceinline__ void wave_max(uint32_t *to, uint32_t v) {
    if (__ballot(v != 0) == 0) return;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, off));
    if ((threadIdx.x & (kWave - 1)) == 0) atomicMax(to, v);
}

__device__ __forceinline__ int segment_position(int c, const int *segp, const int *segd, int nseg) {
    int lo = 0, hi = (nseg > 0 ? nseg : 1) - 1;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (c >= segp[mid + 1]) lo = mid + 1; else hi = mid;
    }
    return c + segd[lo];
}

// The batch rule over entries in scan order (replay_batches; the state of a batch that the next
// call goes on with is kept in frozen_b and tau_f).  cl: candidate number; the first k candidates
// are the seed: a batch of their own (-1) with no threshold.
template <int E>
__device__ __forceinline__ int replay_entries(ResultRegs<E> &R, int &frozen_b, float &tau_f, const int32_t *s_cl, const float *s_g,
                                              const float *s_d2, const int32_t *s_id, int np, int batch, uint32_t *mask_row,
                                              int64_t mask_words) {
    int total = 0;
    for (int i0 = 0; i0 < np; i0 += kWave) {
        // Four chunks at once where nothing in them beats the k-th distance (most of a long scan): they only
        // count, each entry against the threshold of its batch.
        if (i0 + 4 * kWave <= np) {
            float g4[4], d4[4];
            int c4[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) { g4[u] = s_g[i0 + u * kWave + R.lane]; d4[u] = s_d2[i0 + u * kWave + R.lane]; c4[u] = s_cl[i0 + u * kWave + R.lane]; }
            bool better = false, on[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int b4 = c4[u] < R.k ? -1 : (c4[u] - R.k) / batch;
                on[u] = b4 < 0 || g4[u] <= (b4 == frozen_b ? tau_f : R.t_d2);
                better = better || (on[u] && d4[u] <= R.t_d2);
            }
            if (!__any(better)) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    total += __popcll(__ballot(on[u]));
                    if (on[u] && mask_row) {
                        const int64_t wi = c4[u] >> 5;
                        if (wi < mask_words) atomicOr(&mask_row[wi], 1u << (c4[u] & 31));
                    }
                }
                i0 += 3 * kWave;
                continue;
            }
        }
        const int i = i0 + R.lane;
        bool pending = i < np;
        int cl = 0, b = 0x7fffffff;
        int32_t id = 0;
        float g = __builtin_inff(), d2 = 0.0f;
        if (pending) {
            cl = s_cl[i]; g = s_g[i]; d2 = s_d2[i]; id = s_id[i];
            b = cl < R.k ? -1 : (cl - R.k) / batch;
            if (b < 0) g = -__builtin_inff();
        }
        auto mark = [&](bool on) {
            total += __popcll(__ballot(on));
            if (on && mask_row) {
                const int64_t wi = cl >> 5;
                if (wi < mask_words) atomicOr(&mask_row[wi], 1u << (cl & 31));
            }
        };
        for (;;) {
            // (see replay_batches: survivors that do not beat the k-th distance are taken all at once)
            pending = pending && g <= (b == frozen_b ? tau_f : R.t_d2);
            const unsigned long long mi = __ballot(pending && R.enters(d2, id));
            int fb = 0x7fffffff;
            if (mi != 0) fb = __builtin_amdgcn_readlane(b, __ffsll((long long)mi) - 1);
            const bool plain = pending && b < fb;
            mark(plain);
            pending = pending && !plain;
            if (mi == 0) break;
            if (fb != frozen_b) { frozen_b = fb; tau_f = R.t_d2; }
            const bool sel = pending && b == fb;
            mark(sel);
            R.insert_pending(sel, d2, id);
            pending = pending && !sel;
        }
    }
    return total;
}

// The batch rule where most entries only count: R changes with those alone whose exact distance was taken (`order`: their
// numbers in scan order), so one wave goes through these and writes down after which batch the k-th distance
// became what; every other entry is then held against the threshold of its batch by whoever comes along
// (threshold_of).  The state of a batch that the next call goes on with is kept in frozen_b and tau_f.
struct TauSteps {
    float tau;             // the k-th distance before the first step ...
    int32_t frozen_b;      // ... but for this batch
    float frozen_tau;
    int32_t count;
};
template <int E>
__device__ __forceinline__ void replay_measured(ResultRegs<E> &R, int &frozen_b, float &tau_f, const int32_t *s_cl, const float *s_g,
                                                const float *s_d2, const int32_t *s_id, const uint16_t *order, int n, int batch,
                                                TauSteps *info, unsigned long long *steps) {
    TauSteps out{R.t_d2, frozen_b, tau_f, 0};
    int last_b = -2;
    for (int i0 = 0; i0 < n; i0 += kWave) {
        bool pending = i0 + R.lane < n;
        const int i = pending ? order[i0 + R.lane] : 0;
        int b = 0x7fffffff;
        float g = __builtin_inff();
        unsigned long long key = ~0ull;
        if (pending) {
            const int cl = s_cl[i];
            g = s_g[i]; key = R.key_of(s_d2[i], s_id[i]);
            b = cl < R.k ? -1 : (cl - R.k) / batch;
            if (b < 0) g = -__builtin_inff();
        }
        // (who does not beat the k-th distance now never will: it only falls)
        unsigned long long left = __ballot(pending && g <= (b == frozen_b ? tau_f : R.t_d2) && key < R.t);
        while (left) {
            const int xb = __builtin_amdgcn_readlane(b, __ffsll((long long)left) - 1);
            if (xb != frozen_b) { frozen_b = xb; tau_f = R.t_d2; }
            // (a batch's entries together: they have one threshold, and only what it leaves counts)
            const bool here = b == xb;
            if (R.insert_keys(here && g <= tau_f, key)) {
                if (xb != last_b) { last_b = xb; ++out.count; }
                if (R.lane == 0) steps[out.count - 1] = ((unsigned long long)(uint32_t)xb << 32) | __float_as_uint(R.t_d2);
            }
            left &= __ballot(!here && key < R.t);
        }
    }
    if (R.lane == 0) *info = out;
}
// The threshold of batch b: what the last step before it left.
__device__ __forceinline__ float threshold_of(int b, const TauSteps &info, const unsigned long long *steps) {
    int lo = 0, hi = info.count;          // steps of batches before b
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if ((int)(steps[mid] >> 32) < b) lo = mid + 1; else hi = mid;
    }
    return lo > 0 ? __uint_as_float((uint32_t)steps[lo - 1]) : b == info.frozen_b ? info.frozen_tau : info.tau;
}

// Ascending bitonic sort of n keys in LDS (n a power of two) by all threads.  Ends with a barrier.
__device__ __forceinline__ void sort_keys(unsigned long long *key, int n) {
    for (int size = 2; size <= n; size <<= 1)
        for (int j = size >> 1; j > 0; j >>= 1) {
            for (int i = threadIdx.x; i < n / 2; i += blockDim.x) {
                const int x = ((i & ~(j - 1)) << 1) | (i & (j - 1)), y = x | j;
                const unsigned long long p = key[x], q = key[y];
                if ((p > q) == ((x & size) == 0)) { key[x] = q; key[y] = p; }
            }
            sync_block();
        }
}

}  // namespace trim
