// The kNN search of few queries (Section 4.2), in two kernels.
//
// search_kernel gives a query one workgroup, and a launch of few queries leaves most of the chip idle while each
// workgroup goes through its chain of dependent steps: one query over 32,000 candidates takes it
// 60 us, whatever the other 255 CUs do.  Here
//
//   bound_kernel   many workgroups per query, each with the query's table: the bounds of ALL candidates, by
//                  the rule, and (where a first batch is small) the exact distances of the seed and the first batch
//   settle_kernel  one workgroup per query: the seed, the first batch, then whoever is not above the
//                  threshold, measured and replayed batch by batch
//
// Over long rows, whose bounds leave thousands to be measured, that is a workgroup's work no longer: settle_kernel ends with the first
// batch, and then, pass by pass,
//
//   few_rows_kernel  many workgroups per query: the exact distances of those that the threshold leaves
//   settle_kernel    replays them
//
// No candidate is abandoned early and no list is passed over: with CUs to spare the lookups cost less than the chain
// of thresholds they would have to wait for.  Bound by latency: launches, the table, the measured rows.
#pragma once

#include "trim_passes.h"
#include "trim_steps.h"

namespace trim {

template <int VEC, bool FS>
// (six waves per SIMD: with 89 registers in place of 80 two workgroups fit a CU, and a grid of little more than two per CU takes
// half as long again)
__global__ __launch_bounds__(kBoundThreads) __attribute__((amdgpu_waves_per_eu(6))) void bound_kernel(const FewArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    float *tab = reinterpret_cast<float *>(smem);
    float *q_lds = reinterpret_cast<float *>(smem + a.off_q);
    int *segp = reinterpret_cast<int *>(smem + a.off_segp), *segd = reinterpret_cast<int *>(smem + a.off_segd);
    const int tid = threadIdx.x, split = blockIdx.x, nsplit = gridDim.x;
    const int64_t slot = blockIdx.y;
    const int64_t q = a.order ? a.order[slot] : slot;
    if (q < 0 || q >= a.nq) return;
    for (int t = tid; t < a.d; t += kBoundThreads) q_lds[t] = a.queries[(size_t)q * a.d + t];
    segment_table(a.list_offsets, a.probes, a.nlist, a.nseg, a.n, a.max_cand, q, segp, segd);
    const int total = segp[a.nseg > 0 ? a.nseg : 1];
    if (split == 0 && tid == 0) {
        a.totals[slot] = total;
        if (a.n_scanned) a.n_scanned[q] = total;
    }
    // exact distances of this workgroup's share of the seed and the first batch, four rows per half wave
    if (a.d2) {
        const int fb = total < a.k + a.batch ? total : a.k + a.batch;
        const int f0 = (int)((int64_t)fb * split / nsplit), f1 = (int)((int64_t)fb * (split + 1) / nsplit);
        const int half = tid >> 5, lane32 = tid & 31;
        float *out = a.d2 + (size_t)slot * (a.k + a.batch);
        for (int c = f0 + half * 4; c < f1; c += kBoundThreads / 32 * 4) {
            const float *rows[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                rows[u] = a.base + (size_t)segment_position(c + u < f1 ? c + u : c, segp, segd, a.nseg) * a.d;
            const float v = exact_d2_half_x4<true>(rows[0], rows[1], rows[2], rows[3], q_lds, a.d, lane32);
            const int mine = c + half_reduce_x4_row(lane32);
            if (half_reduce_x4_writer(lane32) && mine < f1) out[mine] = v;
        }
    }
    const int chunk = ((total + nsplit - 1) / nsplit + 63) & ~63;
    const int64_t cb = (int64_t)split * chunk;
    if (cb >= total) return;
    const int c0 = (int)cb, c1 = c0 + chunk < total ? c0 + chunk : total;
    float *row_g = a.g + (size_t)slot * a.stride;
    for (int ph = 0; ph < a.P; ++ph) {
        if (ph > 0) sync_block();
        if (a.lut) {
            const float4 *src = reinterpret_cast<const float4 *>(a.lut + ((size_t)q * a.M + ph * a.Mp) * kByteEntries<FS>);
            float4 *dst = reinterpret_cast<float4 *>(tab);
            for (int e = tid; e < a.Mp * (kByteEntries<FS> / 4); e += kBoundThreads) dst[e] = src[e];
        } else {
            build_table_rows<FS>(tab, q_lds, a.codebooks, a.dsub, ph * a.Mp, a.Mp);
        }
        sync_block();
        const bool last = ph == a.P - 1;
        // (a wave has 64 candidates that begin at a multiple of 64)
        for (int cw = c0 + (tid & ~63); cw < c1; cw += kBoundThreads) {
            const bool on = cw + (tid & 63) < c1;
            const int c = on ? cw + (tid & 63) : c1 - 1;
            const int pos = segment_position(c, segp, segd, a.nseg);
            const uint8_t *code = a.codes + (size_t)pos * a.M + ph * a.Mp;
            const float b = last ? a.dlx[pos] : 0.0f;
            float sum = ph > 0 ? row_g[c] : 0.0f;
            constexpr int kAhead = 2;
            for (int j = 0; j < a.Mp; j += kAhead * 4 * VEC) {
                uint32_t w[kAhead][VEC];
#pragma unroll
                for (int i = 0; i < kAhead; ++i)
                    if (j + i * 4 * VEC < a.Mp) load_codes<VEC>(w[i], code + j + i * 4 * VEC);
#pragma unroll
                for (int i = 0; i < kAhead; ++i)
                    if (j + i * 4 * VEC < a.Mp)
                        sum = gather_add<VEC, false, FS>(sum, (j + i * 4 * VEC) * kByteRow<FS>, w[i], __builtin_inff());
            }
            const float g = last ? plb_from_s(sum, b, a.two_gamma) : sum;
            if (on) row_g[c] = g;
            if (last) {
                float m = g;                          // (what is no number passes no threshold)
                m = __builtin_fminf(m, lane_xor<1>(m));
                m = __builtin_fminf(m, lane_xor<2>(m));
                m = __builtin_fminf(m, lane_xor<4>(m));
                m = __builtin_fminf(m, lane_xor<8>(m));
                m = __builtin_fminf(m, lane_xor<16>(m));
                m = __builtin_fminf(m, __shfl_xor(m, 32));
                if ((tid & 63) == 0) a.least[(size_t)slot * ((a.stride + 63) / 64) + (cw >> 6)] = m;
            }
        }
    }
}

// One workgroup per query.  R after the first batch is its k least distances: a histogram of the distances' bit
// patterns leaves little more than k of them to sort.  Then stretches of candidates, each about as long as what
// has been seen (4,096 or 16,384; half of that with wide R), listed against the threshold at their start, measured, and replayed
// by the first wave; a stretch whose bounds' least (one of every 64, from bound_kernel) is above the threshold is not looked
// at.  Bound by latency: bounds of 84,000 candidates read stretch by stretch, first-batch bounds read one after the other and a
// sort across the lanes took 46,000 of a single query's 59,000 clocks (25.2 us; now 10.6).
// PART: 0 all of it; 1 the seed and the first batch; 2 a pass after that, measured already.
template <int E, int PART>
__global__ __launch_bounds__(settle_threads(E)) void settle_kernel(const FewArgs a) {
    constexpr int T = settle_threads(E);
    extern __shared__ __align__(16) unsigned char smem[];
    float *q_lds = reinterpret_cast<float *>(smem + a.off_q);
    int *segp = reinterpret_cast<int *>(smem + a.off_segp), *segd = reinterpret_cast<int *>(smem + a.off_segd);
    float *rd2 = reinterpret_cast<float *>(smem + a.off_rd2);
    int32_t *rid = reinterpret_cast<int32_t *>(smem + a.off_rid);
    float *f_d2 = reinterpret_cast<float *>(smem + a.off_fd2);                              // [k + batch]
    unsigned long long *s_key = reinterpret_cast<unsigned long long *>(smem + a.off_key);   // [kSettleFirst]
    uint16_t *s_todo = reinterpret_cast<uint16_t *>(smem + a.off_todo);                     // [kSettleFirst]
    // (stretches; over the keys)
    int32_t *s_cl = reinterpret_cast<int32_t *>(smem + a.off_key), *s_id = s_cl + kSettleList;
    float *s_g = reinterpret_cast<float *>(s_id + kSettleList), *s_d2 = s_g + kSettleList;
    __shared__ TauSteps s_steps;
    __shared__ uint32_t s_bit[kSettleList / 32];
    unsigned long long *s_step = reinterpret_cast<unsigned long long *>(smem + a.off_fd2);  // [kSettleList] (passes; over the distances)
    static_assert(kSettleList / 32 == kWave && kSettleList * 8 <= kSettleFirst * 4, "a word of the measured ones per lane; room for the steps");
    __shared__ int hist[256], part[T / kWave];
    __shared__ uint32_t s_most, s_least;
    __shared__ int s_n, s_count, s_frozen;
    __shared__ int s_nk;          // (the sorted ones are not counted in s_n: it is read while they already are)
    __shared__ float s_tau, s_tau_f;
    __shared__ uint32_t s_ahead;  // of the T / 64 stretches looked at: those that have something to list
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t slot = blockIdx.x;
    const int64_t q = a.order ? a.order[slot] : slot;
    if (q < 0 || q >= a.nq) return;
    const float *row_g = a.g + (size_t)slot * a.stride;
    float *const r_d2 = PART ? a.r_d2 + (size_t)slot * a.r_stride : nullptr;
    int32_t *const r_id = PART ? a.r_id + (size_t)slot * a.r_stride : nullptr;
    uint32_t *mask_row = a.mask ? a.mask + (size_t)q * a.mask_words : nullptr;
    const int total = a.totals[slot];
    const int ns = total < a.k ? total : a.k, fb = total < a.k + a.batch ? total : a.k + a.batch;
    const int from = PART == 2 ? a.lo : fb, until = PART == 2 && a.hi < total ? a.hi : total;      // (of the rest)
    if (PART == 2 && from >= until) return;
    // exact distances of n candidates at(i), four rows per half wave; put(i, d2, storage position)
    auto measure = [&](int n, auto at, auto put) {
        const int half = tid >> 5, lane32 = tid & 31;
        for (int i = half * 4; i < n; i += T / 32 * 4) {
            int pos[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) pos[u] = segment_position(at(i + u < n ? i + u : i), segp, segd, a.nseg);
            const float v = exact_d2_half_x4<true>(a.base + (size_t)pos[0] * a.d, a.base + (size_t)pos[1] * a.d,
                                                   a.base + (size_t)pos[2] * a.d, a.base + (size_t)pos[3] * a.d, q_lds, a.d, lane32);
            const int r = half_reduce_x4_row(lane32);
            const int p = r == 0 ? pos[0] : r == 1 ? pos[1] : r == 2 ? pos[2] : pos[3];
            if (half_reduce_x4_writer(lane32) && i + r < n) put(i + r, v, p);
        }
        sync_block();
    };
    if constexpr (PART == 2) {
        for (int i = tid; i < kWave * E; i += T) { rd2[i] = r_d2[i]; rid[i] = r_id[i]; }
        if (tid == 0) s_count = a.r_n[slot];
        segment_table(a.list_offsets, a.probes, a.nlist, a.nseg, a.n, a.max_cand, q, segp, segd);
    } else {
    // the first batch's bounds and distances on their way (what lies beyond it is not used)
    constexpr int kPre = 2;
    float pre_g[kPre], pre_d2[kPre] = {};
#pragma unroll
    for (int u = 0; u < kPre; ++u) {
        pre_g[u] = row_g[tid + u * T < a.stride ? tid + u * T : 0];
        if (a.d2) pre_d2[u] = a.d2[(size_t)slot * (a.k + a.batch) + (tid + u * T < a.k + a.batch ? tid + u * T : 0)];
    }
    for (int t = tid; t < a.d; t += T) q_lds[t] = a.queries[(size_t)q * a.d + t];
    if (tid < 256) hist[tid] = 0;
    if (tid == 0) { s_most = 0; s_least = ~0u; s_n = 0; s_nk = 0; s_count = 0; }
    segment_table(a.list_offsets, a.probes, a.nlist, a.nseg, a.n, a.max_cand, q, segp, segd);
    // ---- the seed: its largest distance is the first batch's threshold ----
    if (a.d2) {
#pragma unroll
        for (int u = 0; u < kPre; ++u)
            if (tid + u * T < fb) f_d2[tid + u * T] = pre_d2[u];
        for (int i = tid + kPre * T; i < fb; i += T) f_d2[i] = a.d2[(size_t)slot * (a.k + a.batch) + i];
        sync_block();
    } else {
        measure(ns, [&](int i) { return i; }, [&](int i, float v, int) { f_d2[i] = v; });
    }
    uint32_t most = 0;
    for (int i = tid; i < ns; i += T) most = max(most, __float_as_uint(f_d2[i]));
    wave_max(&s_most, most);
    sync_block();
    // (a distance that is no number is never in R: then R is not full yet)
    const bool full = ns == a.k && s_most <= 0x7f800000u;
    const float tau1 = full ? __uint_as_float(s_most) : __builtin_inff();
    // ---- the first batch ----
    {
        int mine = 0;
        // (one atomic a wave: nearly all of them are in)
        auto first = [&](int i, float g) {
            const bool on = i < fb && (i < ns || g <= tau1);
            mine += on;
            if (on && mask_row && (i >> 5) < a.mask_words) atomicOr(&mask_row[i >> 5], 1u << (i & 31));
            const unsigned long long put = __ballot(on && (a.d2 != nullptr || i >= ns));
            if (put == 0) return;
            int to = 0;
            if (lane == 0) to = atomicAdd(&s_n, __popcll(put));
            to = __builtin_amdgcn_readfirstlane(to) + __popcll(put & ((1ull << lane) - 1ull));
            if ((put >> lane) & 1ull) s_todo[to] = (uint16_t)i;
        };
#pragma unroll
        for (int u = 0; u < kPre; ++u) first(tid + u * T, pre_g[u]);
        for (int i0 = kPre * T; i0 < fb; i0 += T) first(i0 + tid, row_g[i0 + tid < fb ? i0 + tid : 0]);
        wave_add(&s_count, mine);
    }
    sync_block();
    int n = s_n;
    if (!a.d2) {
        measure(n, [&](int i) { return (int)s_todo[i]; }, [&](int i, float v, int) { f_d2[s_todo[i]] = v; });
        for (int i = tid; i < ns; i += T) s_todo[n + i] = (uint16_t)i;
        n += ns;
        sync_block();
    }
    // the k least distances by (distance, id)
    const uint32_t top = full ? __float_as_uint(tau1) : 0x7f800000u;    // (nothing above it can be among them)
    uint32_t least = ~0u, cut = top;
    int nk = 0;
    for (int i = tid; i < n; i += T) least = min(least, __float_as_uint(f_d2[s_todo[i]]));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) least = min(least, (uint32_t)__shfl_xor((int)least, off));
    if (lane == 0) atomicMin(&s_least, least);
    sync_block();
    least = s_least;
    if (full) {                                  // (else all of them are wanted, as far as they go)
        const uint32_t span = top - least;       // least <= top: the seed is among them
        const int shift = span < 256 ? 0 : 24 - __clz((int)span);
        for (int i = tid; i < n; i += T) {
            const uint32_t key = __float_as_uint(f_d2[s_todo[i]]);
            if (key <= top) atomicAdd(&hist[(key - least) >> shift], 1);
        }
        sync_block();
        if (wave == 0) {
            int h[4], sum = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) { h[u] = hist[4 * lane + u]; sum += h[u]; }
            int incl = sum;
#pragma unroll
            for (int off = 1; off < kWave; off <<= 1) {
                const int v = __shfl_up(incl, off);
                if (lane >= off) incl += v;
            }
            int before = incl - sum;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (before < a.k && before + h[u] >= a.k) s_least = least + (((uint32_t)(4 * lane + u + 1)) << shift) - 1u;
                before += h[u];
            }
        }
        sync_block();
        cut = s_least < top ? s_least : top;
    }
    for (int i = tid; i < n; i += T) {
        const int c = s_todo[i];
        const uint32_t key = __float_as_uint(f_d2[c]);
        if (key <= cut) {
            const int pos = segment_position(c, segp, segd, a.nseg);
            const int32_t id = a.ids ? a.ids[pos] : pos;
            s_key[atomicAdd(&s_nk, 1)] = ((unsigned long long)key << 32) | ((uint32_t)id ^ 0x80000000u);   // (ids order as signed)
        }
    }
    sync_block();
    nk = s_nk;
    const int have = nk < a.k ? nk : a.k;
    if (nk <= 256) {                             // (a rank each; two entries may be one and the same)
        if (tid < nk) {
            const unsigned long long key = s_key[tid];
            int rank = 0;
#pragma unroll 8
            for (int j = 0; j < nk; ++j) {
                const unsigned long long o = s_key[j];
                rank += o < key || (o == key && j < tid);
            }
            if (rank < have) {
                rd2[rank] = __uint_as_float((uint32_t)(key >> 32));
                rid[rank] = (int32_t)((uint32_t)key ^ 0x80000000u);
            }
        }
        for (int i = have + tid; i < kWave * E; i += T) { rd2[i] = __builtin_inff(); rid[i] = kEmptyId; }
    } else {
        int size = 1;
        while (size < nk) size <<= 1;
        for (int i = nk + tid; i < size; i += T) s_key[i] = ~0ull;
        sync_block();
        sort_keys(s_key, size);
        for (int i = tid; i < kWave * E; i += T) {
            rd2[i] = i < have ? __uint_as_float((uint32_t)(s_key[i] >> 32)) : __builtin_inff();
            rid[i] = i < have ? (int32_t)((uint32_t)s_key[i] ^ 0x80000000u) : kEmptyId;
        }
    }
    sync_block();
    }
    ResultRegs<E> R;
    int frozen_b = -2, survivors = s_count, counted = 0;       // (counted: this thread's)
    float tau_f = 0.0f;
    if (wave == 0) {
        R.load(rd2, rid, a.k, lane);
        if (lane == 0) { s_tau = R.t_d2; s_frozen = -2; s_tau_f = 0.0f; }
    }
    sync_block();
    // ---- the rest ----
    if constexpr (PART != 1) {
    const float *least_of = a.least + (size_t)slot * ((a.stride + 63) / 64);
    int looked = 0;                              // up to here s_ahead is known
    uint32_t ahead = 0;
    for (int w0 = from; w0 < until;) {
        const int V = a.nseg == 0 && w0 < 16384 ? 4 : 16, base = w0 & ~3;
        const int w1 = until - base < V * T ? until : base + V * T;
        if (V == 16) {
            // the next stretches, a wave each (thresholds only fall: who is above this one stays out)
            if (w0 >= looked) {
                sync_block();                 // (the last look has been read)
                if (tid == 0) s_ahead = 0;
                sync_block();
                const float tau = __builtin_fmaxf(s_tau, s_tau_f);
                const int64_t first = (int64_t)base + (int64_t)wave * 16 * T, to = first + 16 * T < until ? first + 16 * T : until;
                constexpr int kLeast = 16 * T / 64 / kWave + 1;
                const int g0 = (int)(first >> 6), g1 = (int)((to - 1) >> 6);
                float v[kLeast];
                bool any = false;
#pragma unroll
                for (int u = 0; u < kLeast; ++u) v[u] = least_of[first < to ? min(g0 + u * kWave + lane, g1) : 0];
#pragma unroll
                for (int u = 0; u < kLeast; ++u) any |= v[u] <= tau;
                any &= first < to;
                if (__any(any) && lane == 0) atomicOr(&s_ahead, 1u << wave);
                sync_block();
                ahead = s_ahead;
                looked = base + 16 * T * (T / kWave) < until ? base + 16 * T * (T / kWave) : until;
            }
            const bool some = ahead & 1u;
            ahead >>= 1;
            if (!some) { w0 = w1; continue; }
        }
        // (the batch that the last stretch ended in keeps the threshold that it began with)
        const float tau = s_tau, tau_b = __builtin_fmaxf(tau, s_tau_f);
        const int end_b = s_frozen >= 0 ? a.k + (s_frozen + 1) * a.batch : 0;
        // (rows are allocated to a multiple of 16 floats)
        float g[16];
        uint32_t m = 0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int c = base + tid * V + 4 * v;
            if (4 * v < V && c < w1) {
                const float4 x = *reinterpret_cast<const float4 *>(row_g + c);
                g[4 * v] = x.x; g[4 * v + 1] = x.y; g[4 * v + 2] = x.z; g[4 * v + 3] = x.w;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (g[4 * v + e] <= (c + e < end_b ? tau_b : tau) && c + e >= w0 && c + e < w1) m |= 1u << (4 * v + e);
            }
        }
        const int cnt = __popc(m);
        int incl = cnt;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int v = __shfl_up(incl, off);
            if (lane >= off) incl += v;
        }
        if (lane == 63) part[wave] = incl;
        sync_block();
        int before = incl - cnt, all = 0;
#pragma unroll
        for (int v = 0; v < T / kWave; ++v) {
            const int p = part[v];
            if (v < wave) before += p;
            all += p;
        }
        for (int e0 = 0; e0 < all; e0 += kSettleList) {
            const int np = all - e0 < kSettleList ? all - e0 : kSettleList;
            int at = before - e0;
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if ((m >> v) & 1u) {
                    if (at >= 0 && at < np) { s_cl[at] = base + tid * V + v; s_g[at] = g[v]; }
                    ++at;
                }
            if (tid == 0) s_n = 0;
            sync_block();
            if constexpr (PART == 2) {
                // All that the pass's first threshold leaves have been measured: the first wave goes through those that can enter R and
                // leaves the thresholds by batch, all threads count the others by these (as in replay_kernel).  (All by the first wave: one
                // query over 500,000 x 768, 20 of 700 lists, 166 -> 103 us, 16 381 -> 311; k = 100 244 -> 145, 457 -> 347.)
                if (tid < kSettleList / 32) s_bit[tid] = 0;
                sync_block();
                const float now = s_tau;
                for (int i = tid; i < np; i += T) {
                    const int c = s_cl[i];
                    const float d2 = a.d2_all[(size_t)slot * a.stride + c];
                    if (!(d2 <= now)) continue;
                    const int pos = segment_position(c, segp, segd, a.nseg);
                    s_d2[i] = d2;
                    s_id[i] = a.ids ? a.ids[pos] : pos;
                    atomicOr(&s_bit[i >> 5], 1u << (i & 31));
                }
                sync_block();
                if (wave == 0) {
                    __builtin_amdgcn_s_setprio(3);       // (the workgroup waits for this wave)
                    uint32_t word = s_bit[lane];
                    const int ones = __popc(word);
                    int place = ones;
#pragma unroll
                    for (int off = 1; off < kWave; off <<= 1) {
                        const int v = __shfl_up(place, off);
                        if (lane >= off) place += v;
                    }
                    const int nt = __builtin_amdgcn_readlane(place, kWave - 1);
                    for (place -= ones; word; word &= word - 1) s_todo[place++] = (uint16_t)(lane * 32 + (__ffs((int)word) - 1));
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    replay_measured<E>(R, frozen_b, tau_f, s_cl, s_g, s_d2, s_id, s_todo, nt, a.batch, &s_steps, s_step);
                    if (lane == 0) { s_tau = R.t_d2; s_frozen = frozen_b; s_tau_f = tau_f; }
                    __builtin_amdgcn_s_setprio(0);
                }
                sync_block();
                const TauSteps steps = s_steps;
                for (int i = tid; i < np; i += T) {
                    const int c = s_cl[i];
                    if (s_g[i] <= threshold_of((c - a.k) / a.batch, steps, s_step)) {
                        ++counted;
                        if (mask_row && (c >> 5) < a.mask_words) atomicOr(&mask_row[c >> 5], 1u << (c & 31));
                    }
                }
                sync_block();
                continue;
            } else {
                // who is a survivor by now (a batch keeps the threshold that it began with) is measured
                const float now = s_tau, tf = s_tau_f;
                const int fz = s_frozen;
                for (int i = tid; i < np; i += T) {
                    const int c = s_cl[i], b = (c - a.k) / a.batch;
                    s_d2[i] = __builtin_inff();
                    s_id[i] = kEmptyId;
                    if (s_g[i] <= (b == fz ? tf : now)) s_todo[atomicAdd(&s_n, 1)] = (uint16_t)i;
                }
                sync_block();
                measure(s_n, [&](int i) { return s_cl[s_todo[i]]; },
                        [&](int i, float v, int pos) { s_d2[s_todo[i]] = v; s_id[s_todo[i]] = a.ids ? a.ids[pos] : pos; });
            }
            if (wave == 0) {
                survivors += replay_entries<E>(R, frozen_b, tau_f, s_cl, s_g, s_d2, s_id, np, a.batch, mask_row, a.mask_words);
                if (lane == 0) { s_tau = R.t_d2; s_frozen = frozen_b; s_tau_f = tau_f; }
            }
            sync_block();
        }
        sync_block();
        w0 = w1;
    }
    }
    if constexpr (PART == 2) {
        wave_add(&s_count, counted);
        sync_block();
        survivors = s_count;
    }
    if (wave == 0) {
        R.store(rd2, rid);
        if (lane == 0 && a.n_exact) a.n_exact[q] = survivors;
        if (PART && lane == 0) a.r_n[slot] = survivors;
    }
    sync_block();
    if constexpr (PART != 0)
        for (int i = tid; i < kWave * E; i += T) { r_d2[i] = rd2[i]; r_id[i] = rid[i]; }
    for (int i = tid; i < a.k; i += T) {
        const int32_t id = rid[i];
        a.out_ids[(size_t)q * a.k + i] = id == kEmptyId ? -1 : id;
        a.out_d2[(size_t)q * a.k + i] = rd2[i];
    }
}

// The exact distances of the candidates [lo, hi) whose bound does not exceed the k-th distance so far: all that can be survivors among them
// (the threshold only falls), and some more.  The candidates of a query are dealt out 64 at a time, since the near ones lie together; a
// wave lists its 64, all half waves measure.  Bound by the rows, which one workgroup reads at 0.15 TB/s: one query over 14,000 unit vectors of 768
// values, nearly all of them wanted, 978 us with settle_kernel alone, 103 so; 33 queries 1703, 483.
constexpr int kFewRowsThreads = 256;
__global__ __launch_bounds__(kFewRowsThreads) void few_rows_kernel(const FewArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    float *q_lds = reinterpret_cast<float *>(smem + a.off_q);
    int *segp = reinterpret_cast<int *>(smem + a.off_segp), *segd = reinterpret_cast<int *>(smem + a.off_segd);
    constexpr int kWaves = kFewRowsThreads / kWave, kHalves = 2 * kWaves;
    __shared__ int s_c[kWaves * kWave], s_n;
    const int tid = threadIdx.x, lane = tid & 63, half = tid >> 5, lane32 = tid & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t slot = blockIdx.y;
    const int64_t q = a.order ? a.order[slot] : slot;
    if (q < 0 || q >= a.nq) return;
    const int total = a.totals[slot], hi = a.hi < total ? a.hi : total;
    if (a.lo >= hi) return;
    const float tau = a.r_d2[(size_t)slot * a.r_stride + a.k - 1];
    const float *row_g = a.g + (size_t)slot * a.stride, *least = a.least + (size_t)slot * ((a.stride + 63) / 64);
    float *out = a.d2_all + (size_t)slot * a.stride;
    const int g0 = a.lo >> 6, g1 = ((hi - 1) >> 6) + 1, step = (int)gridDim.x;
    bool ready = false;
    for (int64_t b0 = g0 + (int)blockIdx.x; b0 < g1; b0 += (int64_t)kWave * step) {
        const int64_t mine = b0 + (int64_t)lane * step;
        unsigned long long left = __ballot(mine < g1 && least[mine < g1 ? mine : g0] <= tau);     // (the same in all waves)
        while (left) {
            if (!ready) {
                ready = true;
                for (int t = tid; t < a.d; t += kFewRowsThreads) q_lds[t] = a.queries[(size_t)q * a.d + t];
                segment_table(a.list_offsets, a.probes, a.nlist, a.nseg, a.n, a.max_cand, q, segp, segd);
            }
            int group = -1;                 // a wave each
            for (int w = 0; w < kWaves && left; ++w) {
                const int at = __ffsll((long long)left) - 1;
                left &= left - 1;
                if (w == wave) group = (int)(b0 + (int64_t)at * step);
            }
            if (tid == 0) s_n = 0;
            sync_block();
            if (group >= 0) {
                const int c = group * 64 + lane;
                const bool on = c >= a.lo && c < hi && row_g[c < hi ? c : a.lo] <= tau;
                const unsigned long long m = __ballot(on);
                int to = 0;
                if (lane == 0) to = atomicAdd(&s_n, __popcll(m));
                to = __builtin_amdgcn_readfirstlane(to);
                if (on) s_c[to + __popcll(m & ((1ull << lane) - 1ull))] = c;
            }
            sync_block();
            const int n = s_n;
            for (int i = half; i < n; i += 2 * kHalves) {
                const int c0 = s_c[i], c1 = s_c[i + kHalves < n ? i + kHalves : i];
                float d2[2];
                exact_d2_half_x2_deep<4>(a.base + (size_t)segment_position(c0, segp, segd, a.nseg) * a.d,
                                         a.base + (size_t)segment_position(c1, segp, segd, a.nseg) * a.d, q_lds, a.d, lane32, d2);
                if (lane32 == 0) { out[c0] = d2[0]; out[c1] = d2[1]; }
            }
            sync_block();
        }
    }
}

}  // namespace trim
