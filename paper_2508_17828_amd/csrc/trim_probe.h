// Probe selection of many queries (Section 6.1: IVFPQ with C' lists, nprobe probed) with the matrix cores in front of the
// exact distances.  The nprobe nearest lists come out in the order of their exact distances (ivf_probe_kernel,
// probe_distance_kernel measure every pair and are bound by the vector ALU); but only who may be among them has
// to be measured:
//
//   operands   queries and centroids as 16-bit operands, relative to the mean of a few centroids, scaled row by row by a power
//              of two, with the lengths of what is stored and what rounding moved
//   scores     S = |q' - c'|^2 by v_mfma_f32_32x32x16_f16; kept: t = sqrt(S - e), 4 bytes a pair
//   nearest    a wave per query: the true distance lies in t - m .. sqrt(t^2 + 2 e) + m, m = moved(q) + moved(c).  The nprobe'th
//              least of the upper ends (of 256 columns' least ones) bounds who can be among the nearest; these, some nprobe
//              and a few, are measured by the exact rule and ranked by (distance, number)
//
//   rest       who has more candidates than kPrbList (a query so far away that what rounding moved exceeds the spread of its
//              distances; rows that are no numbers; many lists in one place): all lists measured, eight of these queries
//              at a time, and selected as for few queries
//
// 10000 queries x 1024 lists of 128 values, 32 probes: 122 -> 71 us, of which nearest 38 (latency: the candidates' rows, eight
// at a time; a workgroup of 256 per query, with its barriers, took 110), scores 17, the two launches of rest 2 where there
// are none.  With 1 to 100 queries 10^5 away 80, with 1000 94, with all 223 (a wave that measured all lists of its query by itself and
// picked them one after the other: 175 to 187, 226, 537); 2500 x 1024 of 768, 64 probes: 72, with one far away 90 (367).
//
// e = (5 d + 128) 2^-24 (|q'|^2 + |c'|^2) bounds the binary32 sums of S and the exact rule's own roundings.  Rows out of the scaled
// range, and what is no number, have m = inf: always candidates, and nobody's bound.
#pragma once

#include "trim_gamma.h"

namespace trim {

// From where on (both sides measured, us, exact kernels / these; 8, 32, 64 probes): 4000 x 1024 lists of 128 values 45, 45, 48 / 38, 40,
// 46, 10000 x 1024 121, 122, 138 / 64, 71, 82, 10000 x 512 75, 76, 94 / 45, 51, 61; 1400 x 1024 of 768 67, 68, 70 / 42, 50, 64, 10000 x 1024
// of 768 457, 459, 470 / 109, 137, 186, 270 x 4096 of 1536 155, 154, 157 / 78, 101, 134.  Even at about 3,000,000 pairs: 3000 x 1024 of 128
// 36, 37, 39 / 34, 35, 41 (2600 x 1024 32, 33, 35 / 33, 34, 39), and where fewer queries leave a wave's chain of candidates in the open, at
// more: 1000 x 2600 35, 36, 38 / 41, 43, 47, 1000 x 4096 50, 51, 53 / 50, 52, 57, 1000 x 1024 of 1000 72, 73, 74 / 47, 59, 77.
// With more than an eighth of the lists probed most rows are measured anyway (10000 x 150 of 1536, 64 probes: 165 / 231).
inline bool probe_ranked_pays(int64_t nq, int d, int nlist, int nprobe) {
    const double pairs = (double)nq * nlist, values = pairs * d;
    return nprobe <= nlist / 8 && ((nq >= 1500 && pairs >= 2.5e6) || (nq >= 1000 && (pairs >= 4.5e6 || values >= 1e9)) ||
                                   (nq >= 100 && values >= 1.6e9));
}

constexpr int kPrbList = 256, kPrbCols = 256, kPrbRows = 32;
constexpr int kPrbLefts = 32, kPrbApart = 32;       // (one counter took 15 ns a query; words from one to the next: a cache line)
struct ProbeArgs {
    const float *queries, *cent;
    int64_t nq;                // queries of this launch
    int32_t d, nlist, nprobe;
    int32_t dpad, lpad;        // values per operand row (a multiple of 16), lists (of kPrbCols)
    int32_t list_groups;       // workgroups of the operands that have centroids
    _Float16 *q16, *c16;       // [block of 32 rows][dpad / 8][32][8]
    float4 *qpar, *cpar;       // 1 / scale, |.|^2, moved, unused
    float2 *cnm;               // of the lists once more: |.|^2, moved
    float *t;                  // [nq][lpad]
    uint32_t *left;            // the queries with more candidates than kPrbList, kPrbLefts lists of them (by q % kPrbLefts): counts, then entries
    int64_t left_pitch;
    int32_t *out;              // [nq][nprobe]
};

// One workgroup per eight rows, a half wave per row: the centroids, then the queries.
__global__ __launch_bounds__(256) void probe_operands_kernel(const ProbeArgs a) {
    typedef _Float16 h8 __attribute__((ext_vector_type(8)));
    extern __shared__ __align__(16) float s_mu[];      // [dpad]
    const int tid = threadIdx.x, part = tid & 31, d = a.d, np = a.dpad >> 3;
    const bool list = (int)blockIdx.x < a.list_groups;
    const int64_t row = (int64_t)(list ? blockIdx.x : blockIdx.x - a.list_groups) * kGrRows + (tid >> 5);
    if (blockIdx.x == 0 && tid < kPrbLefts) a.left[tid * kPrbApart] = 0;
    for (int t = tid; t < a.dpad; t += 256) {
        float v[8], sum = 0.0f;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = a.cent[(size_t)((int64_t)i * a.nlist >> 3) * d + (t < d ? t : 0)];
#pragma unroll
        for (int i = 0; i < 8; ++i) sum += __builtin_fabsf(v[i]) < 1e18f ? v[i] : 0.0f;
        s_mu[t] = t < d ? sum * 0.125f : 0.0f;
    }
    sync_block();
    const int64_t rows = list ? a.nlist : a.nq;
    const float *x = (list ? a.cent : a.queries) + (size_t)(row < rows ? row : rows - 1) * d;
    auto values = [&](int p, float (&v)[8]) {          // (d is a multiple of four)
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const int k = 8 * p + 4 * g;
            const float4 f = *reinterpret_cast<const float4 *>(x + (k < d ? k : 0));
            const float w[4] = {f.x, f.y, f.z, f.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * g + e] = k < d ? w[e] - s_mu[k + e] : 0.0f;
        }
    };
    float most = 0.0f, bad = 0.0f;                     // (a NaN is passed over by the maximum: the sum keeps it)
    for (int p = part; p < np; p += 32) {
        float v[8];
        values(p, v);
#pragma unroll
        for (int e = 0; e < 8; ++e) { most = __builtin_fmaxf(most, __builtin_fabsf(v[e])); bad += v[e] - v[e]; }
    }
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) { most = __builtin_fmaxf(most, __shfl_xor(most, off)); bad += __shfl_xor(bad, off); }
    const float scale = gamma_scale(most);
    const bool usable = bad == 0.0f && scale > 0.0f;
    float n2 = 0.0f, moved = 0.0f;
    for (int p = part; p < np; p += 32) {
        float v[8];
        values(p, v);
        h8 h;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float f = usable ? v[e] * scale : 0.0f;
            h[e] = (_Float16)f;
            const float r = (float)h[e], m = f - r;
            n2 = __builtin_fmaf(r, r, n2);
            moved = __builtin_fmaf(m, m, moved);
        }
        reinterpret_cast<h8 *>(list ? a.c16 : a.q16)[((size_t)(row >> 5) * np + p) * 32 + (row & 31)] = h;
    }
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) { n2 += __shfl_xor(n2, off); moved += __shfl_xor(moved, off); }
    if (part != 0) return;
    const float inv = usable ? 1.0f / scale : 0.0f;
    // (rounding, the subtraction of the mean, 16-bit subnormals that may count as zero)
    const float m = usable ? (sqrt_rn(moved) * 1.001f + sqrt_rn(n2) * (1.0f / 4194304.0f) + sqrt_rn((float)d) * (1.0f / 16384.0f)) * inv : __builtin_inff();
    (list ? a.cpar : a.qpar)[row] = make_float4(inv, n2 * inv * inv, m, 0.0f);
    if (list) a.cnm[row] = make_float2(n2 * inv * inv, m);
}

// A wave: 32 queries x 64 lists.
__global__ __launch_bounds__(256) void probe_scores_kernel(const ProbeArgs a) {
    typedef _Float16 h8 __attribute__((ext_vector_type(8)));
    typedef float v16f __attribute__((ext_vector_type(16)));
    __shared__ float4 s_q[kPrbRows];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 31, half = lane >> 5;
    const int l0 = blockIdx.x * kPrbCols + wave * 64, np = a.dpad >> 3;
    const int64_t qb = blockIdx.y;
    if (threadIdx.x < kPrbRows) s_q[threadIdx.x] = a.qpar[qb * 32 + threadIdx.x];
    const h8 *qp = reinterpret_cast<const h8 *>(a.q16) + (size_t)qb * np * 32 + lane;
    const h8 *cp = reinterpret_cast<const h8 *>(a.c16) + (size_t)(l0 >> 5) * np * 32 + lane;
    v16f acc[2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[u][i] = 0.0f;
    // three steps of 16 values on their way while one is used
    h8 f[4][3];
    const int steps = np >> 1;
    auto load = [&](int step, h8 (&to)[3]) {
        const size_t k = (size_t)(step < steps ? step : steps - 1) * 64;
        to[0] = qp[k];
        to[1] = cp[k];
        to[2] = cp[(size_t)np * 32 + k];
    };
    load(0, f[0]);
    load(1, f[1]);
    load(2, f[2]);
    for (int s = 0; s < steps; s += 4) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            load(s + i + 3, f[(i + 3) & 3]);
            if (s + i < steps) {
#pragma unroll
                for (int u = 0; u < 2; ++u) acc[u] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[i][0], f[i][1 + u], acc[u], 0, 0, 0);
            }
        }
    }
    sync_block();
    const float e2 = (5.0f * a.d + 128.0f) * (1.0f / 16777216.0f);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int l = l0 + u * 32 + col;
        const float4 c = a.cpar[l];
        const float inv = -2.0f * c.x;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int r = 8 * (i >> 2) + 4 * half + (i & 3);
            const int64_t q = qb * 32 + r;
            const float4 p = s_q[r];
            const float sum = p.y + c.y, low = __builtin_fmaf(acc[u][i], p.x * inv, sum) - e2 * sum;
            if (q < a.nq) a.t[(size_t)q * a.lpad + l] = low > 0.0f ? __builtin_amdgcn_sqrtf(low) * 0.9999998f : 0.0f;
        }
    }
}

// One wave per query.  Lists are 256 columns (lane, 0..3); what a lane's own columns hold stays in its registers.
template <bool ONE_STEP>
__global__ __launch_bounds__(kWave) void probe_nearest_kernel(const ProbeArgs a) {
    extern __shared__ __align__(16) float q_lds[];     // [d]
    __shared__ unsigned long long s_key[kPrbList];
    __shared__ uint16_t s_list[kPrbList];
    const int lane = threadIdx.x, lane32 = lane & 31;
    const int64_t q = blockIdx.x;
    const float *x = a.queries + (size_t)q * a.d;
    const float *row = a.t + (size_t)q * a.lpad;
    const float4 qp = a.qpar[q];
    const float inf = __builtin_inff(), e2 = 2.0f * (5.0f * a.d + 128.0f) * (1.0f / 16777216.0f) * 1.0001f;
    for (int t = lane; t < a.d >> 2; t += kWave) reinterpret_cast<float4 *>(q_lds)[t] = reinterpret_cast<const float4 *>(x)[t];
    uint32_t least[4] = {0x7f800000u, 0x7f800000u, 0x7f800000u, 0x7f800000u};
#pragma unroll 4
    for (int l = 4 * lane; l < a.lpad; l += 4 * kWave) {
        const float4 t4 = *reinterpret_cast<const float4 *>(row + l);
        const float t[4] = {t4.x, t4.y, t4.z, t4.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float2 c = a.cnm[l + e];
            const float up = __builtin_amdgcn_sqrtf(__builtin_fmaf(t[e], t[e] * 1.000001f, e2 * (qp.y + c.x))) * 1.000001f + (qp.z + c.y) * 1.000001f;
            // (what is no number bounds nobody, and neither do the lists beyond the last)
            const uint32_t key = l + e < a.nlist ? __float_as_uint(__builtin_fminf(up, inf)) : 0x7f800000u;
            least[e] = key < least[e] ? key : least[e];
        }
    }
    // the nprobe'th least of the columns, to 12 bits of its fraction and from above
    uint32_t cut = 0;
#pragma unroll 4
    for (int bit = 30; bit > 10; --bit) {
        const uint32_t at = cut | 1u << bit;
        int below = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) below += __popcll(__ballot(least[e] < at));
        if (below < a.nprobe) cut = at;
    }
    cut |= 0x7ffu;
    const float bound = cut < 0x7f800000u ? __uint_as_float(cut) : inf;
    int n = 0;
    for (int l = 4 * lane; l < a.lpad; l += 4 * kWave) {   // (every lane takes part in the ballots: lpad is a multiple of 256)
        const float4 t4 = *reinterpret_cast<const float4 *>(row + l);
        const float t[4] = {t4.x, t4.y, t4.z, t4.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float low = t[e] - (qp.z + a.cnm[l + e].y) * 1.000001f;
            const bool take = l + e < a.nlist && !(low > bound);
            const unsigned long long m = __ballot(take);
            const int to = n + __popcll(m & ((1ull << lane) - 1ull));
            if (take && to < kPrbList) s_list[to] = (uint16_t)(l + e);
            n += __popcll(m);
        }
    }
    sync_block();
    if (n > kPrbList) {                                // (probe_rest_kernel)
        if (lane == 0) {
            const int list = (int)(q % kPrbLefts);
            a.left[kPrbLefts * kPrbApart + list * a.left_pitch + atomicAdd(&a.left[list * kPrbApart], 1u)] = (uint32_t)q;
        }
        return;
    }
    // the exact distances, four rows to a half wave
    for (int i0 = (lane >> 5) * 4; i0 < n; i0 += 8) {
        int l[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) l[i] = s_list[i0 + i < n ? i0 + i : i0];
        const float dist = exact_d2_half_x4<!ONE_STEP, ONE_STEP>(a.cent + (size_t)l[0] * a.d, a.cent + (size_t)l[1] * a.d, a.cent + (size_t)l[2] * a.d,
                                                                 a.cent + (size_t)l[3] * a.d, q_lds, a.d, lane32);
        const int i = half_reduce_x4_row(lane32), mine = i == 0 ? l[0] : i == 1 ? l[1] : i == 2 ? l[2] : l[3];
        if (half_reduce_x4_writer(lane32) && i0 + i < n) s_key[i0 + i] = ((unsigned long long)__float_as_uint(dist) << 32) | (uint32_t)mine;
    }
    sync_block();
    int32_t *out = a.out + (size_t)q * a.nprobe;
    for (int i = lane; i < n; i += kWave) {
        const unsigned long long k = s_key[i];
        int rank = 0;
#pragma unroll 8
        for (int j = 0; j < n; ++j) rank += s_key[j] < k;
        if (rank < a.nprobe) out[rank] = (int32_t)(k & 0xffffffffu);
    }
}

// The queries with more candidates than nearest takes: all lists measured, 32 lists by eight of these queries a workgroup and turn, the
// distances kept where the scores were; then a wave each selects as probe_select_kernel does.  Both end with the list of them.  (One launch,
// the workgroup with the last turn of eight queries selecting: 0.3 us less where there are none, but its fences: 548 us in place of 91 for
// 3000 x 1024 x 128, all far.)
constexpr int kPrbRestGrid = 1024;
// How many there are; s_first: the lists' first numbers.  By the first wave and all threads that read it; ends with a barrier.
__device__ __forceinline__ int rest_count(const ProbeArgs &a, uint32_t *s_first) {
    if (threadIdx.x < kWave) {
        const int lane = threadIdx.x;
        uint32_t v = lane < kPrbLefts ? a.left[lane * kPrbApart] : 0u;
#pragma unroll
        for (int off = 1; off < kPrbLefts; off <<= 1) {
            const uint32_t o = (uint32_t)__shfl_up((int)v, off);
            if (lane >= off) v += o;
        }
        if (lane < kPrbLefts) s_first[lane + 1] = v;
        if (lane == 0) s_first[0] = 0;
    }
    sync_block();
    return (int)s_first[kPrbLefts];
}
__device__ __forceinline__ uint32_t rest_query(const ProbeArgs &a, const uint32_t *s_first, int i) {
    int list = 0;
#pragma unroll
    for (int step = kPrbLefts / 2; step > 0; step >>= 1)
        if (s_first[list + step] <= (uint32_t)i) list += step;
    return a.left[kPrbLefts * kPrbApart + list * a.left_pitch + ((uint32_t)i - s_first[list])];
}
__global__ __launch_bounds__(kProbeThreads) void probe_rest_kernel(const ProbeArgs a) {
    extern __shared__ __align__(16) float q_lds[];     // [8][d]
    __shared__ uint32_t s_q[8], s_first[kPrbLefts + 1];
    constexpr int kRows = kProbeThreads / 32 * 4;
    const int tid = threadIdx.x, count = rest_count(a, s_first), groups = (count + 7) >> 3;
    // lists per turn: 32; as many as leave every workgroup two turns where the queries are many (they are brought less often)
    int per = kRows;
    while (per < a.nlist && (int64_t)groups * ((a.nlist + 2 * per - 1) / (2 * per)) >= 2 * gridDim.x) per *= 2;
    const int tiles = (a.nlist + per - 1) / per;
    const int64_t units = (int64_t)groups * tiles;
    for (int64_t u = blockIdx.x; u < units; u += gridDim.x) {
        const int g0 = (int)(u / tiles) * 8, first = (int)(u % tiles) * per, nqt = count - g0 < 8 ? count - g0 : 8;
        const int end = first + per < a.nlist ? first + per : a.nlist;
        sync_block();                               // (the turn before is done with)
        if (tid < 8) s_q[tid] = rest_query(a, s_first, g0 + (tid < nqt ? tid : 0));
        sync_block();
        for (int t = tid; t < 8 * a.d; t += kProbeThreads) {
            const int qi = t / a.d;
            q_lds[t] = a.queries[(size_t)s_q[qi] * a.d + (t - qi * a.d)];
        }
        sync_block();
        for (int l0 = first + (tid >> 5) * 4; l0 < end; l0 += kRows)
            probe_distances<8>(q_lds, a.d, a.cent, a.nlist, l0, tid & 31, [&](int qi, int l, float v) {
                if (qi < nqt) a.t[(size_t)s_q[qi] * a.lpad + l] = v;
            });
    }
}
__global__ __launch_bounds__(kWave) void probe_rest_select_kernel(const ProbeArgs a) {
    __shared__ unsigned long long s_key[kSelectList];
    __shared__ uint32_t s_first[kPrbLefts + 1];
    const int count = rest_count(a, s_first);
    for (int i = blockIdx.x; i < count; i += gridDim.x) {
        const uint32_t q = rest_query(a, s_first, i);
        sync_block();                               // (the keys before these have been read)
        select_least(reinterpret_cast<const uint32_t *>(a.t) + (size_t)q * a.lpad, a.nlist, a.nprobe, a.out + (size_t)q * a.nprobe, s_key, threadIdx.x);
    }
}

}  // namespace trim
