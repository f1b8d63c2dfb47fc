// Gamma from a confidence level (Section 3.2, empirical route) with the matrix cores in front of the exact values.
//
// gamma_x is ONE value of the Q that a sampled vector x has, the one of a given rank.  gamma_kernel (trim_aux.h) computes
// all of them and is bound by the vector ALU; here
//
//   operands   landmarks l, differences u = x - l and queries as 16-bit operands (relative to the mean of a few queries,
//              scaled row by row by a power of two), with their lengths and what rounding moved
//   bins       q.l and q.u by v_mfma_f32_32x32x16_f16, and from them, per pair, two bins of 1 - cos(u, q - l) (2048
//              bins over [0, 2]): the value lies in neither a lower nor a higher one.  16 bits per pair.
//   rank       per vector: with lo and hi the rank'th of the lower and of the upper bins, the value wanted lies in lo .. hi;
//              who is certainly below is counted, who is certainly above is dropped, the others (some hundred of
//              10,000) are evaluated by the exact rule, and the rank is found among them.
//
// so that the result is gamma_kernel's bit for bit.  1000 vectors x 10,000 queries x 128: 67 us (258 with gamma_kernel): operands 13,
// bins 22, rank 36, all of them latency; 100 x 1000 x 384: 33 us (34); 1000 x 10,000 x 768: 308 (837), the
// values around the rank.  4096 bins leave fewer of those and cost more in the counting (76 us, 75 -> 81 for 1667 x 768).  Queries' lengths over four
// decades: 70 us (256; 304 where the mean is not kept within the vectors' range).  Vectors at their landmarks have one value
// with all queries, known without them: 108 us (229; evaluated 482).  What cannot be told apart at all is evaluated, a vector
// at a time where gamma_kernel takes two: 10,000 equal queries 486 us (228).
//
// Bound of the error, with Q', L', U' the rounded operands in the units of the
// data, moved(.) their distances from the true ones, r = |Q' - L'|, a = U'.(Q' - L') / |U'|, delta = moved(q) + moved(l):
//     |cos' - cos| <= (2 delta + 2 moved(u) / |U'| (r + delta) + eA + e2 / r) / r + (d / 8 + 64) 2^-24
// where e2 = (4 d + 64) 2^-24 (|Q'|^2 + |L'|^2) and eA = (2 d + 64) 2^-24 (|Q'| + |L'|) bound the binary32 sums and the last
// term the exact rule's own roundings.  What has no finite bound below 1 may lie in any bin (rows out of the scaled
// range, a query at its landmark, values that are no numbers): such pairs are all evaluated exactly.
#pragma once

#include "trim_aux.h"

namespace trim {

constexpr int kGrBins = 2048, kGrWide = 15;     // a key: lower bin << 4 | bins up to the upper one (kGrWide: unknown)
constexpr int kGrQueries = 256;
constexpr int kGrList = 2048;                   // keys to be evaluated that fit the LDS
struct GammaRankArgs {
    GammaArgs g;
    int32_t s0, ns;            // the sampled vectors of this chunk
    int32_t dpad, qpad;        // values per operand row (a multiple of 16), queries (of kGrQueries)
    int32_t vector_blocks;     // blocks of 32 vectors
    _Float16 *l16, *u16, *q16; // [block of 32 rows][dpad / 8][32][8]
    float *vpar;               // [vector][8]: 1 / scale of l, |L'|^2, moved(l), |L'|, 1 / |u'|, U'.L' / |U'|, 2 moved(u) / |U'|
    float4 *qpar;              // 1 / scale, |Q'|^2, moved(q), |Q'|
    uint16_t *keys;            // [vector][qpad]
    uint32_t *lists;           // [vector][qpad]: the keys to be evaluated where they are more than kGrList
};

// The power of two that brings m to 2^9 .. 2^10; 1 for m = 0; 0 where squares could leave the binary32 range.
__device__ __forceinline__ float gamma_scale(float m) {
    if (m == 0.0f) return 1.0f;
    if (!(m > 1e-12f && m < 1e12f)) return 0.0f;
    return __uint_as_float((uint32_t)(9 - ((int)(__float_as_uint(m) >> 23) - 127) + 127) << 23);
}

// One workgroup per eight rows, a half wave per row: first the vectors (l and u), then the queries.  Two passes: the
// scale, the operands.  (Eight threads per row took 90 us for rows of 768 values: a chain of gathers.)
constexpr int kGrRows = 8;
__global__ __launch_bounds__(256) void gamma_operands_kernel(const GammaRankArgs a) {
    typedef _Float16 h8 __attribute__((ext_vector_type(8)));
    extern __shared__ __align__(16) float s_mu[];      // [dpad]
    const int tid = threadIdx.x, part = tid & 31, d = a.g.d, np = a.dpad >> 3;
    const int vector_groups = a.vector_blocks * (32 / kGrRows);
    const bool vec = (int)blockIdx.x < vector_groups;
    const int row = (vec ? blockIdx.x : blockIdx.x - vector_groups) * kGrRows + (tid >> 5);
    if (blockIdx.x == 0 && a.s0 == 0 && tid == 0) *a.g.gamma_bits = 0x7f800000u;      // +inf: the minimum comes later
    for (int t = tid; t < a.dpad; t += 256) {
        // (within the range of a few stored vectors: a query far away would cost all of them their low bits)
        float v[8], x[8], sum = 0.0f, least = __builtin_inff(), most = -__builtin_inff();
        const int k = t < d ? t : 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = a.g.queries[(size_t)((int64_t)i * a.g.Q >> 3) * d + k];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = a.g.base[(size_t)(i * a.g.n >> 3) * d + k];
#pragma unroll
        for (int i = 0; i < 8; ++i) { least = __builtin_fminf(least, x[i]); most = __builtin_fmaxf(most, x[i]); }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float c = __builtin_fminf(__builtin_fmaxf(v[i], least), most);
            sum += __builtin_fabsf(c) < 1e18f ? c : 0.0f;
        }
        s_mu[t] = t < d ? sum * 0.125f : 0.0f;
    }
    sync_block();
    const int dsub = d / a.g.M;
    const float *x;                   // a vector, or a query
    const uint8_t *code = nullptr;
    if (vec) {
        int64_t at = a.g.rows[a.s0 + (row < a.ns ? row : a.ns - 1)];
        at = at < 0 ? 0 : (at >= a.g.n ? a.g.n - 1 : at);
        x = a.g.base + (size_t)at * d;
        code = a.g.codes + (size_t)at * a.g.M;
    } else {
        x = a.g.queries + (size_t)(row < a.g.Q ? row : a.g.Q - 1) * d;
    }
    // first: l - mu (or q - mu), second: u (or nothing)
    auto values = [&](int p, float (&first)[8], float (&second)[8]) {
        int j = 8 * p / dsub, o = 8 * p - j * dsub;                // subspace, place in it
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int t = 8 * p + e < d ? 8 * p + e : d - 1;       // (past the end: no value)
            const float xt = x[t];
            float lt = xt;
            if (vec) {
                const int js = j < a.g.M ? j : a.g.M - 1;
                lt = a.g.codebooks[((size_t)js * kC + code[js]) * dsub + o];
                if (++o == dsub) { o = 0; ++j; }
            }
            first[e] = 8 * p + e < d ? lt - s_mu[t] : 0.0f;
            second[e] = 8 * p + e < d ? xt - lt : 0.0f;
        }
    };
    // (a NaN is passed over by the maximum: the sum keeps it)
    float most[2] = {0.0f, 0.0f}, bad = 0.0f;
    for (int p = part; p < np; p += 32) {
        float v[8], w[8];
        values(p, v, w);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            most[0] = __builtin_fmaxf(most[0], __builtin_fabsf(v[e]));
            most[1] = __builtin_fmaxf(most[1], __builtin_fabsf(w[e]));
            bad += (v[e] - v[e]) + (w[e] - w[e]);
        }
    }
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) {
        most[0] = __builtin_fmaxf(most[0], __shfl_xor(most[0], off));
        most[1] = __builtin_fmaxf(most[1], __shfl_xor(most[1], off));
        bad += __shfl_xor(bad, off);
    }
    const float sf = gamma_scale(most[0]), su = gamma_scale(most[1]);
    const bool usable = bad == 0.0f && sf > 0.0f && (!vec || (su > 0.0f && most[1] > 0.0f));
    // |L'|^2, moved(l)^2, |U'|^2, moved(u)^2, U'.L' (scaled)
    float sum[5] = {};
    for (int p = part; p < np; p += 32) {
        float v[8], w[8];
        values(p, v, w);
        h8 hv, hw;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float fv = usable ? v[e] * sf : 0.0f, fw = usable ? w[e] * su : 0.0f;
            hv[e] = (_Float16)fv;
            hw[e] = (_Float16)fw;
            const float rv = (float)hv[e], rw = (float)hw[e], mv = fv - rv, mw = fw - rw;
            sum[0] = __builtin_fmaf(rv, rv, sum[0]);
            sum[1] = __builtin_fmaf(mv, mv, sum[1]);
            sum[2] = __builtin_fmaf(rw, rw, sum[2]);
            sum[3] = __builtin_fmaf(mw, mw, sum[3]);
            sum[4] = __builtin_fmaf(rv, rw, sum[4]);
        }
        const size_t at = ((size_t)(row >> 5) * np + p) * 32 + (row & 31);
        reinterpret_cast<h8 *>(vec ? a.l16 : a.q16)[at] = hv;
        if (vec) reinterpret_cast<h8 *>(a.u16)[at] = hw;
    }
#pragma unroll
    for (int off = 16; off > 0; off >>= 1)
#pragma unroll
        for (int i = 0; i < 5; ++i) sum[i] += __shfl_xor(sum[i], off);
    if (part != 0) return;
    const float lost = sqrt_rn((float)d) * (1.0f / 16384.0f);      // (subnormal 16-bit operands may count as zero)
    const float inv = usable ? 1.0f / sf : 0.0f, n2 = sum[0] * inv * inv, n = sqrt_rn(n2);
    const float moved = usable ? (sqrt_rn(sum[1]) * 1.001f + sqrt_rn(sum[0]) * (1.0f / 4194304.0f) + lost) * inv : __builtin_inff();
    if (vec) {
        float *out = a.vpar + (size_t)row * 8;
        const float iu = 1.0f / sqrt_rn(sum[2]);      // (infinite, or no number, only where moved is infinite)
        out[0] = inv; out[1] = n2; out[2] = moved; out[3] = n;
        out[4] = iu;
        out[5] = sum[4] * inv * iu;
        out[6] = 2.0f * (sqrt_rn(sum[3]) * 1.001f + lost) * iu;
    } else {
        a.qpar[row] = make_float4(inv, n2, moved, n);
    }
}

// A wave: 32 vectors x 64 queries.  An operand is read as it is stored, 1 KB per wave and load; q.l and q.u of a pair
// end in the same lane.
__global__ __launch_bounds__(256) void gamma_bins_kernel(const GammaRankArgs a) {
    typedef _Float16 h8 __attribute__((ext_vector_type(8)));
    typedef float v16f __attribute__((ext_vector_type(16)));
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 31, half = lane >> 5;
    const int q0 = blockIdx.x * kGrQueries + wave * 64, vb = blockIdx.y, np = a.dpad >> 3;
    __shared__ float4 s_qpar[kGrQueries];
    s_qpar[threadIdx.x] = a.qpar[blockIdx.x * kGrQueries + threadIdx.x];
    const h8 *lp = reinterpret_cast<const h8 *>(a.l16) + (size_t)vb * np * 32 + lane;
    const h8 *up = reinterpret_cast<const h8 *>(a.u16) + (size_t)vb * np * 32 + lane;
    const h8 *qp = reinterpret_cast<const h8 *>(a.q16) + (size_t)(q0 >> 5) * np * 32 + lane;
    v16f al[2], au[2];
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int i = 0; i < 16; ++i) al[v][i] = au[v][i] = 0.0f;
    // two steps of 16 values on their way while one is used
    h8 f[3][4];
    const int steps = np >> 1;
    auto load = [&](int step, h8 (&to)[4]) {
        const size_t k = (size_t)(step < steps ? step : steps - 1) * 64;
        to[0] = lp[k];
        to[1] = up[k];
        to[2] = qp[k];
        to[3] = qp[(size_t)np * 32 + k];
    };
    load(0, f[0]);
    load(1, f[1]);
    for (int s = 0; s < steps; s += 3) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            load(s + i + 2, f[(i + 2) % 3]);
            if (s + i < steps) {
#pragma unroll
                for (int v = 0; v < 2; ++v) {
                    al[v] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[i][2 + v], f[i][0], al[v], 0, 0, 0);
                    au[v] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[i][2 + v], f[i][1], au[v], 0, 0, 0);
                }
            }
        }
    }
    sync_block();
    constexpr float kUlp = 1.0f / 16777216.0f;
    const float d = (float)a.g.d;
    const float *vp = a.vpar + (size_t)(vb * 32 + col) * 8;
    const float il = -2.0f * vp[0], n2l = vp[1], ml = vp[2], nl = vp[3], iu = vp[4], cl = vp[5], ru = vp[6];
    const float c0 = (d * 0.125f + 64.0f) * kUlp + 1e-6f, c2 = (4.0f * d + 64.0f) * kUlp, ca = (2.0f * d + 64.0f) * kUlp;
    uint16_t *out = a.keys + (size_t)(vb * 32 + col) * a.qpad + q0;
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int i = 0; i < 16; i += 4) {
            const int at = v * 32 + 2 * i + 4 * half;
            uint32_t key[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float4 q = s_qpar[wave * 64 + at + e];
                const float ss = q.y + n2l, r2 = __builtin_fmaf(al[v][i + e], q.x * il, ss);
                const float ri = __builtin_amdgcn_rsqf(r2), r = r2 * ri;
                const float cosv = __builtin_fmaf(au[v][i + e], q.x * iu, -cl) * ri;
                const float delta = q.z + ml;
                const float err = ((2.0f * delta + ru * (r + delta) + ca * (q.w + nl)) + c2 * ss * ri) * ri * 1.01f + c0;
                const float mid = 1.0f - cosv;
                int lo = (int)((mid - err) * (kGrBins / 2)), hi = (int)((mid + err) * (kGrBins / 2));   // (below 0: towards 0, clamped)
                lo = lo < 0 ? 0 : (lo > kGrBins - 1 ? kGrBins - 1 : lo);
                hi = hi < 0 ? 0 : (hi > kGrBins - 1 ? kGrBins - 1 : hi);
                // (r2 not above zero: ri is no finite number, and neither is err)
                key[e] = err < 1.0f ? (uint32_t)(lo << 4 | (hi - lo < kGrWide ? hi - lo : kGrWide)) : (uint32_t)kGrWide;
            }
            uint2 w;
            w.x = key[0] | key[1] << 16;
            w.y = key[2] | key[3] << 16;
            *reinterpret_cast<uint2 *>(out + at) = w;
        }
}

// One workgroup per vector.  LDS: l and u, the bins (lower counts in the low halves, upper counts in the high ones; Q
// is at most 16384), the numbers, then the keys, of those to be evaluated.  Bound by latency, a chain of short steps:
// the LDS is kept small enough for four workgroups per CU and more.  T: 256 threads; 512 where there are few vectors.
inline size_t gamma_rank_lds(int d) { return ((size_t)2 * d * 4 + 15) / 16 * 16 + (kGrBins + kGrList) * 4; }
template <int T>
__global__ __launch_bounds__(T, 4) void gamma_rank_kernel(const GammaRankArgs a) {
    constexpr int kPer = kGrBins / T, kWaves = T / kWave;
    extern __shared__ __align__(16) unsigned char smem[];
    const int d = a.g.d, Q = a.g.Q;
    float *l = reinterpret_cast<float *>(smem), *u = l + d;
    uint32_t *hist = reinterpret_cast<uint32_t *>(smem + ((size_t)2 * d * 4 + 15) / 16 * 16);
    uint32_t *list = hist + kGrBins;
    __shared__ float norm_part[kGammaThreads / kWave];
    __shared__ uint32_t part[kWaves];
    __shared__ int s_lo, s_hi, s_n;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int64_t s = (int64_t)a.s0 + blockIdx.x;
    int64_t at = a.g.rows[s];
    at = at < 0 ? 0 : (at >= a.g.n ? a.g.n - 1 : at);
    const int dsub = d / a.g.M;
    for (int b = tid; b < kGrBins; b += T) hist[b] = 0;
    if (tid == 0) s_n = 0;
    sync_block();
    const uint4 *src = reinterpret_cast<const uint4 *>(a.keys + (size_t)blockIdx.x * a.qpad);
    auto each = [&](auto &&f) {                      // f(query, lower bin, upper bin)
        for (int i = tid; i * 8 < Q; i += T) {
            const uint4 w4 = src[i];
            const uint32_t w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t k = w[e >> 1] >> (16 * (e & 1)) & 0xffffu;
                const int lo = (int)(k >> 4), wide = (int)(k & 15u);
                if (8 * i + e < Q) f(8 * i + e, lo, wide == kGrWide ? kGrBins - 1 : lo + wide);
            }
        }
    };
    each([&](int, int lo, int hi) {
        atomicAdd(&hist[lo], 1u);
        atomicAdd(&hist[hi], 0x10000u);
    });
    // |u|^2, summed as gamma_kernel's threads do
    for (int v = tid; v < kGammaThreads; v += T) {
        float p = 0.0f;
        for (int t = v; t < d; t += kGammaThreads) {
            const int j = t / dsub;
            const float lt = a.g.codebooks[((size_t)j * kC + a.g.codes[(size_t)at * a.g.M + j]) * dsub + (t - j * dsub)];
            const float ut = a.g.base[(size_t)at * d + t] - lt;
            l[t] = lt;
            u[t] = ut;
            p = __builtin_fmaf(ut, ut, p);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) p += __shfl_xor(p, off);
        if (lane == 0) norm_part[v >> 6] = p;
    }
    sync_block();
    float norm2 = 0.0f;
    for (int w = 0; w < kGammaThreads / kWave; ++w) norm2 += norm_part[w];
    const float nu = sqrt_rn(norm2);
    if (nu == 0.0f) {                                // at its landmark: the angle counts as a right one with every query
        if (tid == 0) gamma_store(a.g, s, ordered_bits(1.0f));
        return;
    }
    uint32_t h[kPer], sum = 0;
    uint4 *mine = reinterpret_cast<uint4 *>(hist) + tid * (kPer / 4);
#pragma unroll
    for (int i = 0; i < kPer; i += 4) {
        const uint4 v = mine[i / 4];
        h[i] = v.x; h[i + 1] = v.y; h[i + 2] = v.z; h[i + 3] = v.w;
        sum += v.x + v.y + v.z + v.w;
    }
    uint32_t incl = sum;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t v = (uint32_t)__shfl_up((int)incl, off);
        if (lane >= off) incl += v;
    }
    if (lane == kWave - 1) part[wave] = incl;
    sync_block();
    uint32_t before = incl - sum;
    for (int w = 0; w < wave; ++w) before += part[w];
    const uint32_t rank = (uint32_t)a.g.rank;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const uint32_t next = before + h[i];
        if (rank >= (before & 0xffffu) && rank < (next & 0xffffu)) s_lo = tid * kPer + i;
        if (rank >= before >> 16 && rank < next >> 16) s_hi = tid * kPer + i;
        h[i] = (before & 0xffff0000u) | (next & 0xffffu);   // upper bins below this one, lower bins up to it
        before = next;
    }
#pragma unroll
    for (int i = 0; i < kPer; i += 4) mine[i / 4] = make_uint4(h[i], h[i + 1], h[i + 2], h[i + 3]);
    sync_block();
    const int lo = s_lo, hi = s_hi, below = (int)(hist[lo] >> 16), n = (int)(hist[hi] & 0xffffu) - below;
    const int want = a.g.rank - below;
    const int lane32 = tid & 31, ng = d >> 2;
    const float4 *l4 = reinterpret_cast<const float4 *>(l), *u4 = reinterpret_cast<const float4 *>(u);
    auto evaluate = [&](uint32_t *keys) {            // LDS, or memory
        each([&](int q, int l0, int h0) {
            if (h0 >= lo && l0 <= hi) keys[atomicAdd(&s_n, 1)] = (uint32_t)q;
        });
        sync_block();
        constexpr int QB = 4;
        for (int i0 = (tid >> 5) * QB; i0 < n; i0 += (T / 32) * QB) {
            const float4 *row[QB];
            float acc[2 * QB];
#pragma unroll
            for (int i = 0; i < QB; ++i) {
                row[i] = reinterpret_cast<const float4 *>(a.g.queries + (size_t)keys[i0 + i < n ? i0 + i : n - 1] * d);
                acc[i] = acc[QB + i] = 0.0f;
            }
            for (int g = lane32; g < ng; g += 32) {
                float4 qv[QB];
#pragma unroll
                for (int i = 0; i < QB; ++i) qv[i] = row[i][g];
                const float4 lv = l4[g], uv = u4[g];
#pragma unroll
                for (int i = 0; i < QB; ++i) gamma_step(qv[i], lv, uv, acc[i], acc[QB + i]);
            }
            const float v = reduce_pairs<2 * QB>(acc, lane32);     // lane: dot / norm (bit 4), query (bits 2..3)
            const float nn = __shfl_xor(v, 16);
            const int i = i0 + (lane32 >> 2 & 3);
            // (numbers of this half wave's own: read above, before they are replaced)
            if (!(lane32 & 19) && i < n) keys[i] = gamma_key(v, nn, nu);
        }
        sync_block();
    };
    if (n > kGrList) {
        uint32_t *keys = a.lists + (size_t)blockIdx.x * a.qpad;
        evaluate(keys);
        const uint32_t k = key_of_rank<T>(keys, n, want, reinterpret_cast<int *>(hist));
        if (tid == 0) gamma_store(a.g, s, k);
        return;
    }
    evaluate(list);
    if (n > T) {
        const uint32_t k = key_of_rank<T>(list, n, want, reinterpret_cast<int *>(hist));
        if (tid == 0) gamma_store(a.g, s, k);
    } else if (tid < n) {        // few: everybody counts who is below
        const uint32_t k = list[tid];
        int less = 0;
        for (int i = 0; i < n; ++i) less += list[i] < k || (list[i] == k && i < tid);
        if (less == want) gamma_store(a.g, s, k);
    }
}

}  // namespace trim
