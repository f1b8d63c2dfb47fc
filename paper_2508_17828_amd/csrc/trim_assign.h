// The nearest list of many vectors of at most 128 values (trim_ivf_probe with one probe, trim_train_ivf) with work space: the lists'
// operands are made once (assign_operands_kernel), and a wave keeps 32 vectors' operands in registers while the lists pass by
// (assign_tiles_kernel).  Scores, their bounds and what is measured exactly: as in assign_rows_kernel (trim_aux.h), which goes without.
#pragma once

#include "trim_aux.h"

namespace trim {

constexpr int kAstThreads = 512, kAstVecs = 256;           // 32 vectors per wave
constexpr int kAstPairs = 16;                               // of a vector that are measured; more: it is marked
constexpr float kAstPiece = 32768.0f, kAstReach = 2.0e9f;
template <int KS>
struct AstShape {                                          // KS: steps of 16 values, 4 or 8
    static constexpr int kRows = 512 / KS, kTiles = kRows / 32;            // lists per stage
    static constexpr int kStage = (2 * KS + 1) * kRows;                    // 16-byte pieces
};
struct AstHead {
    float twice[kAsrCols];         // 2 mu scale (0 past d)
    float scale, pad[3];
};
struct AstLayout {
    int nst;
    size_t off_most, off_ops, total;
};
inline AstLayout ast_layout(int d, int nlist) {
    AstLayout L{};
    const int ks = d <= kAsrCols / 2 ? 4 : 8, rows = 512 / ks;
    L.nst = (nlist + rows - 1) / rows;
    L.off_most = (sizeof(AstHead) + 255) & ~size_t(255);
    L.off_ops = (L.off_most + (size_t)L.nst * 8 + 255) & ~size_t(255);
    L.total = L.off_ops + (size_t)L.nst * (2 * ks + 1) * rows * 16;
    return L;
}

// A stage of lists per workgroup: operands in the order in which assign_tiles_kernel's instructions take them, [2 KS + 1][rows] pieces of
// 16 bytes, and the stage's largest |c'|^2 and largest square of what rounding moved.
template <int KS>
__global__ __launch_bounds__(512) void assign_operands_kernel(const float *__restrict__ cent, int nlist, int d, AstHead *__restrict__ head,
                                                              uint32_t *__restrict__ most_of, uint4 *__restrict__ ops) {
    typedef _Float16 h8 __attribute__((ext_vector_type(8)));
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    typedef _Float16 h4 __attribute__((ext_vector_type(4)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef float f4 __attribute__((ext_vector_type(4)));
    using Shape = AstShape<KS>;
    __shared__ __align__(16) float s_mu[kAsrCols];
    __shared__ uint32_t s_top[2], s_cmax, s_mmax;
    const int tid = threadIdx.x, lane = tid & 63, st = blockIdx.x;
    const int s_row = tid / KS, s_ks = tid & (KS - 1), c = st * Shape::kRows + s_row;
    f4 a[4];                        // KS lanes bring a row, 16 bytes each at a time
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int k = 4 * (g * KS + s_ks);
        a[g] = *reinterpret_cast<const f4 *>(cent + (size_t)(c < nlist ? c : nlist - 1) * d + (k < d ? k : 0));
    }
    if (tid < kAsrCols) {           // mean and spread of 16 centroids
        float v[16], sum = 0.0f;
        const int t = tid < d ? tid : 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = cent[(size_t)((int64_t)i * nlist >> 4) * d + t];
#pragma unroll
        for (int i = 0; i < 16; ++i) sum += v[i];
        const float mu = sum * (1.0f / 16.0f);
        uint32_t top = 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) top = max(top, __float_as_uint(__builtin_fabsf(v[i] - mu)));
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) top = max(top, (uint32_t)__shfl_xor((int)top, off));
        s_mu[tid] = mu;
        if (lane == 0) s_top[tid >> 6] = top;
    }
    if (tid == 0) s_cmax = s_mmax = 0;
    sync_block();
    const uint32_t top = max(s_top[0], s_top[1]);
    const bool usable = __uint_as_float(top) > 1e-30f && __uint_as_float(top) < 1e30f;
    const float sc = __uint_as_float((uint32_t)((usable ? 6 - ((int)(top >> 23) - 127) : 0) + 127) << 23);     // (the spread: 2^6 .. 2^7)
    if (st == 0) {
        if (tid < kAsrCols) head->twice[tid] = tid < d ? 2.0f * (s_mu[tid] * sc) : 0.0f;
        if (tid == 0) head->scale = sc;
    }
    uint4 *to = ops + (size_t)st * Shape::kStage;
    float norm = 0.0f, moved = 0.0f;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int k = 4 * (g * KS + s_ks);
        const f4 m = *reinterpret_cast<const f4 *>(s_mu + k);
        const float by = k < d ? sc : 0.0f;
        h2 f[2];
#pragma unroll
        for (int e = 0; e < 4; e += 2) {       // (the power of two: one rounding, that of the difference)
            const f2 v = {__builtin_fmaf(a[g][e], by, -(m[e] * by)), __builtin_fmaf(a[g][e + 1], by, -(m[e + 1] * by))};
            const h2 h = __builtin_convertvector(v, h2);
            const f2 back = __builtin_convertvector(h, f2);
            const float r0 = v[0] - back[0], r1 = v[1] - back[1];
            moved = __builtin_fmaf(r0, r0, moved);
            moved = __builtin_fmaf(r1, r1, moved);
            norm = __builtin_amdgcn_fdot2(h, h, norm, false);
            f[e / 2] = h;
        }
        *reinterpret_cast<h4 *>(reinterpret_cast<unsigned char *>(to + (k >> 3) * Shape::kRows + s_row) + (k & 4) * 2) =
            h4{f[0][0], f[0][1], f[1][0], f[1][1]};
    }
#pragma unroll
    for (int off = 1; off < KS; off <<= 1) {
        norm = norm + __shfl_xor(norm, off);
        moved = moved + __shfl_xor(moved, off);
    }
    if (s_ks == 0) {
        const _Float16 kp = (_Float16)kAstPiece;
        h8 f = {(_Float16)65504.0f, (_Float16)65504.0f, (_Float16)65504.0f, kp, kp, kp, 0, 0};      // (rows past the end: far away)
        if (c < nlist) {
            // (bit patterns: a centroid that is no number is the largest, and everybody is measured exactly)
            atomicMax(&s_cmax, norm < kAstReach ? __float_as_uint(norm) : 0x7f800000u);
            atomicMax(&s_mmax, __float_as_uint(moved));
            const float q = norm * (1.0f / kAstPiece);          // three pieces of the norm; the other side of them is kAstPiece
            const _Float16 p1 = (_Float16)q, p2 = (_Float16)(q - (float)p1), p3 = (_Float16)((q - (float)p1) - (float)p2);
            f[0] = p1; f[1] = p2; f[2] = p3;
        }
        *reinterpret_cast<h8 *>(to + 2 * KS * Shape::kRows + s_row) = f;
    }
    sync_block();
    if (tid == 0) { most_of[2 * st] = s_cmax; most_of[2 * st + 1] = s_mmax; }
}

//   operands  -2 x' of 32 vectors per wave, through the LDS once (rows are read 128 bytes at a time); |x'|^2 and |c'|^2 as one more step
//             (three binary16 pieces each against 2^15)
//   trackers  a lane sees 16 lists of every tile of 32 for its vector.  Of every tile the least score is kept, the four least of these with
//             the tile's number in the low bits; and of every place in a tile the least over all tiles: 1.3 operations a score (four with
//             three numbered least ones of all scores).  A list within the bound is in a tile and at a place within it.
//   decision  one tile and one place: that list.  Otherwise the lists at these places of these tiles are measured by the exact rule, four
//             pairs to a half wave; the vector is marked where there are more than kAstPairs, or the fourth tile is within the bound too
// Two workgroups of eight waves per CU (128 registers): one reads its rows while the other multiplies.  1,000,000 x 128 against 1024 lists:
// 320 us with the kernels before and after it (650 with assign_rows_kernel, whose every workgroup converts the lists), 65,536 x 128 45 (55),
// 200,000 x 128 against 450 62 (105), 500,000 x 96 against 2049 280 (545), 4096 x 128 against 64 16 (16).  Of a workgroup's 64,000 clocks
// with another beside it 16,000 pass until its rows are there, 40,000 over the lists (37,000 of products in both), 5,000 for the decision.
// (64 vectors per wave, half as many waves: 350 us; one half of the waves multiplying while the other tracks, or the next rows asked for
// before the decision: registers spill.)
template <int KS>
__global__ __launch_bounds__(kAstThreads, 4) void assign_tiles_kernel(const float *__restrict__ xs, int64_t n, int d,
                                                                      const float *__restrict__ cent, int nlist, int nst,
                                                                      const AstHead *__restrict__ head, const uint32_t *__restrict__ most_of,
                                                                      const uint4 *__restrict__ ops, int32_t *__restrict__ out) {
    typedef _Float16 h8 __attribute__((ext_vector_type(8)));
    typedef _Float16 h4 __attribute__((ext_vector_type(4)));
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    typedef float v16f __attribute__((ext_vector_type(16)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef float f4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    using Shape = AstShape<KS>;
    constexpr int kWaves = kAstThreads / kWave, kFetch = (Shape::kStage + kAstThreads - 1) / kAstThreads;
    constexpr int kChunks = KS / 2, kPitch = 34;                                // of 32 values; 16-byte pieces from one eight values to the next
    __shared__ __align__(16) u4 s_ops[2][Shape::kStage];                        // (the vectors' operands before that)
    __shared__ float s_xn[kAstVecs], s_xm[kAstVecs];
    __shared__ uint32_t s_pair[kWaves][32 * kAstPairs];                         // vector of the wave | list << 5
    __shared__ unsigned long long s_best[kAstVecs];
    __shared__ int s_np[kWaves];
    static_assert(kWaves * 8 * kPitch <= 2 * Shape::kStage, "room");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    u4 ahead[kFetch];
    auto fetch = [&](int st) {
        const u4 *from = reinterpret_cast<const u4 *>(ops) + (size_t)st * Shape::kStage;
#pragma unroll
        for (int i = 0; i < kFetch; ++i) {
            const int p = i * kAstThreads + tid;
            ahead[i] = from[p < Shape::kStage ? p : 0];
        }
    };
    auto place = [&](int buf) {
#pragma unroll
        for (int i = 0; i < kFetch; ++i) {
            const int p = i * kAstThreads + tid;
            if ((i + 1) * kAstThreads <= Shape::kStage || p < Shape::kStage) s_ops[buf][p] = ahead[i];
        }
    };
    auto in_order = [] {           // of the wave's own LDS accesses
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    const int64_t x0 = (int64_t)blockIdx.x * kAstVecs + wave * 32;
    // ---- the wave's vectors ----
    h8 xo[KS + 1];
    {
        const int r8 = lane >> 3, k4 = 4 * (lane & 7);         // eight lanes bring 128 bytes of a row
        f4 v[4][kChunks];
#pragma unroll
        for (int i = 0; i < kChunks; ++i)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int64_t r = x0 + g * 8 + r8;
                const int k = i * 32 + k4;
                v[g][i] = *reinterpret_cast<const f4 *>(xs + (size_t)(r < n ? r : n - 1) * d + (k < d ? k : 0));
            }
        const float by = -2.0f * head->scale;
        float norm[4] = {}, moved[4] = {};
        h8 *area = reinterpret_cast<h8 *>(&s_ops[0][0]) + wave * 8 * kPitch;
#pragma unroll
        for (int c = 0; c < kChunks; c += 2) {
#pragma unroll
            for (int i = c; i < c + 2; ++i) {
                const int k = i * 32 + k4;
                const f4 m = *reinterpret_cast<const f4 *>(head->twice + k);
                const float f = k < d ? by : 0.0f;              // (columns past d: nothing)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    h4 o4;
#pragma unroll
                    for (int e = 0; e < 4; e += 2) {            // (a power of two: one rounding, that of the difference)
                        const f2 w = {__builtin_fmaf(v[g][i][e], f, m[e]), __builtin_fmaf(v[g][i][e + 1], f, m[e + 1])};
                        const h2 o = __builtin_convertvector(w, h2);
                        const f2 back = __builtin_convertvector(o, f2);
                        const float r0 = w[0] - back[0], r1 = w[1] - back[1];
                        moved[g] = __builtin_fmaf(r0, r0, moved[g]);
                        moved[g] = __builtin_fmaf(r1, r1, moved[g]);
                        norm[g] = __builtin_amdgcn_fdot2(o, o, norm[g], false);
                        o4[e] = o[0];
                        o4[e + 1] = o[1];
                    }
                    *reinterpret_cast<h4 *>(reinterpret_cast<unsigned char *>(area + (((k >> 3) & 7) * kPitch + g * 8 + r8)) + (k & 4) * 2) = o4;
                }
            }
            in_order();
#pragma unroll
            for (int ks = 2 * c; ks < 2 * c + 4; ++ks) xo[ks] = area[((ks * 2 + half) & 7) * kPitch + col];
            in_order();
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            norm[g] = norm[g] + lane_xor<1>(norm[g]);
            moved[g] = moved[g] + lane_xor<1>(moved[g]);
            norm[g] = norm[g] + lane_xor<2>(norm[g]);
            moved[g] = moved[g] + lane_xor<2>(moved[g]);
            norm[g] = norm[g] + lane_xor<4>(norm[g]);
            moved[g] = moved[g] + lane_xor<4>(moved[g]);
            if ((lane & 7) == 0) {
                s_xn[wave * 32 + g * 8 + r8] = 0.25f * norm[g];
                s_xm[wave * 32 + g * 8 + r8] = 0.25f * moved[g];
            }
        }
    }
    fetch(0);
    if (lane == 0) s_np[wave] = 0;
    if (half == 0) s_best[wave * 32 + col] = ~0ull;
    sync_block();
    place(0);
    fetch(nst > 1 ? 1 : 0);
    // a vector per column from here on, in both half waves
    float xn = s_xn[wave * 32 + col];
    {
        const bool fits = xn < kAstReach;                       // (else out of the 16-bit range: nothing is known)
        const float q = fits ? xn * (1.0f / kAstPiece) : 0.0f;
        if (!fits) xn = __builtin_nanf("");
        const _Float16 kp = (_Float16)kAstPiece, p1 = (_Float16)q, p2 = (_Float16)(q - (float)p1), p3 = (_Float16)((q - (float)p1) - (float)p2);
        const u4 w = __builtin_bit_cast(u4, h8{kp, kp, kp, p1, p2, p3, 0, 0});
        u4 lower;
#pragma unroll
        for (int i = 0; i < 4; ++i) lower[i] = half == 0 ? w[i] : 0u;
        xo[KS] = __builtin_bit_cast(h8, lower);
    }
    // ---- the lists ----
    int t1 = 0x7f800000, t2 = t1, t3 = t1, t4 = t1, at[16];             // (of half of the lists)
#pragma unroll
    for (int i = 0; i < 16; ++i) at[i] = 0x7f800000;
    const int bits = 32 - __builtin_clz(nst * Shape::kTiles - 1);
    const uint32_t number = (1u << bits) - 1u;
#pragma unroll 1
    for (int st = 0; st < nst; ++st) {
        sync_block();
        if (st + 1 < nst) {
            place((st + 1) & 1);
            fetch(st + 2 < nst ? st + 2 : nst - 1);
        }
        const h8 *b = reinterpret_cast<const h8 *>(s_ops[st & 1]) + col;
#pragma unroll
        for (int tt = 0; tt < Shape::kTiles; tt += 2) {
            v16f acc[2] = {};
#pragma unroll
            for (int ks = 0; ks <= KS; ++ks)                    // (the last piece: the same for both halves, the vectors' side of the upper one is zero)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(b[(ks < KS ? ks * 2 + half : 2 * KS) * Shape::kRows + (tt + t) * 32], xo[ks],
                                                                    acc[t], 0, 0, 0);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                // (one below zero is within the bound of zero, as signed numbers too)
                int g = __float_as_int(acc[t][0]);
#pragma unroll
                for (int i = 1; i < 16; ++i) g = min(g, __float_as_int(acc[t][i]));
                g = (int)(((uint32_t)g & ~number) | (uint32_t)(st * Shape::kTiles + tt + t));
                t4 = max(min(g, t4), min(max(g, t4), t3));      // the middle one of the three
                t3 = max(min(g, t3), min(max(g, t3), t2));
                t2 = max(min(g, t2), min(max(g, t2), t1));
                t1 = min(t1, g);
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) at[i] = min(min(at[i], __float_as_int(acc[0][i])), __float_as_int(acc[1][i]));
        }
    }
    // ---- decision ----
    auto both = [](uint32_t a) { return __builtin_amdgcn_permlane32_swap(a, a, false, false); };       // the lower and the upper half wave's
    uint32_t cmax = 0, mmax = 0;
    for (int i = lane; i < nst; i += kWave) { cmax = max(cmax, most_of[2 * i]); mmax = max(mmax, most_of[2 * i + 1]); }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        cmax = max(cmax, (uint32_t)__shfl_xor((int)cmax, off));
        mmax = max(mmax, (uint32_t)__shfl_xor((int)mmax, off));
    }
    const auto least = both((uint32_t)t1);
    const float best = __int_as_float(min((int)least[0], (int)least[1]));
    const float sc = head->scale;
    constexpr float kUlp = 1.0f / 16777216.0f;
    const float lost = trim::sqrt_rn((float)d) * (1.0f / 16384.0f);             // (subnormal 16-bit operands may count as zero)
    const float mc = trim::sqrt_rn(__uint_as_float(mmax)) * 1.001f, mx = trim::sqrt_rn(s_xm[wave * 32 + col]) * 1.001f;
    const float cl = trim::sqrt_rn(__uint_as_float(cmax)) + mc, xl = trim::sqrt_rn(xn) + mx;
    // what moved an operand: rounding, the subtraction of mu, flushing; errors of a score: sums, flushed operands, the pieces of
    // the norms; the exact rule's own
    const float shift = mc + mx + (cl + xl) * 2.0f * kUlp + 2.0f * lost;
    const float e = (4.0f * d + 64.0f) * kUlp * (xl * cl + cl * cl + xl * xl) + 8.0f + (d / 32 + 8) * kUlp * (xl + cl) * (xl + cl);
    const float coarse = 1.0f + __uint_as_float((uint32_t)(127 - 21 + bits) << 23);      // (what the numbers took)
    const float reach = trim::sqrt_rn(__builtin_fmaxf(best, 0.0f) * coarse + e) + 2.0f * shift;
    const float thr = (reach * reach + e) * coarse, real = (e / sc) / sc;
    const bool known = real < 1e30f && real > 1e-30f && thr < 1e30f;
    uint32_t in = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) in |= __int_as_float(at[i]) <= thr ? 1u << i : 0u;
    const int tiles = (__int_as_float(t1) <= thr ? 1 : 0) + (__int_as_float(t2) <= thr ? 1 : 0) + (__int_as_float(t3) <= thr ? 1 : 0);
    const uint32_t count = (uint32_t)(tiles * __builtin_popcount(in)) + (__int_as_float(t4) > thr ? 0u : 1u << 16);
    auto list_of = [&](int key, int i) { return ((uint32_t)key & number) * 32 + 8 * (i >> 2) + 4 * half + (i & 3); };
    const auto counts = both(count), ones = both(count == 1u ? list_of(t1, __ffs((int)in) - 1) : 0u);
    const uint32_t total = counts[0] + counts[1], only = ones[0] + ones[1];
    int answer = known && total == 1u && only < (uint32_t)nlist ? (int)only : -1;
    const bool several = known && total > 1u && total <= (uint32_t)kAstPairs && x0 + col < n;
    if (several)
        for (int t = 0; t < tiles; ++t)
            for (uint32_t left = in; left; left &= left - 1) {
                const uint32_t id = list_of(t == 0 ? t1 : t == 1 ? t2 : t3, __ffs((int)left) - 1);
                if (id < (uint32_t)nlist) s_pair[wave][atomicAdd(&s_np[wave], 1)] = (uint32_t)col | id << 5;
            }
    in_order();
    const int np = s_np[wave], at4 = 4 * col < d ? 4 * col : 0;                 // (at most 32 groups of four)
    for (int i0 = half * 4; i0 < np; i0 += 8) {
        uint32_t pair[4];
        float part[4];
        f4 q[4], c[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            pair[i] = s_pair[wave][i0 + i < np ? i0 + i : i0];
            q[i] = *reinterpret_cast<const f4 *>(xs + (size_t)(x0 + (pair[i] & 31u)) * d + at4);
            c[i] = *reinterpret_cast<const f4 *>(cent + (size_t)(pair[i] >> 5) * d + at4);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {                        // (exact_d2_half's order)
            float sum = 0.0f;
#pragma unroll
            for (int j = 0; j < 4; ++j) { const float v = q[i][j] - c[i][j]; sum = __builtin_fmaf(v, v, sum); }
            part[i] = 4 * col < d ? sum : 0.0f;
        }
        const float dist = half_reduce_x4(part, col);
        const int i = half_reduce_x4_row(col);
        const uint32_t p = i == 0 ? pair[0] : i == 1 ? pair[1] : i == 2 ? pair[2] : pair[3];
        if (half_reduce_x4_writer(col) && i0 + i < np)
            atomicMin(&s_best[wave * 32 + (p & 31u)], ((unsigned long long)__float_as_uint(dist) << 32) | (p >> 5));
    }
    in_order();
    if (several && s_best[wave * 32 + col] != ~0ull) answer = (int)(s_best[wave * 32 + col] & 0xffffffffu);
    if (half == 0 && x0 + col < n) out[x0 + col] = answer;
}

}  // namespace trim
