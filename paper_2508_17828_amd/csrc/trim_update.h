// The update step of centroid training (Lloyd's k-means; Sections 2.2, 3.1, 6.1) with work space: the rule of
// kmeans_update_kernel (trim_aux.h), whose workgroups each look through all assignments for the rows of their clusters.  Here
// the rows are put in cluster order once:
//
//   kmeans_sort_kernel   a chunk of rows per workgroup, stable counting sort by cluster (ranks inside a wave by matching ballots, a
//                        counter per wave and cluster in the LDS); leaves the clusters' first places in the chunk and the rows' numbers
//   kmeans_sums_kernel   short rows: all threads bring the rows of some clusters to the LDS, one per (cluster, coordinate) adds them
//   kmeans_rows_kernel   long rows: a workgroup per cluster lists its rows, a thread per coordinate adds them straight from memory
//
// Rows are ascending inside a chunk's run of a cluster and from chunk to chunk, so every sum is added in row order.
//
// 65,536 rows: 32 x 256 x 4 coordinates 62 -> 43 us an iteration (sort 13.6, sums 29) and 13 us once for the columns; 1024 x 128 coordinates
// 41 -> 21 to 25 us by machine (sort 5.3, rows 15.4 to 19.6).  Bound by latency: a workgroup's first places, then its rows' numbers, then its rows come one after
// the other from beyond the L2, 4000 clocks each, and a clusters' longest run in a chunk takes 20 clocks a value; the sort by its
// ballots.  (Values stored in cluster order instead of numbers: sort 23 us, and as much again to read them.)
#pragma once

#include "trim_aux.h"

namespace trim {

constexpr int kSortThreads = 1024, kShortRow = 16;                     // values of a short row at most
constexpr int kSortCounters = 128 * 1024;                              // bytes of counters at most
constexpr int kSumThreads = 256, kSumFloats = 4096, kSumChunks = kWave, kSumMaxLog2 = 5;     // values, chunks at a time; clusters per workgroup
constexpr int kRowsFly = 32, kRowsCap = 2048;
struct SortArgs {
    const float *x;            // [ns][stride]
    const void *assign;        // of row r in clustering y: element r * astride + y * ystride
    int64_t ns, stride, astride, ystride;
    int64_t xstep;             // from one clustering's columns to the next's
    int32_t dim, K, kbits, ny, nchunk, rows;    // rows per chunk
    int32_t cg_log2;
    uint16_t *starts;          // [ny][nchunk][K + 1] first place of a cluster in the chunk
    uint16_t *list;            // [ny][ns] a chunk's rows in cluster order, less its first
    float *cent;
};
inline size_t kmeans_sort_lds(int threads, int K) { return (size_t)(threads / kWave) * ((K + 1) & ~1) * 2; }

// ABYTES, LOOPS: bytes of an assignment; rows per lane.
template <int ABYTES, int LOOPS>
__global__ __launch_bounds__(kSortThreads) void kmeans_sort_kernel(const SortArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_part[kSortThreads / kWave], s_carry;
    const int chunk = blockIdx.x, y = blockIdx.y, K = a.K, pitch = (K + 1) & ~1;
    const int tid = threadIdx.x, T = blockDim.x, lane = tid & (kWave - 1), wave = tid >> 6, waves = T >> 6;
    uint16_t *cnt = reinterpret_cast<uint16_t *>(smem), *mine = cnt + wave * pitch;      // [waves][pitch]
    const int64_t r0 = (int64_t)chunk * a.rows;
    const int nr = a.ns - r0 < a.rows ? (int)(a.ns - r0) : a.rows;
    uint32_t c[LOOPS];
#pragma unroll
    for (int s = 0; s < LOOPS; ++s) {
        const int i = (wave * LOOPS + s) * kWave + lane;
        const size_t e = (size_t)(r0 + (i < nr ? i : 0)) * a.astride + (size_t)y * a.ystride;
        c[s] = ABYTES == 1 ? static_cast<const uint8_t *>(a.assign)[e] : static_cast<const uint32_t *>(a.assign)[e];
        if (i >= nr) c[s] = 0xffffffffu;
    }
    for (int i = tid; i < waves * pitch / 2; i += T) reinterpret_cast<uint32_t *>(cnt)[i] = 0u;
    if (tid == 0) s_carry = 0;
    sync_block();
    const unsigned long long below = (1ull << lane) - 1ull;
    int rank[LOOPS];
#pragma unroll
    for (int s = 0; s < LOOPS; ++s) {
        const bool in = c[s] < (uint32_t)K;
        unsigned long long same = __ballot(in);
        for (int b = 0; b < a.kbits; ++b) {
            const bool bit = (c[s] >> b) & 1u;
            const unsigned long long m = __ballot(bit);
            same &= bit ? m : ~m;
        }
        const int before = __popcll(same & below);
        rank[s] = in ? (int)mine[c[s]] + before : -1;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (in && before == 0) mine[c[s]] = (uint16_t)(mine[c[s]] + __popcll(same));
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    sync_block();
    // counts -> first places
    uint16_t *starts = a.starts + ((size_t)y * a.nchunk + chunk) * (K + 1);
    for (int c0 = 0; c0 < K; c0 += T) {
        const int k = c0 + tid;
        int run = 0;
        if (k < K)
            for (int v = 0; v < waves; ++v) run += cnt[v * pitch + k];
        int incl = run;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int o = __shfl_up(incl, off);
            if (lane >= off) incl += o;
        }
        if (lane == kWave - 1) s_part[wave] = incl;
        sync_block();
        int at = s_carry + incl - run;
        for (int v = 0; v < wave; ++v) at += s_part[v];
        if (k < K) {
            starts[k] = (uint16_t)at;
            for (int v = 0, to = at; v < waves; ++v) {
                const int n = cnt[v * pitch + k];
                cnt[v * pitch + k] = (uint16_t)to;
                to += n;
            }
        }
        sync_block();
        if (tid == T - 1) {
            s_carry = at + run;
            if (c0 + T >= K) starts[K] = (uint16_t)(at + run);
        }
        sync_block();
    }
    uint16_t *list = a.list + (size_t)y * a.ns + r0;
#pragma unroll
    for (int s = 0; s < LOOPS; ++s)
        if (rank[s] >= 0) list[(int)mine[c[s]] + rank[s]] = (uint16_t)((wave * LOOPS + s) * kWave + lane);
}

// A workgroup takes 2^cg_log2 clusters, whose values lie together in every chunk: all threads bring them to the LDS, a piece of
// several chunks at a time, the next piece on its way meanwhile; a thread per (cluster, coordinate) adds them.
// DIM: coordinates, or 0 where they are not known before; VEC: four of them at a time, from memory.
template <int DIM, bool VEC>
__global__ __launch_bounds__(kSumThreads) void kmeans_sums_kernel(const SortArgs a) {
    constexpr int kPer = kSumFloats / kSumThreads, kFly = 8;
    __shared__ __align__(16) float s_vals[2][kSumFloats + kFly * kShortRow];      // (a group of values more)
    __shared__ int s_run[kSumChunks * ((1 << kSumMaxLog2) + 1)];           // [chunk][CG + 1] where the clusters' rows begin, in the workgroup's numbers
    __shared__ int s_off[kSumChunks], s_adj[kSumChunks], s_end[kSumChunks];   // a chunk's: row in memory less number, number less row of the chunk, end
    // an XCD takes neighbouring subspaces, whose columns stay in its L2
    const int groups = (a.K + (1 << a.cg_log2) - 1) >> a.cg_log2, all_wg = groups * a.ny;
    const int per_xcd = (all_wg + kXcds - 1) / kXcds, wg = (int)(blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
    if (wg >= all_wg || (int)(blockIdx.x / kXcds) >= per_xcd) return;
    const int y = wg / groups, CG = 1 << a.cg_log2, c0 = (wg - y * groups) << a.cg_log2, ncl = a.K - c0 < CG ? a.K - c0 : CG;
    const int dim = DIM > 0 ? DIM : a.dim, step = dim, K = a.K, tid = threadIdx.x, lane = tid & (kWave - 1), P = CG + 1;
    constexpr int kPieces = VEC ? kPer / 4 : kPer;                        // of a thread
    const int g = VEC ? dim >> 2 : dim, cap = kSumFloats / dim;           // pieces of a row; rows in the LDS at a time
    const uint32_t inv = 0xffffffffu / (uint32_t)g + 1u;
    const float *src = a.x + (size_t)y * a.xstep;
    const uint16_t *list = a.list + (size_t)y * a.ns;
    const uint16_t *starts = a.starts + (size_t)y * a.nchunk * (K + 1) + c0;
    const int cl = tid / dim, t = tid - cl * dim;
    const bool on = cl < ncl;
    double sum = 0.0;
    int64_t count = 0;
    for (int i0 = 0; i0 < a.nchunk; i0 += kSumChunks) {
        const int nc = a.nchunk - i0 < kSumChunks ? a.nchunk - i0 : kSumChunks;
        sync_block();
        for (int e = tid; e < nc * (ncl + 1); e += kSumThreads) {
            const int i = e / (ncl + 1), c = e - i * (ncl + 1);
            s_run[i * P + c] = starts[(size_t)(i0 + i) * (K + 1) + c];
        }
        sync_block();
        const int first = lane < nc ? s_run[lane * P] : 0, n = lane < nc ? s_run[lane * P + ncl] - first : 0;
        int incl = n;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int o = __shfl_up(incl, off);
            if (lane >= off) incl += o;
        }
        const int total = __builtin_amdgcn_readlane(incl, kWave - 1);      // (the same in every wave)
        if (total == 0) continue;          // (no row to look up: the search below would end behind the last chunk)
        if (tid < kWave) {
            s_off[lane] = (i0 + lane) * a.rows + first - (incl - n);
            s_adj[lane] = incl - n - first;
            s_end[lane] = lane < nc ? incl : 0x7fffffff;
        }
        sync_block();
        for (int e = tid; e < nc * (ncl + 1); e += kSumThreads) {
            const int i = e / (ncl + 1), c = e - i * (ncl + 1);
            s_run[i * P + c] += s_adj[i];
        }
        sync_block();
        float f[kPer];
        int row[kPieces];                  // a piece's rows are known before its values are asked for: in their chunk,
        int from[kPieces];                 // and the chunk's first (added up later: nothing waits for one before the next is asked for)
        auto row_of = [&](int e) { return g == 1 ? e : (int)__umulhi((uint32_t)e, inv); };
        auto look_up = [&](int p0) {
            const int all = (total - p0 < cap ? total - p0 : cap) * g;
#pragma unroll
            for (int u = 0; u < kPieces; ++u) {
                const int e = tid + u * kSumThreads;
                const int r = p0 + row_of(e < all ? e : 0);
                int at = 0;                // the chunk: as many as end before the row
#pragma unroll
                for (int half = kSumChunks / 2; half > 0; half >>= 1) at += s_end[at + half - 1] <= r ? half : 0;
                from[u] = (i0 + at) * a.rows;
                row[u] = list[r + s_off[at]];
            }
        };
        auto load = [&](int p0) {
            const int all = (total - p0 < cap ? total - p0 : cap) * g;
#pragma unroll
            for (int u = 0; u < kPieces; ++u) {
                const int e = tid + u * kSumThreads;
                if (e < all) {
                    const float *at = src + (size_t)(from[u] + row[u]) * a.stride + (VEC ? 4 : 1) * (e - row_of(e) * g);
                    if constexpr (VEC) {
                        const float4 v = *reinterpret_cast<const float4 *>(at);
                        f[4 * u] = v.x; f[4 * u + 1] = v.y; f[4 * u + 2] = v.z; f[4 * u + 3] = v.w;
                    } else {
                        f[u] = *at;
                    }
                }
            }
        };
        auto store = [&](float *to) {       // (what was not loaded goes where nobody looks)
#pragma unroll
            for (int u = 0; u < kPieces; ++u) {
                if constexpr (VEC) reinterpret_cast<float4 *>(to)[tid + u * kSumThreads] = make_float4(f[4 * u], f[4 * u + 1], f[4 * u + 2], f[4 * u + 3]);
                else to[tid + u * kSumThreads] = f[u];
            }
        };
        look_up(0);
        load(0);
        if (cap < total) look_up(cap);
        int i = 0, buf = 0;                // i: the first chunk with rows in the piece or after it
        for (int p0 = 0; p0 < total; p0 += cap, buf ^= 1) {
            store(s_vals[buf]);
            sync_block();
            const int p1 = p0 + cap < total ? p0 + cap : total;
            if (p1 < total) load(p1);
            if (p1 + cap < total) look_up(p1 + cap);
            if (on) {
                // a group of values is on its way while the one before it is added (read past a run's end where the run ends early)
                auto read = [&](const float *v, float (&x)[kFly]) {
#pragma unroll
                    for (int u = 0; u < kFly; ++u) x[u] = v[u * step];
                };
                auto add = [&](const float (&x)[kFly]) {
#pragma unroll
                    for (int u = 0; u < kFly; ++u) sum += (double)x[u];
                };
                int b = s_run[i * P + cl], e = s_run[i * P + cl + 1], end = s_run[i * P + ncl];
                for (;;) {
                    const int lo = b > p0 ? b : p0, hi = e < p1 ? e : p1, here = end;
                    const bool more = i + 1 < nc && here <= p1;            // (else the rest of the chunk, if any, is in the next piece)
                    const int j = more ? i + 1 : i;
                    b = s_run[j * P + cl]; e = s_run[j * P + cl + 1]; end = s_run[j * P + ncl];
                    if (hi > lo) {
                        count += hi - lo;
                        const float *v = s_vals[buf] + (lo - p0) * step + t;
                        float x[kFly], z[kFly];
                        int n = hi - lo;
                        read(v, x);
                        while (n >= kFly) {
                            read(v + kFly * step, z);
                            add(x);
                            v += 2 * kFly * step;
                            if ((n -= kFly) < kFly) {
#pragma unroll
                                for (int u = 0; u < kFly; ++u) x[u] = z[u];
                                break;
                            }
                            read(v, x);
                            add(z);
                            n -= kFly;
                        }
                        // (a value that is not there adds +0, which changes no sum that began with +0)
#pragma unroll
                        for (int u = 0; u < kFly - 1; ++u) sum += (double)(u < n ? x[u] : 0.0f);
                    }
                    i = j;
                    if (!more || here == p1) break;
                }
            }
        }
    }
    if (on && count > 0) a.cent[((size_t)y * K + c0 + cl) * dim + t] = (float)(sum / (double)count);
}

// The rows' sub-vectors side by side, clustering by clustering: [ny][ns][dim].  Once per training: read out of whole rows,
// kmeans_sums_kernel would bring a cache line for every 16 or 32 bytes, in every iteration.  64 rows per workgroup.
__global__ __launch_bounds__(256) void kmeans_columns_kernel(const float *__restrict__ x, int64_t ns, int64_t stride, int dim, int ny,
                                                             float *__restrict__ out) {
    const int64_t r = (int64_t)blockIdx.x * kWave + (threadIdx.x & (kWave - 1));
    if (r >= ns) return;
    const float *row = x + (size_t)r * stride;
    for (int y = threadIdx.x >> 6; y < ny; y += 4) {
        float *to = out + ((size_t)y * ns + r) * dim;
        if ((dim & 3) == 0)
            for (int t = 0; t < dim; t += 4) *reinterpret_cast<float4 *>(to + t) = *reinterpret_cast<const float4 *>(row + (size_t)y * dim + t);
        else
            for (int t = 0; t < dim; ++t) to[t] = row[(size_t)y * dim + t];
    }
}

// One workgroup per (cluster, up to 256 coordinates); grid.y: clusterings.
__global__ __launch_bounds__(kUpdCols) void kmeans_rows_kernel(const SortArgs a) {
    __shared__ int s_rows[kRowsCap], s_part[kUpdCols / kWave], s_end[kUpdCols], s_off[kUpdCols];   // a chunk's last number and one; place in the list less number
    const int nz = (a.dim + kUpdCols - 1) / kUpdCols, c = blockIdx.x / nz, t0 = (blockIdx.x - c * nz) * kUpdCols, y = blockIdx.y;
    const int tid = threadIdx.x, T = blockDim.x, lane = tid & (kWave - 1), wave = tid >> 6, K = a.K;
    const int t = t0 + tid;
    const bool on = t < a.dim;
    const float *x = a.x + (size_t)y * a.xstep + (on ? t : 0);
    const uint16_t *starts = a.starts + (size_t)y * a.nchunk * (K + 1) + c;
    const uint16_t *list = a.list + (size_t)y * a.ns;
    double sum = 0.0;
    int64_t count = 0;
    for (int i0 = 0; i0 < a.nchunk; i0 += T) {          // a chunk per thread
        const int i = i0 + tid;
        int s = 0, n = 0;
        if (i < a.nchunk) {
            s = starts[(size_t)i * (K + 1)];
            n = starts[(size_t)i * (K + 1) + 1] - s;
        }
        int incl = n;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int o = __shfl_up(incl, off);
            if (lane >= off) incl += o;
        }
        if (lane == kWave - 1) s_part[wave] = incl;
        sync_block();
        int before = incl - n, total = 0;
        for (int v = 0; v < T >> 6; ++v) {
            if (v < wave) before += s_part[v];
            total += s_part[v];
        }
        count += total;
        s_end[tid] = before + n;
        s_off[tid] = i * a.rows + s - before;
        sync_block();
        for (int p0 = 0; p0 < total; p0 += kRowsCap) {
            const int np = total - p0 < kRowsCap ? total - p0 : kRowsCap;
            for (int k = tid; k < np; k += T) {
                int at = 0;                    // the chunk: as many as end before
                for (int half = T >> 1; half > 0; half >>= 1) at += s_end[at + half - 1] <= p0 + k ? half : 0;
                s_rows[k] = (i0 + at) * a.rows + list[p0 + k + s_off[at]];
            }
            sync_block();
            float f[kRowsFly], h[kRowsFly];
            auto load = [&](int k, float (&to)[kRowsFly]) {
#pragma unroll
                for (int u = 0; u < kRowsFly; ++u) to[u] = x[(size_t)s_rows[k + u < np ? k + u : np - 1] * a.stride];
            };
            auto add = [&](int k, const float (&from)[kRowsFly]) {
                if (k + kRowsFly <= np) {
#pragma unroll
                    for (int u = 0; u < kRowsFly; ++u) sum += (double)from[u];
                    return;
                }
                // (a value that is not there adds +0, which changes no sum that began with +0)
#pragma unroll
                for (int u = 0; u < kRowsFly; ++u) sum += (double)(k + u < np ? from[u] : 0.0f);
            };
            load(0, f);
            for (int k = 0; k < np; k += 2 * kRowsFly) {
                if (k + kRowsFly < np) load(k + kRowsFly, h);
                add(k, f);
                if (k + kRowsFly >= np) break;
                if (k + 2 * kRowsFly < np) load(k + 2 * kRowsFly, f);
                add(k + kRowsFly, h);
            }
            sync_block();
        }
        sync_block();       // s_part is read
    }
    if (on && count > 0) a.cent[((size_t)y * K + c) * a.dim + t] = (float)(sum / (double)count);
}

}  // namespace trim
