// Kernels around the scan: PQ encode, stand-alone distance tables, range-search output
// assembly, coarse-probe selection, small fills.
#pragma once

#include <type_traits>

#include "trim_device.h"

namespace trim {

// ---- fills (used instead of memset nodes so that callers may capture the stream) ----
__global__ void fill_u32_kernel(uint32_t *p, size_t count, uint32_t v) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// Several areas cleared by one launch (a launch of its own for each costs a small search 3 to 5 us).
struct ZeroAreas {
    static constexpr int kMost = 10;
    uint32_t *at[kMost];
    size_t words[kMost];
    int count = 0;
    void add(void *p, size_t n) {
        if (!p || n == 0) return;
        if (count < kMost) {
            at[count] = static_cast<uint32_t *>(p);
            words[count] = n;
        }
        ++count;             // (more than there is room for: zero_areas refuses)
    }
};
__global__ __launch_bounds__(256) void zero_areas_kernel(const ZeroAreas z) {
    for (int i = 0; i < z.count; ++i)
        for (size_t w = (size_t)blockIdx.x * 256 + threadIdx.x; w < z.words[i]; w += (size_t)gridDim.x * 256) z.at[i][w] = 0u;
}

// ---- ceilings of the machine for the two resources the scan leans on (measurement aids) ----
// Streaming read: every 16-byte piece of the buffer is read once, four loads in flight per
// thread; the xor of everything read goes to sink[block] so that the loads cannot be dropped.
__global__ __launch_bounds__(512) void stream_read_kernel(const uint4 *__restrict__ p, size_t n16,
                                                          uint32_t *__restrict__ sink) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint32_t acc = 0;
    for (; i + 3 * stride < n16; i += 4 * stride) {
        const uint4 a = p[i], b = p[i + stride], c = p[i + 2 * stride], e = p[i + 3 * stride];
        acc ^= a.x ^ a.y ^ a.z ^ a.w ^ b.x ^ b.y ^ b.z ^ b.w ^ c.x ^ c.y ^ c.z ^ c.w ^ e.x ^ e.y ^ e.z ^ e.w;
    }
    for (; i < n16; i += stride) {
        const uint4 a = p[i];
        acc ^= a.x ^ a.y ^ a.z ^ a.w;
    }
    for (int off = 32; off > 0; off >>= 1) acc ^= __shfl_xor(acc, off);
    __shared__ uint32_t part[8];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    sync_block();
    if (threadIdx.x == 0) {
        uint32_t r = 0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) r ^= part[w];
        sink[blockIdx.x] = r;
    }
}

// Table gathers: the inner step of the scan and nothing else.  Each lane owns 32 code bytes
// (8 words) and sums, per iteration, the 32 entries T[j][byte j] of a [32][256] binary32 table
// in LDS with the scan's own gather routine; the code words are stirred between iterations so
// that the reads stay random.  gathers = grid * 512 * iters * 32.
__global__ __launch_bounds__(512) void lds_gather_kernel(int iters, uint32_t seed,
                                                         float *__restrict__ sink) {
    extern __shared__ __align__(16) unsigned char smem[];
    float *tab = reinterpret_cast<float *>(smem);  // [32][256]
    for (int i = threadIdx.x; i < 32 * kC; i += blockDim.x) tab[i] = (float)((i * 2654435761u) >> 20);
    sync_block();
    const uint32_t tab_base = lds_addr(tab);
    uint32_t w[8];
    uint32_t h = seed ^ ((blockIdx.x * 512u + threadIdx.x) * 0x9e3779b9u);
#pragma unroll
    for (int v = 0; v < 8; ++v) {
        h ^= h << 13; h ^= h >> 17; h ^= h << 5;
        w[v] = h;
    }
    float s = 0.0f;
    for (int it = 0; it < iters; ++it) {
        const uint32_t lo[4] = {w[0], w[1], w[2], w[3]};
        const uint32_t hi[4] = {w[4], w[5], w[6], w[7]};
        s = gather_add<4>(s, tab_base, lo, __builtin_inff());
        s = gather_add<4>(s, tab_base + 16 * kC * 4, hi, __builtin_inff());
        const uint32_t t = w[0];
#pragma unroll
        for (int v = 0; v < 7; ++v) w[v] = w[v + 1];
        w[7] = (t << 7 | t >> 25) ^ (uint32_t)it;
    }
    sink[(size_t)blockIdx.x * blockDim.x + threadIdx.x] = s;
}

// The same for 4-bit codes: a [64][16] table (32 code bytes of two subspaces each); every lane
// sums, per iteration, the 64 entries its 32 code bytes select, with the scan's own routine.
// A row of 16 consecutive words spans 16 banks, so these lookups never collide: this is also the
// rate of conflict-free 4-byte LDS reads.  lookups = grid * 512 * iters * 64.
__global__ __launch_bounds__(512) void lds_gather_fs_kernel(int iters, uint32_t seed,
                                                            float *__restrict__ sink) {
    extern __shared__ __align__(16) unsigned char smem[];
    float *tab = reinterpret_cast<float *>(smem);  // [64][16]
    for (int i = threadIdx.x; i < 64 * kC4; i += blockDim.x) tab[i] = (float)((i * 2654435761u) >> 20);
    sync_block();
    const uint32_t tab_base = lds_addr(tab);
    uint32_t w[8];
    uint32_t h = seed ^ ((blockIdx.x * 512u + threadIdx.x) * 0x9e3779b9u);
#pragma unroll
    for (int v = 0; v < 8; ++v) {
        h ^= h << 13; h ^= h >> 17; h ^= h << 5;
        w[v] = h;
    }
    float s = 0.0f;
    for (int it = 0; it < iters; ++it) {
        const uint32_t lo[4] = {w[0], w[1], w[2], w[3]};
        const uint32_t hi[4] = {w[4], w[5], w[6], w[7]};
        s = gather_add<4, false, true>(s, tab_base, lo, __builtin_inff());
        s = gather_add<4, false, true>(s, tab_base + 16 * kByteRow<true>, hi, __builtin_inff());
        const uint32_t t = w[0];
#pragma unroll
        for (int v = 0; v < 7; ++v) w[v] = w[v + 1];
        w[7] = (t << 7 | t >> 25) ^ (uint32_t)it;
    }
    sink[(size_t)blockIdx.x * blockDim.x + threadIdx.x] = s;
}

// The same with entries of W binary32 values (W = 2, 4: what a table shared by W queries would
// hold): 8 rows of 256 entries, every thread performs iters * 8 lookups of one whole entry and
// adds its W values up.
template <int W>
__global__ __launch_bounds__(512) void lds_gather_wide_kernel(int iters, uint32_t seed,
                                                              float *__restrict__ sink) {
    extern __shared__ __align__(16) unsigned char smem[];
    float *tab = reinterpret_cast<float *>(smem);  // [8][256][W]
    for (int i = threadIdx.x; i < 8 * kC * W; i += blockDim.x) tab[i] = (float)(i & 1023);
    sync_block();
    uint32_t h = seed ^ ((blockIdx.x * 512u + threadIdx.x) * 0x9e3779b9u);
    h ^= h << 13; h ^= h >> 17; h ^= h << 5;
    uint32_t w0 = h;
    h ^= h << 13; h ^= h >> 17; h ^= h << 5;
    uint32_t w1 = h;
    float s = 0.0f;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t c = ((j < 4 ? w0 : w1) >> (8 * (j & 3))) & 255u;
            const float *e = tab + (j * kC + c) * W;
            if (W == 2) {
                const float2 v = *reinterpret_cast<const float2 *>(e);
                s += v.x; s += v.y;
            } else {
                const float4 v = *reinterpret_cast<const float4 *>(e);
                s += v.x; s += v.y; s += v.z; s += v.w;
            }
        }
        const uint32_t t = w0;
        w0 = w1;
        w1 = (t << 7 | t >> 25) ^ (uint32_t)it;
    }
    sink[(size_t)blockIdx.x * blockDim.x + threadIdx.x] = s;
}

// ---- per-list summaries for list-level pruning (record layout: list_record_bytes) ----
// One workgroup per inverted list: a presence bitmap of 256 bits per subspace is filled from
// the list's codes, then one wave per subspace writes the set codes in ascending order.
// A thread takes four code bytes at a time, neighbouring threads neighbouring ones, and sets a bit only where it is not set yet: a
// list holds some twenty codes per subspace, so that nearly always it is.  The longest list decides (lists of twenty
// times the mean length are usual): 1024 threads, 16 looks at the bitmap under way together; 256 for many short lists (see
// trim_pack_list_bounds).  1,000,000 x 32 in 1024 lists: 102 -> 39 us.
constexpr int kBoundsPitch = 9;      // words per subspace, one of them spare (bank spread)
template <int T>
__global__ __launch_bounds__(T) void list_bounds_kernel(const uint8_t *__restrict__ codes,
                                                          const float *__restrict__ dlx, int64_t n,
                                                          int M, const int64_t *__restrict__ list_offsets,
                                                          uint8_t *__restrict__ out) {
    extern __shared__ __align__(16) unsigned char smem[];
    uint32_t *bits = reinterpret_cast<uint32_t *>(smem);  // [M][kBoundsPitch]
    __shared__ float red[T / kWave];
    const int l = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    uint8_t *rec = out + (size_t)l * list_record_bytes(M);
    for (int i = tid; i < M * kBoundsPitch; i += T) bits[i] = 0;
    int64_t lo = list_offsets[l], hi = list_offsets[l + 1];
    lo = lo < 0 ? 0 : (lo > n ? n : lo);
    hi = hi < lo ? lo : (hi > n ? n : hi);
    float bmax = 0.0f;
    for (int64_t x = lo + tid; x < hi; x += T) bmax = fmaxf(bmax, dlx[x]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) bmax = fmaxf(bmax, __shfl_xor(bmax, off));
    if (lane == 0) red[tid >> 6] = bmax;
    sync_block();
    if (tid == 0) {
        for (int w = 1; w < T / kWave; ++w) bmax = fmaxf(bmax, red[w]);
        *reinterpret_cast<float *>(rec + list_record_bmax_offset(M)) = bmax;
    }
    const uint32_t *words = reinterpret_cast<const uint32_t *>(codes + (size_t)lo * M);     // (M % 4 == 0, the codes are aligned)
    const int per = M / 4;
    const int64_t all = (hi - lo) * per;
    constexpr int kFly = 4;
    for (int64_t e = tid; e < all; e += kFly * T) {
        uint32_t w[kFly], have[4 * kFly];
        int j[kFly];
#pragma unroll
        for (int u = 0; u < kFly; ++u) {
            const int64_t at = e + u * T < all ? e + u * T : e;
            w[u] = words[at];
            j[u] = 4 * (int)(at % per);
        }
#pragma unroll
        for (int i = 0; i < 4 * kFly; ++i) have[i] = bits[(j[i >> 2] + (i & 3)) * kBoundsPitch + (w[i >> 2] >> (8 * (i & 3) + 5) & 7u)];
#pragma unroll
        for (int i = 0; i < 4 * kFly; ++i) {
            const uint32_t c = w[i >> 2] >> (8 * (i & 3)) & 255u;
            if (!(have[i] >> (c & 31) & 1u)) atomicOr(&bits[(j[i >> 2] + (i & 3)) * kBoundsPitch + (c >> 5)], 1u << (c & 31));
        }
    }
    sync_block();
    for (int j = tid >> 6; j < M; j += T >> 6) {   // one wave per subspace
        const uint32_t nib = (bits[j * kBoundsPitch + (lane >> 3)] >> ((lane & 7) * 4)) & 15u;  // codes 4*lane..4*lane+3
        const int cnt = __popc(nib);
        int incl = cnt;                                  // inclusive prefix over the lanes
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_up(incl, off);
            if (lane >= off) incl += v;
        }
        const int total = __shfl(incl, 63);
        uint8_t *row = rec + (size_t)j * kSetCap;
        if (total == 0 || total > kSetCap) {
            row[lane] = 0;
            if (lane == 0) rec[(size_t)M * kSetCap + j] = total == 0 ? 0 : (uint8_t)kSetAny;
            continue;
        }
        const unsigned long long have = __ballot(nib != 0);
        const int fl = __ffsll((long long)have) - 1;
        const uint32_t fn = (uint32_t)__shfl((int)nib, fl);
        const uint8_t first = (uint8_t)(4 * fl + (__ffs((int)fn) - 1));
        if (lane >= total) row[lane] = first;            // padding
        int at = incl - cnt;
        for (int b = 0; b < 4; ++b)
            if ((nib >> b) & 1u) row[at++] = (uint8_t)(4 * lane + b);
        if (lane == 0) rec[(size_t)M * kSetCap + j] = (uint8_t)total;
    }
}

// ---- scan head: {code bytes 0..7, landmark distance} of every vector as one 12-byte record ----
__global__ void pack_scan_head_kernel(const uint8_t *__restrict__ codes, const float *__restrict__ dlx,
                                      int64_t n, int M, uint32_t *__restrict__ head) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const uint2 c = *reinterpret_cast<const uint2 *>(codes + (size_t)i * M);  // M % 8 == 0
        head[3 * i + 0] = c.x;
        head[3 * i + 1] = c.y;
        head[3 * i + 2] = __float_as_uint(dlx[i]);
    }
}

// ---- tiled codes: blocks of 64 vectors, 16-byte pieces of a block's vectors contiguous ----
// One thread per (vector slot, piece); slots beyond n are written as zeros.
__global__ void pack_codes_tiled_kernel(const uint8_t *__restrict__ codes, int64_t n, int M,
                                        uint4 *__restrict__ tiled) {
    const int npiece = M >> 4;
    const int64_t total = ((n + 63) / 64) * 64 * npiece;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
         t += (int64_t)gridDim.x * blockDim.x) {
        // t enumerates the output in order: block, piece, lane
        const int lane = (int)(t & 63);
        const int64_t bp = t >> 6;
        const int piece = (int)(bp % npiece);
        const int64_t x = (bp / npiece) * 64 + lane;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (x < n) v = *reinterpret_cast<const uint4 *>(codes + (size_t)x * M + piece * 16);
        tiled[t] = v;
    }
}

// ---- centroid training (Lloyd's k-means; Sections 2.2, 3.1, 6.1) ----
// Initial centroids: cent[y][c][t] = x[init_rows[c]][y*dim + t]; grid.y = clusterings (PQ subspaces).
__global__ void kmeans_init_kernel(const float *__restrict__ x, int64_t ns, int64_t stride, int dim,
                                   const int32_t *__restrict__ init_rows, int K, float *__restrict__ cent) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= K * dim) return;
    int64_t r = init_rows[e / dim];
    r = r < 0 ? 0 : (r >= ns ? ns - 1 : r);
    cent[(size_t)blockIdx.y * K * dim + e] = x[(size_t)r * stride + (size_t)blockIdx.y * dim + e % dim];
}

// Update step with every rounding fixed: for cluster c and coordinate t the float64 sum, in
// ascending row order, of that coordinate over the rows assigned to c; the centroid becomes
// sum / count rounded once to binary32; a cluster without rows keeps its centroid.
// Assignments are bytes (ABYTES = 1) or 32-bit integers (ABYTES = 4); clustering y (a PQ subspace) uses the elements
// assign[row * astride + y * ystride], columns y*dim.., centroid block y.
//
// A workgroup serves 2^cg_log2 clusters.  Its rows are found first: kUpdChunk assignments at a time are looked at, 16
// consecutive rows per lane, and the rows of its clusters are appended to a list, in row order.  The
// list, some 1/8 of the rows, is put in cluster order by a stable counting sort (ranks
// inside a wave by matching ballots, wave offsets through LDS) when it is full or the rows are through; then a thread per
// (cluster, coordinate) adds its rows, straight from memory where that is work for 256 threads and more (long rows),
// else from LDS, where all threads bring the rows found together.
// (Sorting the assignments chunk by chunk ranked all of them in every workgroup.)  65,536 rows, 32 x 256 x 4 coordinates: 59 us
// an iteration (134), 1024 x 128 coordinates: 38 .. 65 us by the largest cluster (72).  Bound by short steps one after
// the other, one workgroup per CU by its list and what sorting it holds in registers; about half of it is bringing the rows: 16 bytes of
// every cache line.  Up to kUpdFew rows leave room for two per CU: 96 x 256 x 8 coordinates, 4 iterations of training, 300
// rows 183 -> 129 us, 4000 258 -> 198, 8000 401 -> 327.
constexpr int kUpdThreads = 512, kUpdRows = 16, kUpdChunk = kUpdThreads * kUpdRows;
constexpr int kUpdMaxLog2 = 5;
constexpr int kUpdList = 16384, kUpdFew = 8192;   // rows found (there is room for kUpdFew where there are no more at all)
constexpr int kUpdVals = 8192, kUpdPiece = 2048;   // row values, rows in LDS at a time
constexpr int kUpdCols = 256;    // coordinates per workgroup at most (grid: slices of that many)
static_assert(kUpdList >= kUpdChunk && kUpdFew <= kUpdChunk, "a chunk's rows fit the list");
__host__ __device__ inline bool kmeans_update_direct(int cg_log2, int cols) { return (cols << cg_log2) >= 256; }
// list, vals: how many rows, values there is room for
inline size_t kmeans_update_lds(int cg_log2, int cols, int list, int vals) {
    return ((size_t)cols << cg_log2) * 8 + (size_t)list * 4 + (kmeans_update_direct(cg_log2, cols) ? 0 : (size_t)vals * 4 + kUpdPiece * 2) + (((size_t)kUpdThreads / kWave + 2) * 4 << cg_log2) + 16 + kUpdThreads / kWave * 4;
}
struct UpdateArgs {
    const float *x;            // [ns][stride]
    const void *assign;
    int64_t ns, stride, astride, ystride;
    int32_t dim, K, cg_log2, groups, ny, total;     // total: workgroups that have work
    int32_t vals;              // kUpdVals, or what fewer rows can fill
    float *cent;
};
template <int ABYTES, int LIST>
__global__ __launch_bounds__(kUpdThreads, LIST < kUpdList ? 4 : 1) void kmeans_update_kernel(const UpdateArgs a) {
    constexpr int kWaves = kUpdThreads / kWave;
    extern __shared__ __align__(16) unsigned char smem[];
    const int CG = 1 << a.cg_log2, dim = a.dim;
    // an XCD takes neighbouring subspaces: their columns share cache lines
    const int per_xcd = (a.total + kXcds - 1) / kXcds, w = (int)(blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
    if (w >= a.total || (int)(blockIdx.x / kXcds) >= per_xcd) return;
    const int group = w % a.groups, y = w / a.groups % a.ny, t0 = w / a.groups / a.ny * kUpdCols;
    const int cols = dim - t0 < kUpdCols ? dim - t0 : kUpdCols;
    float *vals = reinterpret_cast<float *>(smem);                         // [rows][cols]
    // (the last slice of columns may be narrower than the others: the launch's layout is that of the first)
    const bool direct = kmeans_update_direct(a.cg_log2, dim < kUpdCols ? dim : kUpdCols);
    double *sums = reinterpret_cast<double *>(vals + (direct ? 0 : a.vals));     // [CG][cols]
    uint32_t *list = reinterpret_cast<uint32_t *>(sums + (size_t)CG * cols);     // [LIST] row << 5 | cluster, direct: then rows by cluster
    int *wcount = reinterpret_cast<int *>(list + LIST);                    // [kWaves][CG]
    int *rows_of = wcount + kWaves * CG;                                   // [CG] rows per cluster so far
    int *start = rows_of + CG;                                             // [CG + 1] runs of list[]
    int *part = start + CG + 4;                                            // [kWaves]
    uint16_t *place = reinterpret_cast<uint16_t *>(part + kWaves);         // [kUpdPiece] in cluster order (not direct)
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int c_first = group << a.cg_log2, wave_id = __builtin_amdgcn_readfirstlane(wave);
    const float *x = a.x + (size_t)y * dim + t0;
    float *cent = a.cent + (size_t)y * a.K * dim + t0;
    for (int e = tid; e < CG * cols; e += kUpdThreads) sums[e] = 0.0;
    for (int c = tid; c < CG; c += kUpdThreads) rows_of[c] = 0;
    int *mine = wcount + wave * CG;
    const unsigned long long below = (1ull << lane) - 1ull;
    const bool vec = ((cols | dim) & 3) == 0 && (a.stride & 3) == 0 && (reinterpret_cast<uintptr_t>(a.x) & 15u) == 0;
    int64_t row0 = 0;        // the list's rows are relative to this one
    int found = 0;           // (the same for all threads)
    // Places in cluster order of the entries list[p0 .. p1), by a stable counting sort: f(entry of the list, what it holds, its
    // place), start[] the clusters' first places.  Barriers before and after.
    auto sort_rows = [&](int p0, int p1, auto loops, auto &&f) {
        constexpr int kLoops = decltype(loops)::value;
        uint32_t mem[kLoops];
        int rank[kLoops];
        const int seg = ((p1 - p0 + kWaves - 1) / kWaves + kWave - 1) / kWave * kWave, s0 = p0 + wave * seg;
        for (int c = lane; c < CG; c += kWave) mine[c] = 0;
#pragma unroll
        for (int s = 0; s < kLoops; ++s) mem[s] = s * kWave < seg && s0 + s * kWave + lane < p1 ? list[s0 + s * kWave + lane] : 0u;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int s = 0; s < kLoops; ++s) {
            rank[s] = -1;
            if (s * kWave >= seg || s0 + s * kWave >= p1) continue;      // same for the wave
            const bool in = s0 + s * kWave + lane < p1;
            const int c = (int)(mem[s] & 31u);
            unsigned long long same = __ballot(in);
            for (int b = 0; b < a.cg_log2; ++b) {
                const bool bit = (c >> b) & 1;
                const unsigned long long m = __ballot(bit);
                same &= bit ? m : ~m;
            }
            const int before = __popcll(same & below);
            if (in) rank[s] = mine[c] + before;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (in && before == 0) mine[c] += __popcll(same);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        sync_block();
        if (wave == 0) {                                 // counts -> first slots
            int n[kWaves], run = 0;
#pragma unroll
            for (int v = 0; v < kWaves; ++v) n[v] = lane < CG ? wcount[v * CG + lane] : 0;
#pragma unroll
            for (int v = 0; v < kWaves; ++v) { const int k = n[v]; n[v] = run; run += k; }
            int incl = run;
#pragma unroll
            for (int off = 1; off < 1 << kUpdMaxLog2; off <<= 1) {
                const int v = __shfl_up(incl, off);
                if (lane >= off) incl += v;
            }
            if (lane < CG) {
                rows_of[lane] += run;
                start[lane] = incl - run;
                if (lane == CG - 1) start[CG] = incl;
#pragma unroll
                for (int v = 0; v < kWaves; ++v) wcount[v * CG + lane] = n[v] + incl - run;
            }
        }
        sync_block();
#pragma unroll
        for (int s = 0; s < kLoops; ++s)
            if (rank[s] >= 0) f(s0 + s * kWave + lane, mem[s], mine[mem[s] & 31u] + rank[s]);
        sync_block();
    };
    // the rows in list[0 .. found) are added
    auto add_rows = [&]() {
        const float *xi = x + (size_t)row0 * a.stride;
        if (direct) {
            sort_rows(0, found, std::integral_constant<int, LIST / kUpdThreads>(), [&](int, uint32_t m, int at) { list[at] = m >> 5; });
            for (int e = tid; e < CG * cols; e += kUpdThreads) {
                const int c = e / cols;
                const float *xt = xi + (e - c * cols);
                int i = start[c];
                const int end = start[c + 1];
                if (i >= end) continue;
                double sum = sums[e];
                constexpr int kFly = LIST < kUpdList ? 16 : 32;       // loads in flight
                for (; i < end; i += kFly) {
                    float v[kFly];
#pragma unroll
                    for (int u = 0; u < kFly; ++u) v[u] = xt[(size_t)list[i + u < end ? i + u : i] * a.stride];
#pragma unroll
                    for (int u = 0; u < kFly; ++u)
                        if (i + u < end) sum += (double)v[u];
                }
                sums[e] = sum;
            }
            sync_block();
            return;
        }
        // Short rows: read in row order, so that workgroups of neighbouring subspaces, whose columns share cache lines, read a
        // line at about the same time, and that all clusters have something to add in a piece; stored in cluster order.
        const int piece = a.vals / cols < kUpdPiece ? a.vals / cols : kUpdPiece;
        for (int p0 = 0; p0 < found; p0 += piece) {
            const int p1 = p0 + piece < found ? p0 + piece : found;
            sort_rows(p0, p1, std::integral_constant<int, kUpdPiece / kUpdThreads>(), [&](int i, uint32_t, int at) { place[i - p0] = (uint16_t)at; });
            const int g4 = vec ? cols >> 2 : cols, all = (p1 - p0) * g4;
            for (int e0 = tid; e0 < all; e0 += 4 * kUpdThreads) {
                float4 v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int e = e0 + u * kUpdThreads < all ? e0 + u * kUpdThreads : e0, i = e / g4;
                    const float *at = xi + (size_t)(list[p0 + i] >> 5) * a.stride;
                    if (vec) v[u] = *reinterpret_cast<const float4 *>(at + 4 * (e - i * g4));
                    else v[u].x = at[e - i * g4];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int e = e0 + u * kUpdThreads, i = e / g4;
                    if (e >= all) continue;
                    float *to = vals + (int)place[i] * cols;
                    if (vec) *reinterpret_cast<float4 *>(to + 4 * (e - i * g4)) = v[u];
                    else to[e - i * g4] = v[u].x;
                }
            }
            sync_block();
            for (int e = tid; e < CG * cols; e += kUpdThreads) {
                const int c = e / cols, t = e - c * cols;
                int i = start[c];
                const int hi = start[c + 1];
                if (i >= hi) continue;
                double sum = sums[e];
                const float *v = vals + t + i * cols;
                // (16 values on their way before the first is added: one by one an addition took 110 clocks)
                constexpr int kFly = 16;
                float f[kFly];
                for (; i + kFly <= hi; i += kFly) {
#pragma unroll
                    for (int u = 0; u < kFly; ++u) { f[u] = *v; v += cols; }
#pragma unroll
                    for (int u = 0; u < kFly; ++u) sum += (double)f[u];
                }
                for (; i < hi; ++i, v += cols) sum += (double)*v;
                sums[e] = sum;
            }
            sync_block();
        }
    };
    constexpr int kWords = 4 * ABYTES;
    const unsigned char *assign = static_cast<const unsigned char *>(a.assign) + (size_t)y * a.ystride * ABYTES;
    uint32_t next[kWords];       // the assignments of this lane's rows of a chunk
    auto load_chunk = [&](int64_t i0) {
        const int64_t r0 = i0 + tid * kUpdRows;
        if (a.astride == 1 && i0 + kUpdChunk <= a.ns) {
            __builtin_memcpy(next, assign + (size_t)r0 * ABYTES, sizeof(next));
            return;
        }
#pragma unroll
        for (int i = 0; i < kWords; ++i) next[i] = 0;
#pragma unroll
        for (int i = 0; i < kUpdRows; ++i) {
            const size_t e = (size_t)(r0 + i < a.ns ? r0 + i : a.ns - 1) * a.astride;      // (not counted past the end)
            if constexpr (ABYTES == 1) next[i / 4] |= (uint32_t)assign[e] << (8 * (i & 3));
            else next[i % kWords] = reinterpret_cast<const uint32_t *>(assign)[e];
        }
    };
    const uint32_t pattern = (uint32_t)c_first * 0x01010101u, group_bits = (uint32_t)(0xff & ~(CG - 1)) * 0x01010101u;
    load_chunk(0);
    sync_block();
    for (int64_t i0 = 0; i0 < a.ns; i0 += kUpdChunk) {
        uint32_t w[kWords], in = 0;               // this lane's rows: assignments, and a bit for each of the group's
#pragma unroll
        for (int i = 0; i < kWords; ++i) {
            w[i] = next[i];
            if constexpr (ABYTES == 1) {          // four bytes at a time: a byte's top bit is set where it is in the group
                const uint32_t v = (w[i] ^ pattern) & group_bits;
                const uint32_t hit = ~(((v & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v | 0x7f7f7f7fu);
                in |= ((hit >> 7) * 0x01020408u >> 24) << (4 * i);
            } else {
                in |= (w[i] - (uint32_t)c_first < (uint32_t)CG ? 1u : 0u) << i;
            }
        }
        const int64_t left = a.ns - i0 - tid * kUpdRows;
        in &= left >= kUpdRows ? 0xffffu : left > 0 ? (1u << left) - 1u : 0u;
        if (i0 + kUpdChunk < a.ns) load_chunk(i0 + kUpdChunk);
        const uint32_t cnt = (uint32_t)__popc(in);
        int lower = 0, total = 0;                 // rows of the lanes below, of the wave
#pragma unroll
        for (int b = 0; b < 5; ++b) {
            const unsigned long long m = __ballot(cnt >> b & 1u);
            lower += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)) << b;
            total += __popcll(m) << b;
        }
        if (lane == 0) part[wave] = total;
        sync_block();
        int n = part[lane & (kWaves - 1)];        // the waves' prefix, in every wave
        int incl = n;
#pragma unroll
        for (int off = 1; off < kWaves; off <<= 1) {
            const int v = __shfl_up(incl, off, kWaves);
            if ((lane & (kWaves - 1)) >= off) incl += v;
        }
        const int before = __builtin_amdgcn_readlane(incl - n, wave_id), all = __builtin_amdgcn_readlane(incl, kWaves - 1);
        for (bool fits = false; !fits;) {         // (once; twice where the rows before these have to be added first)
            fits = found + all <= LIST && i0 - row0 <= (int64_t(1) << 26);      // (a row takes 27 bits of an entry)
            if (fits) {
                int to = found + before + lower;
                const uint32_t r = (uint32_t)(i0 - row0) + tid * kUpdRows;
                while (in) {
                    const int i = __ffs((int)in) - 1;
                    in &= in - 1;
                    uint32_t c = 0;
                    if constexpr (ABYTES == 1) {
                        const uint32_t v = i & 8 ? (i & 4 ? w[3] : w[2]) : (i & 4 ? w[1] : w[0]);
                        c = v >> (8 * (i & 3));
                    } else {
#pragma unroll
                        for (int k = 0; k < kWords; ++k) c = k == i ? w[k] : c;
                        c -= (uint32_t)c_first;
                    }
                    list[to++] = (r + i) << 5 | (c & (uint32_t)(CG - 1));
                }
                found += all;
                sync_block();
            }
            if (!fits || i0 + kUpdChunk >= a.ns) {
                if (found > 0) add_rows();
                found = 0;
                row0 = i0;
            }
        }
    }
    for (int e = tid; e < CG * cols; e += kUpdThreads) {
        const int c = e / cols;
        if (c_first + c < a.K && rows_of[c] > 0)
            cent[(size_t)(c_first + c) * dim + (e - c * cols)] = (float)(sums[e] / (double)rows_of[c]);
    }
}

// ---- gamma from a confidence level p (Section 3.2), empirical route ----
// A workgroup takes kGammaRows (2; 1 where the values of two do not fit the LDS) sampled data vectors x: landmark l = PQ reconstruction of x; for
// every sampled query the value 1 - cos(x - l, q - l); the value of the given rank is gamma_x;
// the global gamma is the minimum over x (values are >= 0, so their bit patterns order like
// the numbers and a 32-bit atomic minimum does it).
// Bound by the vector ALU: three operations per coordinate, vector and query, plus the sums over
// lanes.  A half wave measures eight queries (one 16-byte group of each per lane and step, eight
// loads in flight) against both vectors and reduces the 32 lane sums together (reduce_pairs).
// The rank is found by histogram, not by sorting: see below.  1000 vectors x 10,000 queries x
// 128: 0.26 ms (2.46 with one vector per workgroup and a bitonic sort of 16,384 values: 105 passes
// over the LDS, 8 waves per CU).
constexpr int kGammaThreads = 1024, kGammaBins = 2048;
struct GammaArgs {
    const float *base;
    const uint8_t *codes;
    const float *codebooks;
    const int32_t *rows;
    const float *queries;
    int64_t n;
    int32_t S, d, M, Q, rank;
    float *gamma_x;
    uint32_t *gamma_bits;
};
// (the bins take the place of the vectors once the values are there)
__host__ __device__ inline size_t gamma_keys_offset(int rows, int d) {
    const size_t v = (size_t)rows * 2 * d * 4;
    return v > kGammaBins * 4 ? v : kGammaBins * 4;
}
inline size_t gamma_lds(int rows, int d, int Q) { return gamma_keys_offset(rows, d) + (size_t)rows * Q * 4; }

// Bits of a binary32 value in an order-preserving form, and back.
__device__ __forceinline__ uint32_t ordered_bits(float v) {
    const uint32_t b = __float_as_uint(v);
    return b & 0x80000000u ? ~b : b | 0x80000000u;
}
__device__ __forceinline__ float from_ordered_bits(uint32_t k) {
    return __uint_as_float(k & 0x80000000u ? k & 0x7fffffffu : ~k);
}

// One 16-byte group of a query against l and u = x - l: w = q - l, dot += w.u, nn += w.w.
__device__ __forceinline__ void gamma_step(const float4 &q, const float4 &l, const float4 &u, float &dot, float &nn) {
    float w;
    w = q.x - l.x; dot = __builtin_fmaf(w, u.x, dot); nn = __builtin_fmaf(w, w, nn);
    w = q.y - l.y; dot = __builtin_fmaf(w, u.y, dot); nn = __builtin_fmaf(w, w, nn);
    w = q.z - l.z; dot = __builtin_fmaf(w, u.z, dot); nn = __builtin_fmaf(w, w, nn);
    w = q.w - l.w; dot = __builtin_fmaf(w, u.w, dot); nn = __builtin_fmaf(w, w, nn);
}
__device__ __forceinline__ uint32_t gamma_key(float dot, float nn, float nu) {
    const float den = trim::sqrt_rn(nn) * nu;
    return ordered_bits(1.0f - (den > 0.0f ? dot / den : 0.0f));
}
__device__ __forceinline__ void gamma_store(const GammaArgs &a, int64_t s, uint32_t key) {
    const float g = from_ordered_bits(key);
    if (a.gamma_x) a.gamma_x[s] = g;
    atomicMin(a.gamma_bits, __float_as_uint(g < 0.0f ? 0.0f : g));
}

// The key of a rank, by all T threads of a workgroup (hist: kGammaBins counts of LDS): the keys in [lo, hi] are counted
// in at most kGammaBins equal bins of integer width, the bin that holds the rank becomes the new [lo, hi] (its
// smallest and largest key).  The range shrinks at least a thousandfold per round, so three
// rounds are the most; two is usual.
template <int T>
__device__ uint32_t key_of_rank(const uint32_t *keys, int count, int rank, int *hist) {
    constexpr int kPer = kGammaBins / T;
    __shared__ uint32_t s_lo, s_hi, s_bin;
    __shared__ int s_rank;
    __shared__ int part[T / kWave];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    if (tid == 0) { s_lo = 0xffffffffu; s_hi = 0u; s_rank = rank; }
    sync_block();
    uint32_t mn = 0xffffffffu, mx = 0u;
    for (int i = tid; i < count; i += T) { const uint32_t k = keys[i]; mn = k < mn ? k : mn; mx = k > mx ? k : mx; }
    atomicMin(&s_lo, mn);
    atomicMax(&s_hi, mx);
    sync_block();
    uint32_t lo = s_lo, hi = s_hi;
    while (lo < hi) {
        const int bits = 32 - __builtin_clz(hi - lo);
        const int sh = bits > 11 ? bits - 11 : 0;      // (hi - lo) >> sh < 2048
        for (int b = tid; b < kGammaBins; b += T) hist[b] = 0;
        sync_block();
        for (int i = tid; i < count; i += T) {
            const uint32_t k = keys[i];
            if (k >= lo && k <= hi) atomicAdd(&hist[(k - lo) >> sh], 1);
        }
        sync_block();
        // the bin of the rank: a few bins per thread, prefix over the lanes, then over the waves
        int h[kPer], sum = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) { h[i] = hist[kPer * tid + i]; sum += h[i]; }
        int incl = sum;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int v = __shfl_up(incl, off);
            if (lane >= off) incl += v;
        }
        if (lane == kWave - 1) part[wave] = incl;
        const int want = s_rank;
        sync_block();
        int before = incl - sum;
        for (int w = 0; w < wave; ++w) before += part[w];
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            if (want >= before && want < before + h[i]) { s_bin = kPer * tid + i; s_rank = want - before; s_lo = 0xffffffffu; s_hi = 0u; }
            before += h[i];
        }
        sync_block();
        const uint32_t bin = s_bin;
        for (int i = tid; i < count; i += T) {
            const uint32_t k = keys[i];
            if (k >= lo && k <= hi && (k - lo) >> sh == bin) { atomicMin(&s_lo, k); atomicMax(&s_hi, k); }
        }
        sync_block();
        lo = s_lo;
        hi = s_hi;
    }
    sync_block();
    return lo;
}

template <int kGammaRows>
__global__ __launch_bounds__(kGammaThreads) void gamma_kernel(const GammaArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    float *lu = reinterpret_cast<float *>(smem);                               // [rows][2][d]: l, x - l
    uint32_t *keys = reinterpret_cast<uint32_t *>(smem + gamma_keys_offset(kGammaRows, a.d));  // [rows][Q], order-preserving bits
    int *hist = reinterpret_cast<int *>(smem);      // [kGammaBins]
    __shared__ float norm2[kGammaRows];
    __shared__ int part[kGammaThreads / kWave];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int s0 = blockIdx.x * kGammaRows;
    const int dsub = a.d / a.M;
    if (tid < kGammaRows) norm2[tid] = 0.0f;
    sync_block();
#pragma unroll
    for (int x = 0; x < kGammaRows; ++x) {
        int64_t r = a.rows[s0 + x < a.S ? s0 + x : s0];
        r = r < 0 ? 0 : (r >= a.n ? a.n - 1 : r);
        float p = 0.0f;
        for (int t = tid; t < a.d; t += kGammaThreads) {
            const int j = t / dsub;
            const float lt = a.codebooks[((size_t)j * kC + a.codes[(size_t)r * a.M + j]) * dsub + t % dsub];
            const float ut = a.base[(size_t)r * a.d + t] - lt;
            lu[(2 * x) * a.d + t] = lt;
            lu[(2 * x + 1) * a.d + t] = ut;
            p = __builtin_fmaf(ut, ut, p);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) p += __shfl_xor(p, off);
        if (lane == 0) part[wave] = __float_as_int(p);
        sync_block();
        if (tid == 0) {
            float sum = 0.0f;
            for (int w = 0; w < kGammaThreads / kWave; ++w) sum += __int_as_float(part[w]);
            norm2[x] = sum;
        }
        sync_block();
    }
    const int lane32 = tid & 31;
    const int ng = a.d >> 2;
    const float4 *lu4 = reinterpret_cast<const float4 *>(lu);
    // lane -> (vector, dot or norm, query) of the reduced sum it is left with
    constexpr int kShift = kGammaRows == 2 ? 0 : 1;
    const int mine = lane32 >> kShift;
    const float nu = trim::sqrt_rn(norm2[mine >> 4]);
    constexpr int QB = 8, NH = kGammaThreads / 32;
    for (int q0 = (tid >> 5) * QB; q0 < a.Q; q0 += NH * QB) {
        const int last = a.Q - 1 - q0;        // queries past the end: the last one again, not stored
        const float4 *row0 = reinterpret_cast<const float4 *>(a.queries + (size_t)q0 * a.d);
        float acc[kGammaRows * 2 * QB];       // [vector][dot, norm][query]
#pragma unroll
        for (int i = 0; i < kGammaRows * 2 * QB; ++i) acc[i] = 0.0f;
        for (int g = lane32; g < ng; g += 32) {
            float4 qv[QB];
#pragma unroll
            for (int i = 0; i < QB; ++i) qv[i] = row0[(size_t)(i < last ? i : last) * ng + g];
#pragma unroll
            for (int x = 0; x < kGammaRows; ++x) {
                const float4 lv = lu4[(2 * x) * ng + g], uv = lu4[(2 * x + 1) * ng + g];
#pragma unroll
                for (int i = 0; i < QB; ++i) {
                    gamma_step(qv[i], lv, uv, acc[2 * x * QB + i], acc[(2 * x + 1) * QB + i]);
                }
            }
        }
        const float sum = reduce_pairs<kGammaRows * 2 * QB>(acc, lane32);   // mine: vector (bit 4), dot / norm (bit 3), query (bits 0..2)
        const float nn = __shfl_xor(sum, 8 << kShift);
        const int qi = q0 + (mine & 7);
        if (!(mine & 8) && qi < a.Q) keys[(size_t)(mine >> 4) * a.Q + qi] = gamma_key(sum, nn, nu);
    }
    sync_block();
    for (int x = 0; x < kGammaRows && s0 + x < a.S; ++x) {
        const uint32_t k = key_of_rank<kGammaThreads>(keys + (size_t)x * a.Q, a.Q, a.rank, hist);
        if (tid == 0) gamma_store(a, s0 + x, k);
    }
}

// ---- gamma from a confidence level p for standard-normal queries (Section 3.2) ----
// The theorem of Section 3.2 gives, for a query Q ~ N(0, I) rotated so that x - l lies on the
// first axis and l in the plane of the first two: Z^2 = A / (A + B + C), A = (Q1 + h1)^2,
// B = (Q2 - h2)^2, C = the sum of the squares of the other d - 2 coordinates,
// h1 = (x - l).l / |x - l|, h2 = sqrt(|l|^2 - h1^2); the transform theorem turns the
// distribution of Z^2 into that of 1 - Z.  Only (Q1, Q2, C) of a variate row matter, and they
// do not depend on x: a first kernel reduces every row of normal variates to that triple.
__global__ void normal_triples_kernel(const float *__restrict__ normals, int64_t Q, int d,
                                      double *__restrict__ triples) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= Q) return;
    const float *row = normals + (size_t)r * d;
    double c = 0.0;
    for (int t = 2; t < d; ++t) c += (double)row[t] * (double)row[t];
    triples[3 * r + 0] = (double)row[0];
    triples[3 * r + 1] = (double)row[1];
    triples[3 * r + 2] = c;
}

// One workgroup per sampled data vector: h1 and h2 in binary64, Z^2 for every triple, a bitonic
// sort of the Z^2 in LDS, then the largest y on the grid y_i = 2 i / (grid - 1) whose
// F_{1-Z}(y_i) = 1/2 -+ F_{Z^2}((1 - y_i)^2) / 2 (minus for y <= 1) is at most 1 - p
// (F_{1-Z} rises with y: binary search over i).  gamma = min over the vectors (32-bit atomic
// minimum on the bit pattern of the non-negative binary32 result).
struct GammaNormalArgs {
    const float *base;
    const uint8_t *codes;
    const float *codebooks;
    const int32_t *rows;
    const double *triples;
    int64_t n;
    int32_t d, M, Q, npow2, grid;
    double one_minus_p;
    float *gamma_x;
    uint32_t *gamma_bits;
};

__global__ __launch_bounds__(256) void gamma_normal_kernel(const GammaNormalArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    double *z2 = reinterpret_cast<double *>(smem);   // [npow2]
    __shared__ double red[3][256];
    const int tid = threadIdx.x;
    int64_t r = a.rows[blockIdx.x];
    r = r < 0 ? 0 : (r >= a.n ? a.n - 1 : r);
    const int dsub = a.d / a.M;
    double ul = 0.0, uu = 0.0, ll = 0.0;
    for (int t = tid; t < a.d; t += blockDim.x) {
        const int j = t / dsub;
        const double lt = (double)a.codebooks[((size_t)j * kC + a.codes[(size_t)r * a.M + j]) * dsub + t % dsub];
        const double ut = (double)a.base[(size_t)r * a.d + t] - lt;
        ul += ut * lt; uu += ut * ut; ll += lt * lt;
    }
    red[0][tid] = ul; red[1][tid] = uu; red[2][tid] = ll;
    sync_block();
    for (int h = 128; h > 0; h >>= 1) {
        if (tid < h) { red[0][tid] += red[0][tid + h]; red[1][tid] += red[1][tid + h]; red[2][tid] += red[2][tid + h]; }
        sync_block();
    }
    // a vector equal to its landmark has no angle: 1 - Z counts as 1 for every query (cos = 0)
    const bool no_angle = !(red[1][0] > 0.0);
    const double h1 = no_angle ? 0.0 : red[0][0] / sqrt(red[1][0]);
    const double h2sq = red[2][0] - h1 * h1;
    const double h2 = h2sq > 0.0 ? sqrt(h2sq) : 0.0;
    for (int i = tid; i < a.npow2; i += blockDim.x) {
        double v = __builtin_inf();
        if (i < a.Q) {
            const double q1 = a.triples[3 * (size_t)i], q2 = a.triples[3 * (size_t)i + 1], c = a.triples[3 * (size_t)i + 2];
            const double A = (q1 + h1) * (q1 + h1), B = (q2 - h2) * (q2 - h2);
            v = no_angle ? 0.0 : A / (A + B + c);
        }
        z2[i] = v;
    }
    sync_block();
    for (int k = 2; k <= a.npow2; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = tid; i < a.npow2; i += blockDim.x) {
                const int p = i ^ j;
                if (p > i) {
                    const double x = z2[i], y = z2[p];
                    const bool up = (i & k) == 0;
                    if ((x > y) == up) { z2[i] = y; z2[p] = x; }
                }
            }
            sync_block();
        }
    }
    if (tid == 0) {
        // F_{1-Z}(y_i) for grid point i: the share of Z^2 values <= (1 - y_i)^2, halved either way
        auto cdf = [&](int i) {
            const double y = i == a.grid - 1 ? 2.0 : (double)i * (2.0 / (double)(a.grid - 1));
            const double v = (1.0 - y) * (1.0 - y);
            int lo = 0, hi = a.Q;                 // first index with z2 > v
            while (lo < hi) { const int mid = (lo + hi) >> 1; if (z2[mid] <= v) lo = mid + 1; else hi = mid; }
            const double f = (double)lo / (double)a.Q;
            return y <= 1.0 ? 0.5 - 0.5 * f : 0.5 + 0.5 * f;
        };
        const double limit = a.one_minus_p + 1e-12;
        int lo = -1, hi = a.grid - 1;             // largest i with cdf(i) <= limit (-1: none)
        if (cdf(hi) <= limit) lo = hi;
        else {
            if (cdf(0) <= limit) lo = 0;
            int l2 = lo < 0 ? -1 : 0;
            while (l2 >= 0 && hi - l2 > 1) {
                const int mid = (l2 + hi) >> 1;
                if (cdf(mid) <= limit) l2 = mid; else hi = mid;
            }
            lo = l2;
        }
        const double y = lo < 0 ? 0.0 : (lo == a.grid - 1 ? 2.0 : (double)lo * (2.0 / (double)(a.grid - 1)));
        const float g = (float)y;
        if (a.gamma_x) a.gamma_x[blockIdx.x] = g;
        atomicMin(a.gamma_bits, __float_as_uint(g));
    }
}

// ---- PQ encode (Section 3.3, preprocessing step 1) ----
// The nearest centroid by the fixed binary32 rule (encode distance, smallest index on ties).
// Evaluating the rule for all 256 centroids is bound by the vector ALU (2 d/M operations and the
// comparison each).  For the usual sub-vector lengths the matrix cores leave eight centroids to it:
//
//   filter   S(c) = |x|^2 + m + |c|^2 - 2 x.c for all 256 centroids, 32 vectors x 32 centroids per
//            v_mfma_f32_32x32x16_f16.  x and c are taken relative to the mean of a few centroids
//            (their difference is what counts, and the margin below grows with their lengths), scaled by a power of two and split into a
//            binary16 value and a binary16 remainder (22 bits); the depth of the instruction
//            holds the three products x_hi c_hi, x_lo c_hi, x_hi c_lo of every coordinate, |c|^2 in three pieces, and
//            |x|^2 + m (m: the margin below) as 2^15 times one or two binary16 values that are rounded up (3 d/M + 4 slots or
//            one more), so the split costs no extra instruction up to d/M = 4, one more up to 9.  |x|^2 + m makes every score positive,
//            so that scores order like their bits (integer minimum of three: half an instruction a score).
//   groups   only the minima of eight consecutive centroids are kept.  Groups whose minimum is within the margin of the best are
//            evaluated by the exact rule; usually one.
//
// A wave takes 64 vectors: a lane prepares one and evaluates its groups; the operands go to the two blocks of 32 that the instruction
// takes, and the groups found come back, by exchanging half waves (v_permlane32_swap).  (A block of 32 at a time, both half waves
// preparing the same vectors and 16 centroids a group: 0.75 ms instead of 0.55 for 1,000,000 x 128.)
//
// The margin is twice a bound of |S - exact distance|: dropped products and remainders 3 * 2^-22 of 2 |x||c|, the
// 16 or 32 binary32 additions of an element (2^-23 each of the sum of magnitudes, at most (1 + 2^-8) (|x| + |c|)^2), the exact rule's own
// roundings (d/M + 2) * 2^-24: below 2^-18 (2^-17 with
// two instructions) of (|x| + |c|max)^2, with what binary16 subnormals lose (both sides are
// scaled so that |c|max is 2^12 .. 2^13) inside the same bound.  Vectors or centroids out of the scaled range get an infinite
// margin: every group is then evaluated exactly.
//
// Bound by the vector ALU (per 64 vectors and subspace at d/M = 4: 128 operations for the minima, 64 for the groups, 60 for the
// operands, 100 for a round of groups, of which there are one or two, 70 or 140 for the centroids).  1,000,000 x 128, d/M = 4: 0.55 ms
// (1.75 without the matrix cores); 83,333 x 1536, d/M = 8: 0.77 ms, 333,333 x 384 0.48.
// across: 0, or (ACROSS) the codes are stored subspace by subspace, that many bytes apart (what training's update reads best).
// T: vectors per workgroup.  512: one half of the waves prepares the centroids of the even subspaces, the other those of the odd ones, a
// step ahead of the others: a barrier per subspace; 256: all waves prepare them, between two barriers.
// With grid.y > 1 a workgroup takes jper subspaces of its vectors and
// encode_dlx_kernel adds the landmark distances up afterwards (their order of summation crosses
// all subspaces).
template <int D> constexpr int kEncBias = D <= 4 ? 1 : 2;               // slots of |x|^2 + m
template <int D> constexpr int kEncSteps = (3 * D + 3 + kEncBias<D> + 15) / 16;
template <int D, int T>
struct EncodeLds {
    static constexpr int kBufs = T / kC;
    _Float16 frag[kBufs][kEncSteps<D>][2][kC][8];   // 8 slots of one centroid
    float cf[kBufs][kC / 8][8 * D + 4];                 // the centroids themselves, eight to a run: runs begin in different banks
    float mean[4][D];                               // of a few centroids
    float par[4][D + 4];                            // -mean * scale; scale; the longest centroid's length, scaled
    float wmax[2][4];
};
template <int D, int T, bool ACROSS>
__global__ __launch_bounds__(T, 4) void encode_mfma_kernel(const float *__restrict__ base, int64_t n, int d,
                                                                      const float *__restrict__ codebooks, int M, int jper,
                                                                      uint8_t *__restrict__ codes, int64_t across,
                                                                      float *__restrict__ dlx) {
    typedef _Float16 h8 __attribute__((ext_vector_type(8)));
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    typedef float v16f __attribute__((ext_vector_type(16)));
    constexpr int KS = kEncSteps<D>, NB = kEncBias<D>, GROUPS = T / kC;       // of threads that prepare centroids
    extern __shared__ __align__(16) unsigned char smem[];
    EncodeLds<D, T> &s = *reinterpret_cast<EncodeLds<D, T> *>(smem);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 31, half = lane >> 5;
    const int64_t xi = (int64_t)blockIdx.x * T + tid;
    const float *row = base + (size_t)(xi < n ? xi : n - 1) * d;
    const bool vec_rows = (d & 3) == 0 && (reinterpret_cast<uintptr_t>(base) & 15u) == 0;
    const int jlo = blockIdx.y * jper, jhi = jlo + jper < M ? jlo + jper : M;    // (multiples of four)
    // ---- centroids ----
    const int ct = tid & (kC - 1), mine = wave >> 2;       // this thread's centroid, in the subspaces of this parity
    // where it sits: a lane of the result holds rows 8 q + 4 half + i of a tile, which are made the consecutive centroids
    // 128 half + 16 tile + 4 q + i
    const int my_row = ((ct >> 4) & 7) << 5 | ((ct >> 2) & 3) << 3 | (ct >> 7) << 2 | (ct & 3);
    float c[D];
    auto fetch = [&](int j) {
#pragma unroll
        for (int t = 0; t < D; ++t) c[t] = codebooks[((size_t)j * kC + ct) * D + t];
    };
    auto measure = [&](int j) {        // mean and longest centroid of a subspace
        float mu[D], n2 = 0.0f;        // (mu: the same values in every lane, scalar loads)
#pragma unroll
        for (int t = 0; t < D; ++t) {
            float sum = 0.0f;
#pragma unroll
            for (int i = 0; i < 8; ++i) sum = sum + codebooks[((size_t)j * kC + 32 * i) * D + t];
            mu[t] = sum * 0.125f;
            const float cc = c[t] - mu[t];
            n2 = __builtin_fmaf(cc, cc, n2);
        }
        float m = n2;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) m = __builtin_fmaxf(m, __shfl_xor(m, off));
        if (lane == 0) s.wmax[j & 1][wave & 3] = m;
        if (ct == 0)
#pragma unroll
            for (int t = 0; t < D; ++t) s.mean[j & 3][t] = mu[t];
    };
    auto operands = [&](int j) {
        const float max2 = __builtin_fmaxf(__builtin_fmaxf(s.wmax[j & 1][0], s.wmax[j & 1][1]), __builtin_fmaxf(s.wmax[j & 1][2], s.wmax[j & 1][3]));
        const bool usable = max2 > 1e-30f && max2 < 1e30f;
        // 2^k with 2^24 <= 2^2k max2 < 2^26
        const int k = usable ? (25 - (int)((__float_as_uint(max2) >> 23) - 127)) >> 1 : 0;
        const float sc = __uint_as_float((uint32_t)(k + 127) << 23);
        _Float16 slot[KS * 16];
#pragma unroll
        for (int i = 0; i < KS * 16; ++i) slot[i] = (_Float16)0.0f;
        float n2 = 0.0f;
#pragma unroll
        for (int t = 0; t < D; ++t) {
            const float cc = c[t] - s.mean[j & 3][t], v = -2.0f * (cc * sc);
            n2 = __builtin_fmaf(cc, cc, n2);
            const _Float16 hi = (_Float16)v;
            slot[t] = hi;
            slot[D + t] = hi;
            slot[2 * D + t] = (_Float16)(v - (float)hi);
        }
        const float q2 = (n2 * sc) * sc * (1.0f / 4096.0f);       // (the vector's side of these slots is 4096)
        const _Float16 p1 = (_Float16)q2;
        const _Float16 p2 = (_Float16)(q2 - (float)p1);
        slot[3 * D] = p1;
        slot[3 * D + 1] = p2;
        slot[3 * D + 2] = (_Float16)((q2 - (float)p1) - (float)p2);
#pragma unroll
        for (int i = 0; i < NB; ++i) slot[3 * D + 3 + i] = (_Float16)32768.0f;
#pragma unroll
        for (int i = 0; i < KS * 2; ++i) {
            h8 f;
#pragma unroll
            for (int e = 0; e < 8; ++e) f[e] = slot[8 * i + e];
            *reinterpret_cast<h8 *>(s.frag[j % GROUPS][i >> 1][i & 1][my_row]) = f;
        }
#pragma unroll
        for (int t = 0; t < D; ++t) s.cf[j % GROUPS][ct >> 3][(ct & 7) * D + t] = c[t];
        if (ct == 0) {
#pragma unroll
            for (int t = 0; t < D; ++t) s.par[j & 3][t] = -(s.mean[j & 3][t] * sc);
            s.par[j & 3][D] = sc;
            s.par[j & 3][D + 1] = usable ? trim::sqrt_rn(max2) * sc : __builtin_inff();
        }
    };
    // ---- vectors ----
    float xs[4 * D];                   // four sub-vectors
    auto read_rows = [&](int j) {
        if (vec_rows) {
#pragma unroll
            for (int g = 0; g < D; ++g) *reinterpret_cast<float4 *>(xs + 4 * g) = *reinterpret_cast<const float4 *>(row + (size_t)j * D + 4 * g);
        } else {
#pragma unroll
            for (int t = 0; t < 4 * D; ++t) xs[t] = row[(size_t)j * D + t];
        }
    };
    read_rows(jlo);
    if (jlo + mine < jhi) {
        fetch(jlo + mine);
        measure(jlo + mine);
    }
    sync_block();
    if (mine == 0) {
        operands(jlo);
        if (jlo + GROUPS < jhi) fetch(jlo + GROUPS);
    }
    sync_block();
    float tot = 0.0f;
    for (int j0 = jlo; j0 < jhi; j0 += 4) {
        uint32_t packed = 0;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            const int j = j0 + jj;
            if constexpr (GROUPS == 1) {
                if (j + 1 < jhi) measure(j + 1);
            } else if (mine != (jj & 1)) {
                if (j + 1 < jhi) operands(j + 1);
                if (j + 3 < jhi) fetch(j + 3);
            } else if (j + 2 < jhi) {
                measure(j + 2);
            }
            float x[D];
#pragma unroll
            for (int t = 0; t < D; ++t) x[t] = xs[jj * D + t];
            if (jj == 3 && j0 + 4 < jhi) read_rows(j0 + 4);
            const float sc = s.par[jj][D], cmax = s.par[jj][D + 1];
            float xn2 = 0.0f, xmax = 0.0f;
            _Float16 slot[KS * 16];
#pragma unroll
            for (int i = 0; i < KS * 16; ++i) slot[i] = (_Float16)0.0f;
#pragma unroll
            for (int t = 0; t < D; ++t) {
                const float v = __builtin_fmaf(x[t], sc, s.par[jj][t]);      // (x - mean) * scale, rounded once
                const _Float16 hi = (_Float16)v;
                slot[t] = hi;
                slot[D + t] = (_Float16)(v - (float)hi);
                slot[2 * D + t] = hi;
                xn2 = __builtin_fmaf(v, v, xn2);
                xmax = __builtin_fmaxf(xmax, __builtin_fabsf(v));
            }
            slot[3 * D] = slot[3 * D + 1] = slot[3 * D + 2] = (_Float16)4096.0f;
            const float reach = __builtin_amdgcn_sqrtf(xn2) + cmax;
            float margin = reach * reach * (KS == 1 ? 1.25f / 131072.0f : 1.0f / 65536.0f);
            if (!(xmax < 16384.0f)) margin = __builtin_inff();
            const float bias = margin < __builtin_inff() ? (xn2 + margin) * ((1.0f + 1.0f / 512.0f) / 32768.0f / NB) : 0.0f;
#pragma unroll
            for (int i = 0; i < NB; ++i) slot[3 * D + 3 + i] = (_Float16)bias;
            h8 xf[2][KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                h8 f0, f1;
#pragma unroll
                for (int e = 0; e < 8; ++e) { f0[e] = slot[16 * ks + e]; f1[e] = slot[16 * ks + 8 + e]; }
                const u4 w0 = __builtin_bit_cast(u4, f0), w1 = __builtin_bit_cast(u4, f1);
                u4 r0, r1;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const auto p = __builtin_amdgcn_permlane32_swap(w0[e], w1[e], false, false);
                    r0[e] = p[0];
                    r1[e] = p[1];
                }
                xf[0][ks] = __builtin_bit_cast(h8, r0);
                xf[1][ks] = __builtin_bit_cast(h8, r1);
            }
            const auto margins = __builtin_amdgcn_permlane32_swap(__float_as_uint(margin), __float_as_uint(margin), false, false);
            float thr[2];
            uint32_t past[2] = {0, 0};       // groups beyond the threshold
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                int gmin[16];
#pragma unroll
                for (int t = 0; t < 8; t += 2) {
                    v16f acc[2] = {};
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                        for (int u = 0; u < 2; ++u)
                            acc[u] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                                *reinterpret_cast<const h8 *>(s.frag[jj % GROUPS][ks][half][(t + u) * 32 + col]), xf[b][ks], acc[u], 0, 0, 0);
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            int g = __float_as_int(acc[u][8 * h]);
#pragma unroll
                            for (int i = 1; i < 8; ++i) g = g < __float_as_int(acc[u][8 * h + i]) ? g : __float_as_int(acc[u][8 * h + i]);
                            gmin[2 * (t + u) + h] = g;
                        }
                }
                int least = gmin[0];
#pragma unroll
                for (int g = 1; g < 16; ++g) least = least < gmin[g] ? least : gmin[g];
                const auto both = __builtin_amdgcn_permlane32_swap((uint32_t)least, (uint32_t)least, false, false);
                thr[b] = __int_as_float((int)both[0] < (int)both[1] ? (int)both[0] : (int)both[1]) + __uint_as_float(margins[b]);
                // by the sign of a difference (scores are positive: they order like their bits)
#pragma unroll
                for (int g = 15; g >= 0; --g) past[b] = __builtin_amdgcn_alignbit(past[b], __float_as_uint(thr[b]) - (uint32_t)gmin[g], 31);
                __builtin_amdgcn_sched_barrier(0);
            }
            const auto mp = __builtin_amdgcn_permlane32_swap(past[0], past[1], false, false);
            uint32_t todo = (half ? thr[1] : thr[0]) < __builtin_inff() ? ~(mp[0] | mp[1] << 16) : ~0u;
            float best = __builtin_inff();
            int arg = 0;
            do {
                if (todo != 0) {
                    const int g = __ffs((int)todo) - 1;
                    todo &= todo - 1;
                    const float *run = s.cf[jj % GROUPS][g];     // ascending from group to group: strict < keeps the smallest index
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        float acc = 0.0f;
#pragma unroll
                        for (int t = 0; t < D; ++t) {
                            const float e = x[t] - run[i * D + t];
                            acc = __builtin_fmaf(e, e, acc);
                        }
                        if (acc < best) { best = acc; arg = g * 8 + i; }
                    }
                }
            } while (__any(todo != 0));
            tot = tot + best;
            if constexpr (ACROSS) {
                if (xi < n) codes[(size_t)j * across + xi] = (uint8_t)arg;
            } else {
                packed |= (uint32_t)arg << (8 * jj);
            }
            sync_block();
            if constexpr (GROUPS == 1) {
                if (j + 1 < jhi) operands(j + 1);
                if (j + 2 < jhi) fetch(j + 2);
                sync_block();
            }
        }
        if constexpr (!ACROSS)
            if (xi < n) *reinterpret_cast<uint32_t *>(codes + (size_t)xi * M + j0) = packed;
    }
    if (jper >= M && dlx && xi < n) dlx[xi] = trim::sqrt_rn(tot);
}

// Landmark distances from finished codes: the same sub-distances, added in subspace order.  A
// workgroup takes kDlxRows vectors; their sub-distances wait in LDS, slices of kDlxSub subspaces.
constexpr int kDlxRows = 16, kDlxSub = 128;
__global__ __launch_bounds__(256) void encode_dlx_kernel(const float *__restrict__ base, int64_t n, int d,
                                                         const float *__restrict__ codebooks, int M, int dsub,
                                                         const uint8_t *__restrict__ codes, float *__restrict__ dlx) {
    __shared__ float part[kDlxRows * (kDlxSub + 1)];
    const int64_t x0 = (int64_t)blockIdx.x * kDlxRows;
    float tot = 0.0f;
    for (int j0 = 0; j0 < M; j0 += kDlxSub) {
        const int nj = M - j0 < kDlxSub ? M - j0 : kDlxSub;
        for (int e = threadIdx.x; e < kDlxRows * nj; e += 256) {
            const int r = e / nj, j = e - r * nj;
            const int64_t x = x0 + r < n ? x0 + r : n - 1;
            const float *xr = base + (size_t)x * d + (size_t)(j0 + j) * dsub;
            const float *c = codebooks + ((size_t)(j0 + j) * kC + codes[(size_t)x * M + j0 + j]) * dsub;
            float acc = 0.0f;
            for (int t = 0; t < dsub; ++t) {
                const float v = xr[t] - c[t];
                acc = __builtin_fmaf(v, v, acc);
            }
            part[r * (kDlxSub + 1) + j] = acc < __builtin_inff() ? acc : __builtin_inff();     // (the least distance begins at infinity: no NaN)
        }
        sync_block();
        if (threadIdx.x < kDlxRows)
            for (int j = 0; j < nj; ++j) tot = tot + part[threadIdx.x * (kDlxSub + 1) + j];
        sync_block();
    }
    if (threadIdx.x < kDlxRows && x0 + threadIdx.x < n) dlx[x0 + threadIdx.x] = trim::sqrt_rn(tot);
}

// Any other sub-vector length: one thread per vector; the block stages one subspace's 256
// centroids in LDS at a time.
__global__ __launch_bounds__(256) void encode_kernel(const float *__restrict__ base, int64_t n,
                                                     int d, const float *__restrict__ codebooks,
                                                     int M, int dsub,
                                                     uint8_t *__restrict__ codes, int64_t across,
                                                     float *__restrict__ dlx) {
    extern __shared__ __align__(16) unsigned char smem[];
    float *cb = reinterpret_cast<float *>(smem);  // [256][dsub]
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = i < n;
    const float *x = base + (size_t)(valid ? i : 0) * d;
    float tot = 0.0f;
    uint32_t packed = 0;
    for (int j = 0; j < M; ++j) {
        sync_block();
        for (int e = threadIdx.x; e < kC * dsub; e += blockDim.x)
            cb[e] = codebooks[(size_t)j * kC * dsub + e];
        sync_block();
        float best = __builtin_inff();
        int arg = 0;
        for (int c = 0; c < kC; ++c) {
            float acc = 0.0f;
            for (int t = 0; t < dsub; ++t) {
                const float e = x[j * dsub + t] - cb[c * dsub + t];
                acc = __builtin_fmaf(e, e, acc);
            }
            if (acc < best) { best = acc; arg = c; }
        }
        tot = tot + best;
        if (across && valid) codes[(size_t)j * across + i] = (uint8_t)arg;
        packed |= (uint32_t)arg << (8 * (j & 3));
        if ((j & 3) == 3) {
            if (valid && !across) *reinterpret_cast<uint32_t *>(codes + (size_t)i * M + (j - 3)) = packed;
            packed = 0;
        }
    }
    if (valid && dlx) dlx[i] = trim::sqrt_rn(tot);
}

// ---- PQ encode with 16 centroids per subspace (4-bit codes; Section 6.1, FastScan variants) ----
// PACKED: two codes per byte, the even subspace's in the low half (the stored index); else one
// byte per subspace (the assignments training works on; across: see encode_mfma_kernel).
//
// Sub-vectors of two values (m = d/2, the paper's variant): one thread per vector; the block's
// rows pass through the LDS 32 columns at a time (whole cache lines from memory, 16-byte reads
// without bank conflicts), a subspace's 16 centroids are the same for every thread and arrive in
// scalar registers.  What is left is the vector ALU: 7 operations per centroid.
// 200,000 x 256: 0.11 ms (11.0 ms when every thread read its own row and centroids came through LDS).
constexpr int kFsRows = 256, kFsCols = 32, kFsStride = kFsCols + 4;
template <bool PACKED>
__global__ __launch_bounds__(kFsRows) void encode_fs2_kernel(const float *__restrict__ base, int64_t n, int d,
                                                             const float *__restrict__ codebooks, int m,
                                                             uint8_t *__restrict__ codes, int64_t across,
                                                             float *__restrict__ dlx) {
    __shared__ __align__(16) float xt[kFsRows * kFsStride];
    const int64_t x0 = (int64_t)blockIdx.x * kFsRows, i = x0 + threadIdx.x;
    const bool valid = i < n;
    const bool vec_rows = (d & 3) == 0 && (reinterpret_cast<uintptr_t>(base) & 15u) == 0;
    const int per_row = PACKED ? m / 2 : m;     // bytes
    const bool vec_out = per_row % (PACKED ? 8 : 16) == 0 && (reinterpret_cast<uintptr_t>(codes) & (PACKED ? 7u : 15u)) == 0;
    float tot = 0.0f;
    for (int c0 = 0; c0 < d; c0 += kFsCols) {
        const int cols = d - c0 < kFsCols ? d - c0 : kFsCols;
        sync_block();
        if (vec_rows) {
            for (int e = threadIdx.x; e < kFsRows * (kFsCols / 4); e += kFsRows) {
                const int r = e / (kFsCols / 4), g = e % (kFsCols / 4);
                const int64_t x = x0 + r < n ? x0 + r : n - 1;
                if (4 * g < cols)
                    *reinterpret_cast<float4 *>(xt + r * kFsStride + 4 * g) =
                        *reinterpret_cast<const float4 *>(base + (size_t)x * d + c0 + 4 * g);
            }
        } else {
            for (int e = threadIdx.x; e < kFsRows * kFsCols; e += kFsRows) {
                const int r = e / kFsCols, g = e % kFsCols;
                const int64_t x = x0 + r < n ? x0 + r : n - 1;
                if (g < cols) xt[r * kFsStride + g] = base[(size_t)x * d + c0 + g];
            }
        }
        sync_block();
        uint32_t out[PACKED ? 2 : 4] = {};
        const float *xr = xt + threadIdx.x * kFsStride;
#pragma clang loop unroll(disable)
        for (int wd = 0; wd < (PACKED ? 2 : 4); ++wd) {    // output words: 8 packed codes, or 4 bytes
            constexpr int kPer = PACKED ? 8 : 4;
            uint32_t word = 0;
#pragma unroll
            for (int u = 0; u < kPer; ++u) {               // one subspace: two values
                const int q = wd * kPer + u;
                if (2 * q < cols) {
                    const float2 xv = *reinterpret_cast<const float2 *>(xr + 2 * q);
                    const float *cb = codebooks + (size_t)(c0 / 2 + q) * kC4 * 2;
                    float best = __builtin_inff();
                    int arg = 0;
#pragma unroll
                    for (int c = 0; c < kC4; ++c) {
                        float e, acc = 0.0f;
                        e = xv.x - cb[2 * c]; acc = __builtin_fmaf(e, e, acc);
                        e = xv.y - cb[2 * c + 1]; acc = __builtin_fmaf(e, e, acc);
                        if (acc < best) { best = acc; arg = c; }
                    }
                    tot = tot + best;
                    word |= (uint32_t)arg << (PACKED ? 4 * u : 8 * u);
                }
            }
#pragma unroll
            for (int o = 0; o < (PACKED ? 2 : 4); ++o) out[o] = o == wd ? word : out[o];
        }
        if (!valid) continue;
        if (!PACKED && across) {
            for (int b = 0; b < cols / 2; ++b) codes[(size_t)(c0 / 2 + b) * across + i] = (uint8_t)(out[b >> 2] >> (8 * (b & 3)));
            continue;
        }
        uint8_t *to = codes + (size_t)i * per_row + (PACKED ? c0 / 4 : c0 / 2);
        if (cols == kFsCols && vec_out) {
            if constexpr (PACKED) *reinterpret_cast<uint2 *>(to) = make_uint2(out[0], out[1]);
            else *reinterpret_cast<uint4 *>(to) = make_uint4(out[0], out[1], out[PACKED ? 0 : 2], out[PACKED ? 1 : 3]);
        } else {
            for (int b = 0; b < cols / (PACKED ? 4 : 2); ++b) to[b] = (uint8_t)(out[b >> 2] >> (8 * (b & 3)));
        }
    }
    if (valid && dlx) dlx[i] = trim::sqrt_rn(tot);
}

// Any other sub-vector length: one thread per vector; the two subspaces of one code byte at a time in LDS.
template <bool PACKED>
__global__ __launch_bounds__(256) void encode_fs_kernel(const float *__restrict__ base, int64_t n, int d,
                                                        const float *__restrict__ codebooks, int m,
                                                        int dsub, uint8_t *__restrict__ codes, int64_t across,
                                                        float *__restrict__ dlx) {
    extern __shared__ __align__(16) unsigned char smem[];
    float *cb = reinterpret_cast<float *>(smem);  // [2][16][dsub]: the two subspaces of one code byte
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = i < n;
    const float *x = base + (size_t)(valid ? i : 0) * d;
    float tot = 0.0f;
    for (int jb = 0; jb < m / 2; ++jb) {
        sync_block();
        for (int e = threadIdx.x; e < 2 * kC4 * dsub; e += blockDim.x)
            cb[e] = codebooks[(size_t)jb * 2 * kC4 * dsub + e];
        sync_block();
        uint32_t byte = 0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int j = 2 * jb + h;
            float best = __builtin_inff();
            int arg = 0;
            for (int c = 0; c < kC4; ++c) {
                float acc = 0.0f;
                for (int t = 0; t < dsub; ++t) {
                    const float e = x[j * dsub + t] - cb[(h * kC4 + c) * dsub + t];
                    acc = __builtin_fmaf(e, e, acc);
                }
                if (acc < best) { best = acc; arg = c; }
            }
            tot = tot + best;
            if (PACKED) byte |= (uint32_t)arg << (4 * h);
            else if (valid) codes[across ? (size_t)j * across + i : (size_t)i * m + j] = (uint8_t)arg;
        }
        if (PACKED && valid) codes[(size_t)i * (m / 2) + jb] = (uint8_t)byte;
    }
    if (valid && dlx) dlx[i] = trim::sqrt_rn(tot);
}

// ---- stand-alone distance table for 4-bit codes: lut[q][j][c], c < 16 ----
// grid (ceil(m/2 / bper), nq); each block writes the entries of bper code bytes of one query.
__global__ __launch_bounds__(256) void lut_fs_kernel(const float *__restrict__ queries, int d,
                                                     const float *__restrict__ codebooks, int m,
                                                     int dsub, int bper, float *__restrict__ lut) {
    extern __shared__ __align__(16) unsigned char smem[];
    float *q_lds = reinterpret_cast<float *>(smem);
    const int64_t q = blockIdx.y;
    const int b0 = blockIdx.x * bper;
    const int nb = b0 + bper <= m / 2 ? bper : m / 2 - b0;
    for (int t = threadIdx.x; t < d; t += blockDim.x) q_lds[t] = queries[(size_t)q * d + t];
    sync_block();
    build_table_rows<true>(lut + ((size_t)q * m + 2 * b0) * kC4, q_lds, codebooks, dsub, b0, nb);
}

// ---- stand-alone distance table (Section 3.3, query-processing operation 1) ----
// grid (ceil(M / jper), nq); each block writes jper table rows of one query.
__global__ __launch_bounds__(256) void lut_kernel(const float *__restrict__ queries, int d,
                                                  const float *__restrict__ codebooks, int M,
                                                  int dsub, int jper, float *__restrict__ lut) {
    extern __shared__ __align__(16) unsigned char smem[];
    float *q_lds = reinterpret_cast<float *>(smem);
    const int64_t q = blockIdx.y;
    const int j0 = blockIdx.x * jper;
    const int nj = j0 + jper <= M ? jper : M - j0;
    for (int t = threadIdx.x; t < d; t += blockDim.x) q_lds[t] = queries[(size_t)q * d + t];
    sync_block();
    build_table_rows(lut + ((size_t)q * M + j0) * kC, q_lds, codebooks, dsub, j0, nj);
}

// ---- distance table on the matrix cores (expanded form) ----
// T[q][j][c] = max(0, (||q_j||^2 + ||c||^2) - 2 q_j.c).  One wave computes a tile of 16 queries
// x 256 centroids of one subspace: the cross terms are 16 MFMA tiles 16x16 with depth 4
// (v_mfma_f32_16x16x4_f32; two of them per tile for sub-vectors of length 8).
// Operand layout of that instruction for lane l: A[row l%16][k l/16], B[k l/16][col l%16],
// D[row 4*(l/16)+r][col l%16] in result register r.
// The contraction depth is only d/M, so each MFMA (256 FMAs ... per 1 KB stored) leaves the
// kernel bound by writing the table, not by the matrix cores.
template <int DSUB>
__global__ __launch_bounds__(256) void lut_mfma_kernel(const float *__restrict__ queries, int64_t nq,
                                                       int d, const float *__restrict__ codebooks,
                                                       int M, float *__restrict__ lut) {
    typedef float v4f __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & 63;
    const int j = blockIdx.y * 4 + (threadIdx.x >> 6);
    if (j >= M) return;  // whole wave
    const int64_t q0 = (int64_t)blockIdx.x * 16;
    const int li = lane & 15, lg = lane >> 4;
    // A operand: query row q0+li, elements k = lg (and lg+4 for DSUB == 8)
    const int64_t qa = q0 + li < nq ? q0 + li : nq - 1;
    const float *qrow = queries + (size_t)qa * d + (size_t)j * DSUB;
    const float a0 = qrow[lg];
    const float a1 = DSUB == 8 ? qrow[lg + 4] : 0.0f;
    // squared norms of the 4 query rows this lane stores (rows 4*lg + r)
    float qn[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t qr = q0 + 4 * lg + r < nq ? q0 + 4 * lg + r : nq - 1;
        const float *p = queries + (size_t)qr * d + (size_t)j * DSUB;
        float acc = 0.0f;
#pragma unroll
        for (int t = 0; t < DSUB; ++t) acc = __builtin_fmaf(p[t], p[t], acc);
        qn[r] = acc;
    }
    const float *cb = codebooks + (size_t)j * kC * DSUB;
    for (int c0 = 0; c0 < kC; c0 += 16) {
        const float *crow = cb + (size_t)(c0 + li) * DSUB;   // centroid column li of this tile
        float cn = 0.0f;
#pragma unroll
        for (int t = 0; t < DSUB; ++t) cn = __builtin_fmaf(crow[t], crow[t], cn);
        v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, crow[lg], acc, 0, 0, 0);
        if (DSUB == 8) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, crow[lg + 4], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t q = q0 + 4 * lg + r;
            if (q < nq) {
                const float t = __builtin_fmaf(-2.0f, acc[r], qn[r] + cn);
                lut[((size_t)q * M + j) * kC + c0 + li] = t > 0.0f ? t : 0.0f;
            }
        }
    }
}

// ---- range search: offsets from per-chunk counts (single workgroup) ----
// counts [nq*nsplit] -> chunk_base [nq*nsplit] (exclusive prefix), out_offsets [nq+1],
// *required = total.
__global__ __launch_bounds__(1024) void range_offsets_kernel(const int32_t *__restrict__ counts,
                                                             int64_t nq, int nsplit,
                                                             int64_t *__restrict__ chunk_base,
                                                             int64_t *__restrict__ out_offsets,
                                                             int64_t *__restrict__ required) {
    __shared__ long long part[16];
    const int64_t total_items = nq * nsplit;
    const int T = 1024, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t per = (total_items + T - 1) / T;
    const int64_t lo = (int64_t)threadIdx.x * per;
    const int64_t hi = lo + per < total_items ? lo + per : total_items;
    int64_t s = 0;
    for (int64_t i = lo; i < hi; ++i) s += counts[i];
    long long incl = s;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const long long v = __shfl_up(incl, off);
        if (lane >= off) incl += v;
    }
    if (lane == 63) part[wave] = incl;
    sync_block();
    int64_t run = incl - s;
    for (int w = 0; w < wave; ++w) run += part[w];
    if (threadIdx.x == 1023) {
        out_offsets[nq] = run + s;
        if (required) *required = run + s;
    }
    for (int64_t i = lo; i < hi; ++i) {
        chunk_base[i] = run;
        if (i % nsplit == 0) out_offsets[i / nsplit] = run;
        run += counts[i];
    }
}

// ---- range search: write the results of one (query, chunk) in scan order ----
struct RangeFillArgs {
    const float *base;
    const int32_t *ids;
    const float *queries;
    const int64_t *list_offsets;
    const int32_t *probes;
    int64_t n;
    int32_t d, nlist, nseg, max_cand, chunk, nsplit;
    const uint32_t *result_mask;
    int64_t rmask_words;
    const float *result_d2;   // exact distance of each result, by scan-order number
    const int64_t *chunk_base;
    int32_t *out_ids;
    float *out_d2;
    int64_t capacity;
    uint32_t off_q, off_segp, off_segd, off_list;
};

__global__ __launch_bounds__(256) void range_fill_kernel(const RangeFillArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    int *segp = reinterpret_cast<int *>(smem + a.off_segp);
    int *segd = reinterpret_cast<int *>(smem + a.off_segd);
    int *list = reinterpret_cast<int *>(smem + a.off_list);  // [2048] scan-order numbers
    __shared__ int s_total;

    const int tid = threadIdx.x, T = blockDim.x;
    const int lane = tid & (kWave - 1);
    const int64_t q = blockIdx.x;
    const int split = blockIdx.y;
    const int nseg = a.nseg > 0 ? a.nseg : 1;

    for (int p = tid; p < nseg; p += T) {
        int64_t s = 0, e = a.n;
        if (a.nseg > 0) {
            const int32_t l = a.probes[(size_t)q * a.nseg + p];
            if (l >= 0 && l < a.nlist) {
                s = a.list_offsets[l];
                e = a.list_offsets[l + 1];
                s = s < 0 ? 0 : (s > a.n ? a.n : s);
                e = e < s ? s : (e > a.n ? a.n : e);
            } else {
                s = e = 0;
            }
        }
        segd[p] = (int)s;
        segp[p + 1] = (int)(e - s);
    }
    sync_block();
    if (tid == 0) {
        int64_t run = 0;
        segp[0] = 0;
        for (int p = 0; p < nseg; ++p) {
            int64_t len = segp[p + 1];
            if (run + len > a.max_cand) len = a.max_cand - run;
            segd[p] = segd[p] - (int)run;
            run += len;
            segp[p + 1] = (int)run;
        }
        s_total = (int)run;
    }
    sync_block();
    const int total = s_total;
    const int c_begin = split * a.chunk;
    if (c_begin >= total) return;
    const int c_end = c_begin + a.chunk < total ? c_begin + a.chunk : total;
    int64_t out = a.chunk_base[(size_t)q * a.nsplit + split];

    // rounds of 64 mask words (2048 candidates); wave 0 expands set bits in order
    for (int r0 = c_begin; r0 < c_end; r0 += 2048) {
        __shared__ int s_cnt;
        if (tid < kWave) {
            const int c_w = r0 + lane * 32;
            uint32_t w = 0;
            if (c_w < c_end) w = a.result_mask[(size_t)q * a.rmask_words + (c_w >> 5)];
            int cnt = __popc(w);
            int incl = cnt;  // inclusive prefix over the wave
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const int v = __shfl_up(incl, o);
                if (lane >= o) incl += v;
            }
            int at = incl - cnt;
            while (w) {
                const int b = __ffs((int)w) - 1;
                w &= w - 1;
                list[at++] = c_w + b;
            }
            if (lane == kWave - 1) s_cnt = incl;
        }
        sync_block();
        const int cnt = s_cnt;
        for (int i = tid; i < cnt; i += T) {
            if (out + i >= a.capacity) break;
            const int c = list[i];
            // segment of c by binary search over the prefix table
            int lo = 0, hi = nseg - 1;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (c >= segp[mid + 1]) lo = mid + 1; else hi = mid;
            }
            const int pos = c + segd[lo];
            a.out_ids[out + i] = a.ids ? a.ids[pos] : pos;
            a.out_d2[out + i] = a.result_d2[(size_t)q * a.rmask_words * 32 + c];   // as the search computed it
        }
        out += cnt;
        sync_block();
    }
}

// ---- coarse probe selection in two kernels: few queries ----
// ivf_probe_kernel gives 8 queries one workgroup, which walks all centroids: 35 us for one query over 1024 lists of
// 128 values, 75 us for 67 over 1024 of 384, on one and nine of the CUs.  Here the lists are split over the grid as
// well (grid.x, 8 kRows per workgroup) and the distances pass through memory: dist [nq][nlist], bit patterns.
constexpr int kProbeThreads = 256;
// Lists l0 .. (eight of them; four with eight queries) against the QT queries in the LDS, by a half wave (the loop of
// ivf_probe_kernel): store(query, list, distance), each pair in one lane.
template <int QT, typename F>
__device__ __forceinline__ void probe_distances(const float *q_lds, int d, const float *__restrict__ centroids, int nlist, int l0,
                                                int lane32, F &&store) {
    constexpr int kRows = QT == 8 ? 4 : 8, NP = kRows * QT;
    constexpr int kShift = NP == 32 ? 0 : NP == 16 ? 1 : 2;
    const int ng = d >> 2;
    const float4 *row0 = reinterpret_cast<const float4 *>(centroids + (size_t)l0 * d);
    const int last = nlist - 1 - l0;     // (rows past the end: the last row again, never stored)
    float acc[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) acc[i] = 0.0f;
    for (int g = lane32; g < ng; g += 32) {
        float4 x[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r) x[r] = row0[(r < last ? r : last) * ng + g];
#pragma unroll
        for (int qi = 0; qi < QT; ++qi) {
            const float4 qv = *reinterpret_cast<const float4 *>(q_lds + qi * d + 4 * g);
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
                float e, a0 = acc[r * QT + qi];
                e = qv.x - x[r].x; a0 = __builtin_fmaf(e, e, a0);
                e = qv.y - x[r].y; a0 = __builtin_fmaf(e, e, a0);
                e = qv.z - x[r].z; a0 = __builtin_fmaf(e, e, a0);
                e = qv.w - x[r].w; a0 = __builtin_fmaf(e, e, a0);
                acc[r * QT + qi] = a0;
            }
        }
    }
    const float v = reduce_pairs<NP>(acc, lane32);
    const int pair = lane32 >> kShift, l = l0 + pair / QT, qi = pair % QT;
    if ((lane32 & ((1 << kShift) - 1)) == 0 && l < nlist) store(qi, l, v);
}
template <int QT>
__global__ __launch_bounds__(kProbeThreads) void probe_distance_kernel(const float *__restrict__ queries, int64_t nq, int d,
                                                                      const float *__restrict__ centroids, int nlist,
                                                                      uint32_t *__restrict__ dist) {
    extern __shared__ __align__(16) unsigned char smem[];
    float *q_lds = reinterpret_cast<float *>(smem);                            // [QT][d]
    const int tid = threadIdx.x, lane32 = tid & 31;
    const int64_t q0 = (int64_t)blockIdx.y * QT;
    const int nqt = (int)(nq - q0 < QT ? nq - q0 : QT);
    for (int t = tid; t < QT * d; t += kProbeThreads) q_lds[t] = t < nqt * d ? queries[(size_t)q0 * d + t] : 0.0f;
    sync_block();
    const int l0 = ((int)blockIdx.x * (kProbeThreads / 32) + (tid >> 5)) * (QT == 8 ? 4 : 8);
    if (l0 >= nlist) return;
    probe_distances<QT>(q_lds, d, centroids, nlist, l0, lane32, [&](int qi, int l, float v) {
        if (qi < nqt) dist[(size_t)(q0 + qi) * nlist + l] = __float_as_uint(v);
    });
}
// The nprobe (at most 64) least (distance, list) of a query: one wave each.  The lists are 256 columns (lane, 0..3); the
// nprobe-th least of the columns' minima, found bit by bit from above, bounds the nprobe-th least of all, so
// whatever is not above it is ranked.  Twenty bits leave few enough nearly always; where more than 128 are left (a query far from all
// lists, whose distances agree in those bits), the other twelve bits are found as well, and where still more are (equal
// distances, or none that is a number) the first nprobe of those at the bound do.  Else (many near lists in one column) the
// least are taken one by one.  With that after the twenty bits already, a query of 128 values at 10^5 from 1024 lists took 58 us
// with its distances (now 11.5), 67 of 384 values with 64 probes 117 (now 15; 13 near the lists), 67 that are no numbers 117 (now 14).
// Bound by its chain of steps across the lanes: two bitonic sorts of 64 (128) keys, 21 (28) exchanges each, in place of the
// ballots and the ranks took 7.4 us of a single query's 46, 1024 lists, 32 probes (now 3.6), and 14.2 of 67 queries' 112 with 64 (now 6.3).
constexpr int kSelectList = 256, kSelectKeep = 16;
__device__ __forceinline__ void select_least(const uint32_t *row, int nlist, int nprobe, int32_t *out, unsigned long long *s_key, int lane) {
    constexpr int kStep = kSelectKeep * kWave;
    auto load = [&](int i0, uint32_t (&v)[kSelectKeep]) {
#pragma unroll
        for (int t = 0; t < kSelectKeep; ++t) {
            const int i = i0 + t * kWave + lane;
            v[t] = row[i < nlist ? i : nlist - 1];
        }
#pragma unroll
        for (int t = 0; t < kSelectKeep; ++t) v[t] = i0 + t * kWave + lane < nlist ? v[t] : ~0u;
    };
    uint32_t v[kSelectKeep], least[4] = {~0u, ~0u, ~0u, ~0u};      // (v: the first lists)
    load(0, v);
#pragma unroll
    for (int t = 0; t < kSelectKeep; ++t) least[t & 3] = min(least[t & 3], v[t]);
    for (int i0 = kStep; i0 < nlist; i0 += kStep) {
        uint32_t w[kSelectKeep];
        load(i0, w);
#pragma unroll
        for (int t = 0; t < kSelectKeep; ++t) least[t & 3] = min(least[t & 3], w[t]);
    }
    uint32_t cut = 0;
    auto narrow = [&](int from, int to) {
#pragma unroll 4
        for (int bit = from; bit > to; --bit) {
            const uint32_t at = cut | 1u << bit;
            int below = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) below += __popcll(__ballot(least[e] < at));
            if (below < nprobe) cut = at;
        }
    };
    const unsigned long long lower = (1ull << lane) - 1ull;
    int n = 0, at_cut = 0;
    auto take = [&](int i0, const uint32_t (&w)[kSelectKeep], uint32_t bound, int ties) {     // (ties: of those at the bound)
#pragma unroll
        for (int t = 0; t < kSelectKeep; ++t) {
            const int i = i0 + t * kWave + lane;
            bool on = i < nlist && w[t] <= bound;
            if (ties >= 0) {
                const bool tie = on && w[t] == bound;
                const unsigned long long m = __ballot(tie);
                on = on && (!tie || at_cut + (int)__popcll(m & lower) < ties);
                at_cut += __popcll(m);
            }
            const unsigned long long m = __ballot(on);
            const int to = n + __popcll(m & lower);
            if (on && to < kSelectList) s_key[to] = ((unsigned long long)w[t] << 32) | (uint32_t)i;
            n += __popcll(m);
        }
    };
    auto collect = [&](uint32_t bound, int ties) {
        n = at_cut = 0;
        take(0, v, bound, ties);
        for (int i0 = kStep; i0 < nlist; i0 += kStep) {
            uint32_t w[kSelectKeep];
            load(i0, w);
            take(i0, w, bound, ties);
        }
    };
    narrow(31, 11);
    collect(cut | 0xfffu, -1);
    if (n > 2 * kWave) {
        narrow(11, -1);
        collect(cut, nprobe);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (n <= kSelectList) {
        for (int i = lane; i < n; i += kWave) {
            const unsigned long long k = s_key[i];
            int rank = 0;
#pragma unroll 8
            for (int j = 0; j < n; ++j) rank += s_key[j] < k;
            if (rank < nprobe) out[rank] = (int32_t)(k & 0xffffffffu);
        }
        return;
    }
    unsigned long long after = 0;                    // the least key not taken yet is at least this
    for (int p = 0; p < nprobe; ++p) {
        unsigned long long m = ~0ull;
        for (int i = lane; i < nlist; i += kWave) {
            const unsigned long long key = ((unsigned long long)row[i] << 32) | (uint32_t)i;
            if (key >= after && key < m) m = key;
        }
#pragma unroll
        for (int j = 32; j > 0; j >>= 1) {
            const unsigned long long other = (unsigned long long)__shfl_xor((long long)m, j);
            m = other < m ? other : m;
        }
        if (lane == 0) out[p] = (int32_t)(m & 0xffffffffu);
        after = m + 1;
    }
}
__global__ __launch_bounds__(kWave) void probe_select_kernel(const uint32_t *__restrict__ dist, int nlist, int nprobe,
                                                             int32_t *__restrict__ probes) {
    __shared__ unsigned long long s_key[kSelectList];
    select_least(dist + (size_t)blockIdx.x * nlist, nlist, nprobe, probes + (size_t)blockIdx.x * nprobe, s_key, threadIdx.x);
}

// ---- coarse probe selection (Section 6.1: IVFPQ with C' lists, nprobe probed) ----
// One workgroup handles QT queries: every centroid row is read once and measured against
// all QT queries (exact distances by half waves, rounding order as in exact_d2_half; the lane
// sums of eight rows x QT queries are reduced together), then
// the nprobe smallest of each query's (distance bits, list id) keys are selected in LDS
// (bitonic runs and pairwise merges) and their ids are written in ascending key order.
template <int QT>
__global__ __launch_bounds__(512) void ivf_probe_kernel(const float *__restrict__ queries,
                                                        int64_t nq, int d,
                                                        const float *__restrict__ centroids,
                                                        int nlist, int npow2, int nprobe,
                                                        int32_t *__restrict__ probes) {
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned long long *keys = reinterpret_cast<unsigned long long *>(smem);  // [QT][npow2]
    float *q_lds = reinterpret_cast<float *>(smem + (size_t)QT * npow2 * 8);  // [QT][d]
    const int tid = threadIdx.x, T = blockDim.x;
    const int64_t q0 = (int64_t)blockIdx.x * QT;
    const int nqt = (int)(nq - q0 < QT ? nq - q0 : QT);
    for (int t = tid; t < QT * d; t += T) {
        const int qi = t / d;
        q_lds[t] = qi < nqt ? queries[(size_t)q0 * d + t] : 0.0f;
    }
    for (int i = tid; i < QT * npow2; i += T) keys[i] = ~0ull;
    sync_block();
    const int lane32 = tid & 31;
    const int ng = d >> 2;
    const int nh = T >> 5;
    // Short vectors (at most 128 values: one 16-byte group per lane of the half wave): the lane's
    // share of every query stays in registers, and the distance loop reads no LDS at all.
    const bool in_regs = ng <= 32;
    float qrx[QT], qry[QT], qrz[QT], qrw[QT];
#pragma unroll
    for (int qi = 0; qi < QT; ++qi) {
        float4 t = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (in_regs && lane32 < ng) t = *reinterpret_cast<const float4 *>(q_lds + qi * d + 4 * lane32);
        qrx[qi] = t.x; qry[qi] = t.y; qrz[qi] = t.z; qrw[qi] = t.w;
    }
    // A half wave takes kRows (8; 4 with 8 queries) consecutive centroid rows per pass (their loads in flight together)
    // against the QT queries: kRows x QT lane sums per lane, reduced together (reduce_pairs), after
    // which lane l of the half wave holds the distance of pair l >> kShift = row * QT + query and
    // the pairs' keys are stored side by side.
    constexpr int kRows = QT == 8 ? 4 : 8, NP = kRows * QT;
    constexpr int kShift = NP == 32 ? 0 : NP == 16 ? 1 : 2;
    for (int l0 = (tid >> 5) * kRows; l0 < nlist; l0 += nh * kRows) {
        // (rows past the end: the last row again, never stored)
        const float4 *row0 = reinterpret_cast<const float4 *>(centroids + (size_t)l0 * d);
        const int last = nlist - 1 - l0;     // >= 0
        float acc[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i) acc[i] = 0.0f;
        for (int g = lane32; g < ng; g += 32) {
            float4 x[kRows];
#pragma unroll
            for (int r = 0; r < kRows; ++r) x[r] = row0[(r < last ? r : last) * ng + g];
#pragma unroll
            for (int qi = 0; qi < QT; ++qi) {
                float4 qv = make_float4(qrx[qi], qry[qi], qrz[qi], qrw[qi]);
                if (!in_regs) qv = *reinterpret_cast<const float4 *>(q_lds + qi * d + 4 * g);
#pragma unroll
                for (int r = 0; r < kRows; ++r) {
                    float e, a0 = acc[r * QT + qi];
                    e = qv.x - x[r].x; a0 = __builtin_fmaf(e, e, a0);
                    e = qv.y - x[r].y; a0 = __builtin_fmaf(e, e, a0);
                    e = qv.z - x[r].z; a0 = __builtin_fmaf(e, e, a0);
                    e = qv.w - x[r].w; a0 = __builtin_fmaf(e, e, a0);
                    acc[r * QT + qi] = a0;
                }
            }
        }
        const float dist = reduce_pairs<NP>(acc, lane32);
        const int pair = lane32 >> kShift;
        const int l = l0 + pair / QT, qi = pair % QT;
        // a distance is >= 0 (or NaN): its bit pattern orders like its value
        if ((lane32 & ((1 << kShift) - 1)) == 0 && l < nlist)
            keys[(size_t)qi * npow2 + l] = ((unsigned long long)__float_as_uint(dist) << 32) | (uint32_t)l;
    }
    sync_block();
    // Short probe lists (nprobe <= 64, at least 256 lists): one wave per query.  The keys are seen
    // as 64 S interleaved columns (S = 1 for nprobe <= 32, else 2; lane l, slot s holds column
    // 64 s + l); the nprobe-th smallest of the column minima (sorted across lanes and slots) is
    // an upper bound of the nprobe-th smallest key, so only the keys not above it can be
    // selected.  If at most 64 S keys qualify they are sorted the same way and the first nprobe
    // are the result; otherwise (rare) the whole workgroup takes the general path below.  Keys
    // are distinct, so either path gives the same list.
    __shared__ int general_path;
    if (nprobe <= 64 && npow2 >= 256) {
        if (tid == 0) general_path = 0;
        sync_block();
        const int wave = tid >> 6, lane = tid & 63;
        const int S = nprobe <= 32 ? 1 : 2;
        // ascending bitonic sort of the 64 S elements (element e = 64 slot + lane)
        auto sort_across = [&](unsigned long long (&key)[2]) {
            for (int size = 2; size <= 64 * S; size <<= 1) {
                for (int j = size >> 1; j > 0; j >>= 1) {
                    if (j >= 64) {            // partner in the other slot of the same lane (S == 2, size 128: ascending)
                        if (key[1] < key[0]) { const unsigned long long t = key[0]; key[0] = key[1]; key[1] = t; }
                        continue;
                    }
#pragma unroll
                    for (int sl = 0; sl < 2; ++sl) {
                        if (sl >= S) break;
                        const uint32_t olo = (uint32_t)__shfl_xor((int)(uint32_t)key[sl], j);
                        const uint32_t ohi = (uint32_t)__shfl_xor((int)(uint32_t)(key[sl] >> 32), j);
                        const unsigned long long other = ((unsigned long long)ohi << 32) | olo;
                        const int e = 64 * sl + lane;
                        const bool keep_min = ((lane & j) == 0) == ((e & size) == 0);
                        if (keep_min ? other < key[sl] : other > key[sl]) key[sl] = other;
                    }
                }
            }
        };
        unsigned long long *kq = keys + ((size_t)(wave < nqt ? wave : 0) * npow2);
        unsigned long long cut = 0;
        int c = 0;
        if (wave < nqt) {
            unsigned long long cmin[2] = {~0ull, ~0ull};
            for (int i = lane; i < npow2; i += 64 * S) {
                cmin[0] = kq[i] < cmin[0] ? kq[i] : cmin[0];
                if (S == 2) cmin[1] = kq[i + 64] < cmin[1] ? kq[i + 64] : cmin[1];
            }
            if (nprobe == 1) {   // the nearest list alone (assignment of a base set): a minimum, no sort
                unsigned long long m = cmin[0];
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) {
                    const uint32_t olo = (uint32_t)__shfl_xor((int)(uint32_t)m, off);
                    const uint32_t ohi = (uint32_t)__shfl_xor((int)(uint32_t)(m >> 32), off);
                    const unsigned long long other = ((unsigned long long)ohi << 32) | olo;
                    m = other < m ? other : m;
                }
                cmin[0] = m;       // every lane holds it: the bound below is the key itself
            } else {
                sort_across(cmin);
            }
            const unsigned long long at = (nprobe - 1) >= 64 ? cmin[1] : cmin[0];   // same choice in every lane
            const int src = (nprobe - 1) & 63;
            cut = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(at >> 32), src) << 32) |
                  (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)at, src);
            for (int i0 = 0; i0 < npow2; i0 += 64) c += __popcll(__ballot(kq[i0 + lane] <= cut));
            if (c > 64 * S) atomicOr(&general_path, 1);
        }
        sync_block();   // nothing has been moved yet: the general path finds every key in place
        if (!general_path) {
            if (wave < nqt) {
                // move the qualifying keys to the front (in place: none moves backwards)
                int at0 = 0;
                for (int i0 = 0; i0 < npow2; i0 += 64) {
                    const unsigned long long key = kq[i0 + lane];
                    const bool take = key <= cut;
                    const unsigned long long m = __ballot(take);
                    if (take) kq[at0 + __popcll(m & ((1ull << lane) - 1ull))] = key;
                    at0 += __popcll(m);
                }
                unsigned long long key[2];
                key[0] = lane < c ? kq[lane] : ~0ull;
                key[1] = (S == 2 && 64 + lane < c) ? kq[64 + lane] : ~0ull;
                if (nprobe > 1) sort_across(key);   // (one probe: c == 1, the key sits in lane 0)
                if (lane < nprobe) probes[(size_t)(q0 + wave) * nprobe + lane] = (int32_t)(key[0] & 0xffffffffu);
                if (64 + lane < nprobe) probes[(size_t)(q0 + wave) * nprobe + 64 + lane] = (int32_t)(key[1] & 0xffffffffu);
            }
            return;
        }
    }
    // Selection of the nprobe smallest keys of each query with bitonic networks; all sizes are
    // powers of two, so the index arithmetic is shifts and masks (lg_* are base-2 logarithms).
    // (1) runs of R >= nprobe keys are sorted, ascending and descending in turn;
    // (2) neighbouring runs are merged pairwise, keeping only the R smallest of the two: the
    //     element-wise minimum of an ascending and a descending run holds them as a bitonic
    //     sequence, which log2(R) exchange stages sort (again ascending / descending in turn);
    //     the surviving run stays where the pair's first run was, so after round r the live
    //     runs sit at multiples of R << r.  The last survivor, at 0, is ascending.
    const int lg_n = 31 - __builtin_clz(npow2);
    const int lg_half = lg_n - 1;
    int lg_r = 0;
    while ((1 << lg_r) < nprobe) ++lg_r;
    for (int lg_size = 1; lg_size <= lg_r; ++lg_size) {
        for (int lg_stride = lg_size - 1; lg_stride >= 0; --lg_stride) {
            const int stride = 1 << lg_stride;
            for (int w = tid; w < (QT << lg_half); w += T) {
                const int qi = w >> lg_half, i = w & ((1 << lg_half) - 1);
                const int lo = ((i >> lg_stride) << (lg_stride + 1)) | (i & (stride - 1));
                const int hi = lo + stride;
                const bool up = ((lo >> lg_size) & 1) == 0;
                unsigned long long *kq = keys + ((size_t)qi << lg_n);
                const unsigned long long x = kq[lo], y = kq[hi];
                if ((x > y) == up) { kq[lo] = y; kq[hi] = x; }
            }
            sync_block();
        }
    }
    const int R = 1 << lg_r;
    for (int lg_gap = lg_r; lg_gap < lg_n; ++lg_gap) {   // partner run = first run + (1 << lg_gap)
        const int lg_pairs = lg_n - lg_gap - 1;          // pairs per query in this round
        // element-wise minimum into the first run of each pair
        for (int w = tid; w < ((QT << lg_pairs) << lg_r); w += T) {
            const int i = w & (R - 1);
            const int pr = (w >> lg_r) & ((1 << lg_pairs) - 1);
            const int qi = w >> (lg_r + lg_pairs);
            unsigned long long *kq = keys + ((size_t)qi << lg_n) + ((size_t)pr << (lg_gap + 1));
            const unsigned long long x = kq[i], y = kq[(1 << lg_gap) + i];
            if (y < x) kq[i] = y;
        }
        sync_block();
        // sort the bitonic survivors: ascending for even pairs, descending for odd ones
        for (int lg_stride = lg_r - 1; lg_stride >= 0; --lg_stride) {
            const int stride = 1 << lg_stride;
            const int lg_ce = lg_r - 1;                  // exchanges per run and stage = R / 2
            for (int w = tid; w < ((QT << lg_pairs) << lg_ce); w += T) {
                const int i = w & ((1 << lg_ce) - 1);
                const int pr = (w >> lg_ce) & ((1 << lg_pairs) - 1);
                const int qi = w >> (lg_ce + lg_pairs);
                const int lo = ((i >> lg_stride) << (lg_stride + 1)) | (i & (stride - 1));
                const bool up = (pr & 1) == 0;
                unsigned long long *kq = keys + ((size_t)qi << lg_n) + ((size_t)pr << (lg_gap + 1));
                const unsigned long long x = kq[lo], y = kq[lo + stride];
                if ((x > y) == up) { kq[lo] = y; kq[lo + stride] = x; }
            }
            sync_block();
        }
    }
    for (int w = tid; w < nqt * nprobe; w += T) {
        const int qi = w / nprobe, p = w - qi * nprobe;
        probes[(size_t)(q0 + qi) * nprobe + p] = (int32_t)(keys[(size_t)qi * npow2 + p] & 0xffffffffu);
    }
}

// ---- nearest list of many vectors (assignment of a base set, training) ----
// The same rule as ivf_probe_kernel with one probe (exact distances in the R-order of exact_d2_half,
// ties to the smaller id).  Measuring every pair exactly is bound by the vector ALU (two
// operations per coordinate and pair).  Here the matrix cores score the pairs and the exact rule
// decides only where scores are too close:
//
//   scores   |x - c|^2 = |x|^2 + |c|^2 - 2 x.c with x and c taken relative to the mean mu of a few centroids,
//            the products by v_mfma_f32_32x32x16_bf16 on values split in two (hi hi + hi lo + lo hi),
//            256 vectors x 256 centroids per workgroup and step, the split made while a 32-column
//            slice is staged in LDS (double buffered), |x|^2 and |c|^2 summed on the way.
//   trackers a lane keeps, per 32 x 32 tile position, the least score, its centroid and the second least: 16
//            trackers per vector, each over a sixteenth of the centroids.
//   decision leasts within the margin of the best are compared by the exact rule (usually there is
//            just one: nothing to compare); a second least within the margin means that a centroid is not known:
//            the vector is marked (-1) and assign_fix_kernel measures it against every centroid.
//
// Margin: twice E = (2^-16 + (3 d + 16) 2^-24) 2 |x||c|max     split, binary32 accumulation
//                 + d 2^-24 |c|max^2 + d 2^-24 |x|^2             the norms
//                 + (d / 32 + 8) 2^-24 (|x| + |c|max)^2          the exact rule's own roundings
// 1,000,000 x 128 against 1024 lists: 1.33 ms with the marked vectors (9.3 ms measured exactly).  Rows of up to 128 values:
// assign_rows_kernel.  Longer ones, with the marked: 500,000 x 256 1.16 ms, x 384 1.63, 170,000 x 768 1.45.
constexpr int kAsgThreads = 512, kAsgTile = 256, kAsgSlice = 32, kAsgMaxD = 4096;
inline size_t assign_lds(int d) { return (size_t)2 * 4 * 4 * kAsgTile * 16 + (size_t)((d + kAsgSlice - 1) / kAsgSlice * kAsgSlice) * 4 + 2 * kAsgTile * 4 + 64; }

__global__ __launch_bounds__(kAsgThreads) void assign_mfma_kernel(const float *__restrict__ xs, int64_t n, int d,
                                                                  const float *__restrict__ cent, int nlist,
                                                                  int32_t *__restrict__ out) {
    typedef __bf16 b8 __attribute__((ext_vector_type(8)));
    typedef float v16f __attribute__((ext_vector_type(16)));
    extern __shared__ __align__(16) unsigned char smem[];
    // a buffer: [x hi, x lo, c hi, c lo][16-column step][8-column half][256 rows] of 8 values
    b8 *buf = reinterpret_cast<b8 *>(smem);
    constexpr int kPart = 4 * kAsgTile, kBuf = 4 * kPart;
    float *mu = reinterpret_cast<float *>(buf + 2 * kBuf);
    const int dpad = (d + kAsgSlice - 1) / kAsgSlice * kAsgSlice;
    float *xn2 = mu + dpad, *cn2 = xn2 + kAsgTile;
    uint32_t *cmax_bits = reinterpret_cast<uint32_t *>(cn2 + kAsgTile);
    int *namb = reinterpret_cast<int *>(cmax_bits + 1);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 31, half = lane >> 5;
    const int xg = wave & 3, cg = wave >> 2;       // this wave: 64 vectors, 128 centroids of the tile
    const int64_t x0 = (int64_t)blockIdx.x * kAsgTile;
    for (int t = tid; t < dpad; t += kAsgThreads) {
        float sum = 0.0f;
        for (int i = 0; i < 16; ++i) sum += t < d ? cent[(size_t)((int64_t)i * nlist >> 4) * d + t] : 0.0f;
        mu[t] = sum * (1.0f / 16.0f);
    }
    if (tid == 0) { *cmax_bits = 0; *namb = 0; }
    sync_block();
    // staging: two threads per row, 16 columns of a slice each
    const int srow = tid >> 1, sstep = tid & 1;
    const int64_t xr = x0 + srow < n ? x0 + srow : n - 1;
    const float *xrow = xs + (size_t)xr * d + sstep * 16;
    float4 xv[4], cv[4];
    float xsum = 0.0f, csum = 0.0f;
    auto load = [&](const float *crow, int k0) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const bool in = k0 + sstep * 16 + 4 * g < d;
            xv[g] = in ? *reinterpret_cast<const float4 *>(xrow + k0 + 4 * g) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            cv[g] = in ? *reinterpret_cast<const float4 *>(crow + k0 + 4 * g) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
    };
    auto split = [&](const float (&v)[16], b8 *hi_at, b8 *lo_at) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            b8 hi, lo;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                hi[e] = (__bf16)v[8 * h + e];
                lo[e] = (__bf16)(v[8 * h + e] - (float)hi[e]);
            }
            hi_at[h * kAsgTile] = hi;
            lo_at[h * kAsgTile] = lo;
        }
    };
    auto stage = [&](int which, int k0) {
        b8 *at = buf + which * kBuf + sstep * 2 * kAsgTile + srow;
        float vx[16], vc[16];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 m = *reinterpret_cast<const float4 *>(mu + k0 + sstep * 16 + 4 * g);   // (columns past d: all zero)
            const float ax[4] = {xv[g].x - m.x, xv[g].y - m.y, xv[g].z - m.z, xv[g].w - m.w};
            const float ac[4] = {cv[g].x - m.x, cv[g].y - m.y, cv[g].z - m.z, cv[g].w - m.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                xsum = __builtin_fmaf(ax[e], ax[e], xsum);
                csum = __builtin_fmaf(ac[e], ac[e], csum);
                vx[4 * g + e] = ax[e];
                vc[4 * g + e] = -2.0f * ac[e];
            }
        }
        split(vx, at, at + kPart);
        split(vc, at + 2 * kPart, at + 3 * kPart);
    };
    uint32_t m1[2][4], m2[2][4];
    int i1[2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int t = 0; t < 4; ++t) { m1[u][t] = m2[u][t] = 0x7f800000u; i1[u][t] = 0; }
    uint32_t cmax2 = 0;        // (bit patterns: a centroid that is no number is the largest, and everybody is measured exactly)
    const int nblk = (nlist + kAsgTile - 1) / kAsgTile, nk = dpad / kAsgSlice;
    for (int cb = 0; cb < nblk; ++cb) {
        const int cr = cb * kAsgTile + srow;
        const float *crow = cent + (size_t)(cr < nlist ? cr : nlist - 1) * d + sstep * 16;
        xsum = 0.0f;
        csum = 0.0f;
        v16f acc[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[u][t][i] = 0.0f;
        load(crow, 0);
        stage(0, 0);
        sync_block();
        for (int kc = 0; kc < nk; ++kc) {
            if (kc + 1 < nk) load(crow, (kc + 1) * kAsgSlice);
            const b8 *b = buf + (kc & 1) * kBuf + half * kAsgTile + col;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                b8 xh[2], xl[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    xh[u] = b[ks * 2 * kAsgTile + xg * 64 + u * 32];
                    xl[u] = b[kPart + ks * 2 * kAsgTile + xg * 64 + u * 32];
                }
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const b8 ch = b[2 * kPart + ks * 2 * kAsgTile + cg * 128 + t * 32];
                    const b8 cl = b[3 * kPart + ks * 2 * kAsgTile + cg * 128 + t * 32];
#pragma unroll
                    for (int u = 0; u < 2; ++u) acc[u][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ch, xh[u], acc[u][t], 0, 0, 0);
#pragma unroll
                    for (int u = 0; u < 2; ++u) acc[u][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ch, xl[u], acc[u][t], 0, 0, 0);
#pragma unroll
                    for (int u = 0; u < 2; ++u) acc[u][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cl, xh[u], acc[u][t], 0, 0, 0);
                }
            }
            if (kc + 1 < nk) stage((kc + 1) & 1, (kc + 1) * kAsgSlice);
            sync_block();
        }
        xsum += __shfl_xor(xsum, 1);
        csum += __shfl_xor(csum, 1);
        if (sstep == 0) {
            xn2[srow] = xsum;
            cn2[srow] = cr < nlist ? csum : __builtin_inff();     // (rows past the end never win)
            if (cr < nlist) cmax2 = max(cmax2, __float_as_uint(csum));
        }
        sync_block();
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const float xb = xn2[xg * 64 + u * 32 + col];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 c2 = *reinterpret_cast<const float4 *>(cn2 + cg * 128 + t * 32 + 8 * q + 4 * half);
                    const float cq[4] = {c2.x, c2.y, c2.z, c2.w};
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        // (a score below zero is one within the margin of zero)
                        const float f = __builtin_fmaxf((acc[u][t][4 * q + s] + xb) + cq[s], 0.0f);
                        const uint32_t v = __float_as_uint(f);
                        const bool less = v < m1[u][t];
                        const uint32_t hi = less ? m1[u][t] : v;
                        m2[u][t] = m2[u][t] < hi ? m2[u][t] : hi;
                        m1[u][t] = less ? v : m1[u][t];
                        i1[u][t] = less ? cb * 16 + 4 * q + s : i1[u][t];
                    }
                }
            }
        }
    }
    // the trackers of every vector side by side (over the staging buffers, which are done with)
    uint32_t *t1 = reinterpret_cast<uint32_t *>(smem), *t2 = t1 + 16 * kAsgTile;
    int *tc = reinterpret_cast<int *>(t2 + 16 * kAsgTile);
    uint32_t *amb = reinterpret_cast<uint32_t *>(tc + 16 * kAsgTile);      // [256] (trackers << 8) | vector
    atomicMax(cmax_bits, cmax2);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int at = ((cg * 2 + half) * 4 + t) * kAsgTile + xg * 64 + u * 32 + col;
            const int i = i1[u][t];
            t1[at] = m1[u][t];
            t2[at] = m2[u][t];
            tc[at] = (i >> 4) * kAsgTile + cg * 128 + t * 32 + 8 * ((i & 15) >> 2) + 4 * half + (i & 3);
        }
    sync_block();
    if (tid < kAsgTile && x0 + tid < n) {
        const float c2 = __uint_as_float(*cmax_bits), x2 = xn2[tid];
        const float xl = trim::sqrt_rn(x2), cl = trim::sqrt_rn(c2);
        constexpr float kUlp = 1.0f / 16777216.0f;
        const float e = (1.0f / 65536.0f + (3.0f * d + 16.0f) * kUlp) * 2.0f * xl * cl + d * kUlp * (c2 + x2) +
                        (d / 32 + 8) * kUlp * (xl + cl) * (xl + cl);
        uint32_t best = 0x7f800000u, sec = 0x7f800000u;
        for (int k = 0; k < 16; ++k) {
            const uint32_t a = t1[k * kAsgTile + tid], b = t2[k * kAsgTile + tid];
            best = a < best ? a : best;
            sec = b < sec ? b : sec;
        }
        const float thr = __uint_as_float(best) + 2.0f * e;
        uint32_t close = 0;
        int one = 0;
        for (int k = 0; k < 16; ++k)
            if (!(__uint_as_float(t1[k * kAsgTile + tid]) > thr)) { close |= 1u << k; one = tc[k * kAsgTile + tid]; }
        if (!(e < 1e30f) || !(e > 1e-30f) || !(__uint_as_float(sec) > thr)) out[x0 + tid] = -1;
        else if ((close & (close - 1)) == 0) out[x0 + tid] = one;
        else amb[atomicAdd(namb, 1)] = (close << 8) | (uint32_t)tid;
    }
    sync_block();
    const int na = *namb;
    for (int i = tid >> 5; i < na; i += kAsgThreads >> 5) {        // a half wave per undecided vector
        const int x = (int)(amb[i] & 255u);
        uint32_t close = amb[i] >> 8;
        const float *q = xs + (size_t)(x0 + x) * d;
        unsigned long long best = ~0ull;
        while (close) {
            const int k = __ffs((int)close) - 1;
            close &= close - 1;
            const int c = tc[k * kAsgTile + x];
            const float dist = exact_d2_half(cent + (size_t)c * d, q, d, lane & 31);
            const unsigned long long key = ((unsigned long long)__float_as_uint(dist) << 32) | (uint32_t)c;
            best = key < best ? key : best;
        }
        if ((lane & 31) == 0) out[x0 + x] = (int32_t)(best & 0xffffffffu);
    }
}

// The same for rows of at most 128 values (KS: steps of 16 values, 4 or 8), where a wave keeps its vectors' operands
// in registers: 64 vectors per wave for all columns, and only the centroids pass through the LDS, converted once per
// workgroup of 256 vectors.
//   operands  values relative to mu, scaled by a power of two, as ONE binary16 value each (x', c'); what is scored is
//             |x' - c'|^2, so that what rounding moved counts against the distance and not against the lengths: with r' = |x' - c'|,
//             whoever may be nearest has r' <= r'min + 2 (moved(x) + moved(c)max).  |x'|^2 and |c'|^2 come in by one
//             more step of the matrix cores, as three binary16 pieces each against 2^15.
//   trackers  scores are ordered by their bits, as signed numbers (one below zero is within the bound of zero), the low ones
//             replaced by the centroid's number; a lane keeps the three least of every other centroid of its quarter:
//             one insertion of the number, one minimum and two medians of three a score
//   schedule  waves 0 to 3 and 4 to 7 share the SIMDs; the ones multiply while the others track
//   decision  everybody within the bound is measured by the exact rule, four pairs to a half wave; the vector is marked only
//             where the third of a tracker is within the bound too
// 1,000,000 x 128 against 1024 lists: 650 us (1215 with the kernel above), 65,536: 41 us (77), and hardly any marks: 5 us
// for them (103).  A workgroup: 18,000 clocks until its vectors are in registers (rows from memory, by all workgroups at once), 3,700 a stage
// of 64 centroids (vector ALU: 4 operations a score, 5 a value converted), 6,000 for the decision.
constexpr int kAsrCols = 128;
template <int KS>
struct AsrShape {
    static constexpr int kTiles = 8 / KS, kRows = 64 * kTiles, kPitch = kRows + 8;     // 32-row tiles per wave; centroids per stage (and spare ones: bank spread)
    static constexpr int kStage = (KS * 2 + 1) * kPitch * 16;                          // bytes
};
template <int KS>
__global__ __launch_bounds__(kAsgThreads, 2) void assign_rows_kernel(const float *__restrict__ xs, int64_t n, int d,
                                                                     const float *__restrict__ cent, int nlist,
                                                                     int32_t *__restrict__ out) {
    typedef _Float16 h8 __attribute__((ext_vector_type(8)));
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    typedef float v16f __attribute__((ext_vector_type(16)));
    typedef _Float16 h4 __attribute__((ext_vector_type(4)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef float f4 __attribute__((ext_vector_type(4)));
    using Shape = AsrShape<KS>;
    constexpr int TT = Shape::kTiles, R = Shape::kRows, P = Shape::kPitch, kTrk = 8;
    constexpr int kAreaA = 2 * Shape::kStage, kAreaB = 3 * kTrk * kAsgTile * 4;
    __shared__ __align__(16) unsigned char s_buf[kAreaA > kAreaB ? kAreaA : kAreaB];   // the stages; then the trackers
    __shared__ __align__(16) float s_mu[kAsrCols];
    __shared__ float s_xn[kAsgTile], s_xm[kAsgTile];
    __shared__ uint32_t s_pair[kAsgTile * 2 * kTrk];                            // vector | centroid << 8
    __shared__ unsigned long long s_best[kAsgTile];
    __shared__ uint32_t s_top[2], s_cmax, s_mmax;
    __shared__ int s_np;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5, xg = wave & 3, cg = wave >> 2;
    const int64_t x0 = (int64_t)blockIdx.x * kAsgTile;
    // KS lanes bring a row, 16 bytes each at a time: values 4 (g KS + s_ks) and the next three
    const int s_row = tid / KS, s_ks = tid & (KS - 1);
    auto bring = [&](const float *row, f4 (&v)[4]) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int k = 4 * (g * KS + s_ks);
            v[g] = *reinterpret_cast<const f4 *>(row + (k < d ? k : 0));       // (columns past d: not used)
        }
    };
    // the vectors, all on their way at once
    constexpr int NX = kAsgTile / R;
    f4 xv[NX][4];
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        const int r = i * R + s_row;
        bring(xs + (size_t)(x0 + r < n ? x0 + r : n - 1) * d, xv[i]);
    }
    if (tid < kAsrCols) {           // mean and spread of 16 centroids
        float v[16], sum = 0.0f, most = 0.0f;
        const int t = tid < d ? tid : 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = cent[(size_t)((int64_t)i * nlist >> 4) * d + t];
#pragma unroll
        for (int i = 0; i < 16; ++i) sum += v[i];
        const float mu = sum * (1.0f / 16.0f);
        uint32_t top = 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) { most = __builtin_fabsf(v[i] - mu); top = max(top, __float_as_uint(most)); }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) top = max(top, (uint32_t)__shfl_xor((int)top, off));
        s_mu[tid] = mu;
        if (lane == 0) s_top[wave] = top;
    }
    if (tid == 0) { s_cmax = s_mmax = 0; s_np = 0; }
    if (tid < kAsgTile) s_best[tid] = ~0ull;
    sync_block();
    const uint32_t top = max(s_top[0], s_top[1]);
    const bool usable = __uint_as_float(top) > 1e-30f && __uint_as_float(top) < 1e30f;
    const float sc = __uint_as_float((uint32_t)((usable ? 6 - ((int)(top >> 23) - 127) : 0) + 127) << 23);     // (the spread: 2^6 .. 2^7)
    constexpr float kPiece = 32768.0f, kReach = 2.0e9f;
    // three pieces of a norm, in the slots from `at` on; the other side of them is kPiece
    auto pieces = [](h8 &f, int at, float norm) {
        const float q = norm * (1.0f / kPiece);
        const _Float16 p1 = (_Float16)q, p2 = (_Float16)(q - (float)p1), p3 = (_Float16)((q - (float)p1) - (float)p2);
        f[at] = p1; f[at + 1] = p2; f[at + 2] = p3;
    };
    // a row's values as operands, times `by`, into buffer b; norm: of what is stored, moved: by rounding (the row's sums, in all its lanes)
    auto put = [&](int b, const f4 (&a)[4], float by, float &norm, float &moved, float &most) {
        norm = moved = most = 0.0f;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int k = 4 * (g * KS + s_ks);
            const f4 m = *reinterpret_cast<const f4 *>(s_mu + k);
            const float scale = k < d ? by : 0.0f;
            h2 f[2];
#pragma unroll
            for (int e = 0; e < 4; e += 2) {       // (the power of two: one rounding, that of the difference)
                const f2 v = {__builtin_fmaf(a[g][e], scale, -(m[e] * scale)), __builtin_fmaf(a[g][e + 1], scale, -(m[e + 1] * scale))};
                const h2 h = __builtin_convertvector(v, h2);
                const f2 back = __builtin_convertvector(h, f2);
                const float r0 = v[0] - back[0], r1 = v[1] - back[1];
                moved = __builtin_fmaf(r0, r0, moved);
                moved = __builtin_fmaf(r1, r1, moved);
                most = __builtin_fmaxf(most, __builtin_fmaxf(__builtin_fabsf(v[0]), __builtin_fabsf(v[1])));
                norm = __builtin_amdgcn_fdot2(h, h, norm, false);
                f[e / 2] = h;
            }
            *reinterpret_cast<h4 *>(s_buf + b * Shape::kStage + ((k >> 3) * P + s_row) * 16 + (k & 4) * 2) = h4{f[0][0], f[0][1], f[1][0], f[1][1]};
        }
        auto over = [&](auto &&f) {
            f(std::integral_constant<int, 1>());
            f(std::integral_constant<int, 2>());
            if constexpr (KS == 8) f(std::integral_constant<int, 4>());
        };
        over([&](auto bit) {
            constexpr int kBit = decltype(bit)::value;
            norm = norm + lane_xor<kBit>(norm);
            moved = moved + lane_xor<kBit>(moved);
            most = __builtin_fmaxf(most, lane_xor<kBit>(most));
        });
    };
    f4 ahead[4];
    auto load = [&](int st) {
        const int c = st * R + s_row;
        bring(cent + (size_t)(c < nlist ? c : nlist - 1) * d, ahead);
    };
    uint32_t cmax2 = 0, mmax2 = 0;        // (bit patterns: a centroid that is no number is the largest, and everybody is measured exactly)
    auto stage = [&](int st) {
        const bool real = st * R + s_row < nlist;
        float norm, moved, most;
        put(st & 1, ahead, sc, norm, moved, most);
        if (s_ks == 0) {
            h8 f = {(_Float16)65504.0f, (_Float16)65504.0f, (_Float16)65504.0f, (_Float16)kPiece, (_Float16)kPiece, (_Float16)kPiece, 0, 0};
            if (real) {              // (rows past the end: far away; should one be within the bound all the same, the vector is marked)
                cmax2 = max(cmax2, norm < kReach ? __float_as_uint(norm) : 0x7f800000u);
                mmax2 = max(mmax2, __float_as_uint(moved));
                pieces(f, 0, norm);
            }
            *reinterpret_cast<h8 *>(s_buf + (st & 1) * Shape::kStage + (KS * 2 * P + s_row) * 16) = f;
        }
    };
    load(0);
    // -2 x: R vectors at a time through the LDS
    h8 xo[2][KS + 1];
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        float norm, moved, most;
        put(i & 1, xv[i], -2.0f * sc, norm, moved, most);
        if (s_ks == 0) {
            norm *= 0.25f;
            const bool fits = most < 65000.0f && norm < kReach;        // (else out of the 16-bit range: nothing is known)
            s_xn[i * R + s_row] = fits ? norm : __builtin_nanf("");
            s_xm[i * R + s_row] = moved * 0.25f;
            h8 f = {(_Float16)kPiece, (_Float16)kPiece, (_Float16)kPiece, 0, 0, 0, 0, 0};
            pieces(f, 3, fits ? norm : 0.0f);
            *reinterpret_cast<h8 *>(s_buf + (i & 1) * Shape::kStage + (KS * 2 * P + s_row) * 16) = f;
        }
        sync_block();
        if (xg * 64 / R == i) {
            const h8 *b = reinterpret_cast<const h8 *>(s_buf + (i & 1) * Shape::kStage) + xg * 64 % R + col;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) xo[u][ks] = b[(ks * 2 + half) * P + u * 32];
                const h8 zero = {0, 0, 0, 0, 0, 0, 0, 0}, f = b[KS * 2 * P + u * 32];
                xo[u][KS] = half == 0 ? f : zero;
            }
        }
    }
    sync_block();
    stage(0);
    const int nst = (nlist + R - 1) / R;
    load(nst > 1 ? 1 : 0);
    int m1[2][2], m2[2][2], m3[2][2];             // [32 vectors][every other centroid]
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int k = 0; k < 2; ++k) m1[u][k] = m2[u][k] = m3[u][k] = 0x7f800000;
    const int bits = 32 - __builtin_clz(nst * TT * 16 - 1);
    const uint32_t number = (1u << bits) - 1u;
    uint32_t keep = ~number;
    asm("" : "+v"(keep));        // (a vector register: an instruction reads one scalar)
    v16f acc[2];
    auto multiply = [&](int st, int tt) {
        const h8 *b = reinterpret_cast<const h8 *>(s_buf + (st & 1) * Shape::kStage) + (cg * TT + tt) * 32 + col;
        h8 c[KS + 1];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) c[ks] = b[(ks * 2 + half) * P];
        c[KS] = b[KS * 2 * P];                     // (the same for both halves: the vectors' side of the upper one is zero)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[u][i] = 0.0f;
#pragma unroll
        for (int ks = 0; ks <= KS; ++ks)
#pragma unroll
            for (int u = 0; u < 2; ++u) acc[u] = __builtin_amdgcn_mfma_f32_32x32x16_f16(c[ks], xo[u][ks], acc[u], 0, 0, 0);
    };
    auto track = [&](int tile) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            uint32_t id = (uint32_t)(tile * 16 + i);
            asm("" : "+s"(id));          // (a scalar of its own: v_and_or_b32)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int k = i & 1;
                // (not in assembly: the compiler has to see who reads a result of the matrix cores)
                const int v = (int)((__float_as_uint(acc[u][i]) & keep) | id);
                asm("v_med3_i32 %0, %1, %2, %0" : "+v"(m3[u][k]) : "v"(v), "v"(m2[u][k]));
                asm("v_med3_i32 %0, %1, %2, %0" : "+v"(m2[u][k]) : "v"(v), "v"(m1[u][k]));
                m1[u][k] = v < m1[u][k] ? v : m1[u][k];
            }
        }
    };
    sync_block();
#pragma unroll 1
    for (int st = 0; st < nst; ++st) {
        if (cg == 0) {
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
                multiply(st, tt);
                if (tt == 0 && st + 1 < nst) {
                    stage(st + 1);
                    load(st + 2 < nst ? st + 2 : nst - 1);
                }
                track(st * TT + tt);
            }
        } else {
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
                if (st + tt > 0) track(st * TT + tt - 1);
                if (tt == 0 && st + 1 < nst) {
                    stage(st + 1);
                    load(st + 2 < nst ? st + 2 : nst - 1);
                }
                multiply(st, tt);
            }
        }
        sync_block();
    }
    if (cg != 0) track(nst * TT - 1);
    // the trackers of every vector side by side (over the stages, which are done with)
    int *trk = reinterpret_cast<int *>(s_buf);                  // [first, second, third][kTrk][256]
    if (cmax2) atomicMax(&s_cmax, cmax2);
    if (mmax2) atomicMax(&s_mmax, mmax2);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            int *at = trk + ((cg * 2 + half) * 2 + k) * kAsgTile + xg * 64 + u * 32 + col;
            at[0] = m1[u][k];
            at[kTrk * kAsgTile] = m2[u][k];
            at[2 * kTrk * kAsgTile] = m3[u][k];
        }
    sync_block();
    if (tid < kAsgTile && x0 + tid < n) {
        int key[2 * kTrk], third = 0x7fffffff;
#pragma unroll
        for (int k = 0; k < 2 * kTrk; ++k) key[k] = trk[k * kAsgTile + tid];
#pragma unroll
        for (int k = 0; k < kTrk; ++k) third = min(third, trk[(2 * kTrk + k) * kAsgTile + tid]);
        int best = key[0];
#pragma unroll
        for (int k = 1; k < kTrk; ++k) best = min(best, key[k]);
        constexpr float kUlp = 1.0f / 16777216.0f;
        const float lost = trim::sqrt_rn((float)d) * (1.0f / 16384.0f);             // (subnormal 16-bit operands may count as zero)
        const float c2 = __uint_as_float(s_cmax), x2 = s_xn[tid];
        const float mc = trim::sqrt_rn(__uint_as_float(s_mmax)) * 1.001f, mx = trim::sqrt_rn(s_xm[tid]) * 1.001f;
        const float cl = trim::sqrt_rn(c2) + mc, xl = trim::sqrt_rn(x2) + mx;
        // what moved an operand: rounding, the subtraction of mu, flushing; errors of a score: sums, flushed operands, the pieces of
        // the norms; the exact rule's own
        const float moved = mc + mx + (cl + xl) * 2.0f * kUlp + 2.0f * lost;
        const float e = (4.0f * d + 64.0f) * kUlp * (xl * cl + cl * cl + xl * xl) + 8.0f + (d / 32 + 8) * kUlp * (xl + cl) * (xl + cl);
        const float coarse = 1.0f + __uint_as_float((uint32_t)(127 - 21 + bits) << 23);      // (what the numbers took)
        const float reach = trim::sqrt_rn(__builtin_fmaxf(__int_as_float(best), 0.0f) * coarse + e) + 2.0f * moved;
        const float thr = (reach * reach + e) * coarse, real = (e / sc) / sc;
        bool known = real < 1e30f && real > 1e-30f && __int_as_float(third) > thr;
        int close = 0, one = 0;
#pragma unroll
        for (int k = 0; k < 2 * kTrk; ++k) {
            const int id = (int)((uint32_t)key[k] & number), tile = id >> 4, i = id & 15, kg = (k % kTrk) >> 2, kh = (k % kTrk) >> 1 & 1;
            const bool in = __int_as_float(key[k]) <= thr;
            key[k] = in ? tile / TT * R + (kg * TT + tile % TT) * 32 + 8 * (i >> 2) + 4 * kh + (i & 3) : -1;
            known = known && key[k] < nlist;
            close += in ? 1 : 0;
            one = in ? key[k] : one;
        }
        if (!known || close == 0) {
            out[x0 + tid] = -1;
        } else if (close == 1) {
            out[x0 + tid] = one;
        } else {
            int at = atomicAdd(&s_np, close);
#pragma unroll
            for (int k = 0; k < 2 * kTrk; ++k)
                if (key[k] >= 0) s_pair[at++] = (uint32_t)tid | (uint32_t)key[k] << 8;
        }
    }
    sync_block();
    const int np = s_np, lane32 = tid & 31, at4 = 4 * lane32 < d ? 4 * lane32 : 0;      // (at most 32 groups of four)
    for (int i0 = (tid >> 5) * 4; i0 < np; i0 += (kAsgThreads >> 5) * 4) {
        uint32_t pair[4];
        float part[4];
        f4 q[4], c[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            pair[i] = s_pair[i0 + i < np ? i0 + i : i0];
            q[i] = *reinterpret_cast<const f4 *>(xs + (size_t)(x0 + (pair[i] & 255u)) * d + at4);
            c[i] = *reinterpret_cast<const f4 *>(cent + (size_t)(pair[i] >> 8) * d + at4);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {                        // (exact_d2_half's order)
            float sum = 0.0f;
#pragma unroll
            for (int e = 0; e < 4; ++e) { const float v = q[i][e] - c[i][e]; sum = __builtin_fmaf(v, v, sum); }
            part[i] = 4 * lane32 < d ? sum : 0.0f;
        }
        const float dist = half_reduce_x4(part, lane32);
        const int i = half_reduce_x4_row(lane32);
        const uint32_t p = i == 0 ? pair[0] : i == 1 ? pair[1] : i == 2 ? pair[2] : pair[3];
        if (half_reduce_x4_writer(lane32) && i0 + i < np)
            atomicMin(&s_best[p & 255u], ((unsigned long long)__float_as_uint(dist) << 32) | (p >> 8));
    }
    sync_block();
    if (tid < kAsgTile && x0 + tid < n && s_best[tid] != ~0ull) out[x0 + tid] = (int32_t)(s_best[tid] & 0xffffffffu);
}

// The vectors that assign_rows_kernel or assign_mfma_kernel marked: every centroid measured by the exact rule, eight
// vectors at a time (ivf_probe_kernel's distance loop).  A workgroup looks after up to kFixSpan
// vectors, so that even a mark in a hundred fills its groups; the last one takes as many vectors' worth of work as it has, or nearly
// (ten iterations of 65,536 x 128 against 1024, two or three marks a workgroup: 208 -> 101 us, 96 to 110 by machine).
// T: 1024 threads where there is at most a workgroup per CU, where few are marked (rows of up to 128 values) and for rows of more than 1024
// (whole assignments, 40,000 x 1536 in 200 lists: 324 / 337 us), else 512 (us, 1024 / 512
// threads: 16,384 x 768 36 / 45, x 1536 126 / 163, 8000 x 768, all marked, 2415 / 3189, whole assignments of 200,000 x 128 171 / 174, x 32
// 114 / 129; 30,000 x 384 37 / 35, 500,000 x 384 172 / 154, 50,000 x 384, all marked, 1365 / 1270).  Norms over four decades mark three
// quarters of 200,000 x 128 by assign_rows_kernel's one binary16 product (1745 us, 1875 in all), half by assign_mfma_kernel's three
// of split values (1350, 1614).
constexpr int kFixSpan = 1024;
template <int T>
__global__ __launch_bounds__(T) void assign_fix_kernel(const float *__restrict__ xs, int64_t n, int d,
                                                                 const float *__restrict__ cent, int nlist,
                                                                 int span, int32_t *__restrict__ out) {
    constexpr int QT = 8, kRows = 4;
    extern __shared__ __align__(16) unsigned char smem[];
    float *q_lds = reinterpret_cast<float *>(smem);                      // [QT][d]
    __shared__ int todo[kFixSpan];
    __shared__ int count;
    __shared__ unsigned long long best[QT];
    const int tid = threadIdx.x;
    const int64_t x0 = (int64_t)blockIdx.x * span;
    if (tid == 0) count = 0;
    sync_block();
    for (int i = tid; i < span; i += T)
        if (x0 + i < n && out[x0 + i] < 0) todo[atomicAdd(&count, 1)] = i;
    sync_block();
    const int total = count, ng = d >> 2;
    for (int g0 = 0; g0 < total; g0 += QT) {
        const int nqt = total - g0 < QT ? total - g0 : QT;
        if (tid < QT) best[tid] = ~0ull;
        for (int t = tid; t < QT * d; t += T) {
            const int qi = t / d;
            q_lds[t] = xs[(size_t)(x0 + todo[g0 + (qi < nqt ? qi : 0)]) * d + (t - qi * d)];
        }
        sync_block();
        auto measure = [&](auto wide) {              // against so many vectors
            int tid = threadIdx.x;                   // (opaque: addresses are made anew, not kept for the other widths as well)
            asm volatile("" : "+v"(tid));
            const int lane32 = tid & 31;
            constexpr int Q = decltype(wide)::value, NP = Q * kRows, kShift = NP == 32 ? 0 : NP == 16 ? 1 : 2;
            unsigned long long mine = ~0ull;
            constexpr int kStep = (T >> 5) * kRows;
            const int g1 = lane32 < ng ? lane32 : 0;         // the first group of the next rows is on its way while these are measured
            float4 x[kRows], next[kRows];
            auto load = [&](int l0, int g, float4 (&to)[kRows]) {
#pragma unroll
                for (int r = 0; r < kRows; ++r) to[r] = reinterpret_cast<const float4 *>(cent)[(size_t)(l0 + r < nlist ? l0 + r : nlist - 1) * ng + g];
            };
            load((tid >> 5) * kRows, g1, next);
            for (int l0 = (tid >> 5) * kRows; l0 < nlist; l0 += kStep) {
                float acc[NP];
#pragma unroll
                for (int i = 0; i < NP; ++i) acc[i] = 0.0f;
#pragma unroll
                for (int r = 0; r < kRows; ++r) x[r] = next[r];
                load(l0 + kStep, g1, next);
                for (int g = lane32; g < ng; g += 32) {
                    if (g != lane32) load(l0, g, x);
#pragma unroll
                    for (int qi = 0; qi < Q; ++qi) {
                        const float4 qv = *reinterpret_cast<const float4 *>(q_lds + qi * d + 4 * g);
#pragma unroll
                        for (int r = 0; r < kRows; ++r) {
                            float e, a0 = acc[r * Q + qi];
                            e = qv.x - x[r].x; a0 = __builtin_fmaf(e, e, a0);
                            e = qv.y - x[r].y; a0 = __builtin_fmaf(e, e, a0);
                            e = qv.z - x[r].z; a0 = __builtin_fmaf(e, e, a0);
                            e = qv.w - x[r].w; a0 = __builtin_fmaf(e, e, a0);
                            acc[r * Q + qi] = a0;
                        }
                    }
                }
                const float dist = reduce_pairs<NP>(acc, lane32);
                const int l = l0 + (lane32 >> kShift) / Q;
                const unsigned long long key = ((unsigned long long)__float_as_uint(dist) << 32) | (uint32_t)l;
                if (l < nlist && key < mine) mine = key;
            }
            atomicMin(&best[(lane32 >> kShift) % Q], mine);
        };
        if (nqt <= 2) measure(std::integral_constant<int, 2>());
        else if (nqt <= 4) measure(std::integral_constant<int, 4>());
        else measure(std::integral_constant<int, 8>());
        sync_block();
        if (tid < nqt) out[x0 + todo[g0 + tid]] = (int32_t)(best[tid] & 0xffffffffu);
        sync_block();
    }
}

// ---- processing order: queries grouped by their first probed list ----
// Single workgroup, counting sort with an LDS histogram (nbucket <= 32768 buckets; list ids
// are folded modulo nbucket, which still puts equal lists together).  Lists appear in
// ascending bucket order; the order of the queries inside a bucket is unspecified.
__global__ __launch_bounds__(1024) void query_order_kernel(const int32_t *__restrict__ probes,
                                                           int64_t nq, int nprobe, int nbucket,
                                                           int32_t *__restrict__ order) {
    extern __shared__ __align__(16) unsigned char smem[];
    int *hist = reinterpret_cast<int *>(smem);  // [nbucket], then running cursors
    __shared__ int part[16];
    const int tid = threadIdx.x, T = blockDim.x;
    for (int b = tid; b < nbucket; b += T) hist[b] = 0;
    // the first kKeep queries of a thread stay in registers for both passes, their loads in flight together
    constexpr int kKeep = 16;
    uint32_t mine[kKeep];
#pragma unroll
    for (int i = 0; i < kKeep; ++i) {
        const int64_t q = tid + (int64_t)i * T;
        mine[i] = q < nq ? (uint32_t)probes[(size_t)q * nprobe] % (uint32_t)nbucket : 0xffffffffu;
    }
    sync_block();
#pragma unroll
    for (int i = 0; i < kKeep; ++i)
        if (mine[i] != 0xffffffffu) atomicAdd(&hist[mine[i]], 1);
    for (int64_t q = tid + (int64_t)kKeep * T; q < nq; q += T) {
        const uint32_t l = (uint32_t)probes[(size_t)q * nprobe];
        atomicAdd(&hist[l % (uint32_t)nbucket], 1);
    }
    sync_block();
    // exclusive prefix over the buckets: each thread owns a contiguous run; the runs' sums are
    // scanned inside each wave, then across the (at most 16) waves
    const int per = (nbucket + T - 1) / T;
    const int lo = tid * per < nbucket ? tid * per : nbucket;
    const int hi = lo + per < nbucket ? lo + per : nbucket;
    int sum = 0;
    for (int b = lo; b < hi; ++b) sum += hist[b];
    const int lane = tid & 63, wave = tid >> 6;
    int incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int v = __shfl_up(incl, off);
        if (lane >= off) incl += v;
    }
    if (lane == 63) part[wave] = incl;
    sync_block();
    int before = 0;
    for (int w = 0; w < wave; ++w) before += part[w];
    int run = before + incl - sum;
    for (int b = lo; b < hi; ++b) { const int c = hist[b]; hist[b] = run; run += c; }
    sync_block();
#pragma unroll
    for (int i = 0; i < kKeep; ++i)
        if (mine[i] != 0xffffffffu) order[atomicAdd(&hist[mine[i]], 1)] = (int32_t)(tid + i * T);
    for (int64_t q = tid + (int64_t)kKeep * T; q < nq; q += T) {
        const uint32_t l = (uint32_t)probes[(size_t)q * nprobe];
        order[atomicAdd(&hist[l % (uint32_t)nbucket], 1)] = (int32_t)q;
    }
}

}  // namespace trim
