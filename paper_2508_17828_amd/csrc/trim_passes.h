// Arguments and sizes of the passes of trim_mark.h: what the host side needs of them.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace trim {

constexpr int kFinishPiece = 32768, kFinishList = 8192;   // candidates, listed candidates at a time (finish)

constexpr float kCertainLow = 1e-30f, kCertainHigh = 1e30f;      // squared radii of which filter_kernel tells who passes for certain
constexpr int kFinishGood = 1, kFinishBad = 2;      // FinishArgs::only
struct FinishArgs {
    // index, queries, candidate structure: as in SearchArgs
    const uint8_t *codes;
    const float *dlx;
    const float *codebooks;
    int64_t n;
    int32_t d, M, dsub;
    const float *queries;
    int64_t nq;
    const int32_t *order;
    int64_t slot0, nslots;    // this launch: places [slot0, slot0 + nslots) of the query order
    int32_t by_query;         // a query's rows of the workspace are at its number, else at its place less slot0
    const float *lut;         // tables by query number, or (lut_by_row) by row of the workspace; null: built here
    int32_t lut_by_row;
    const uint32_t *bad;      // by query number: the table is not the centroids' (or null)
    int32_t only;             // 0: all queries; else those that are not bad, or those that are
    const int64_t *list_offsets;
    const int32_t *probes;
    const int32_t *seg;       // see InvertArgs (null: no lists)
    int32_t nlist, nseg, max_cand;
    int32_t P, Mp;
    float two_gamma;
    // this pass: candidates [lo, hi) of every query
    int32_t lo, hi;
    int32_t all;              // every candidate of the pass counts as marked, and stays it
    int32_t range;            // the threshold is radius2; else tau_of[q * tau_stride], or +inf where tau_of is null
    float radius2;
    const float *tau_of;
    int32_t tau_stride;
    // by scan-order number
    int32_t *totals;          // [rows] candidates of the query
    uint32_t *possible;       // [rows][words] marks
    const uint32_t *certain;  // range: of these, who passes whatever the table sums to in detail (or null)
    float *g;                 // [rows][words * 32] bounds of the marked (and partial sums between table phases)
    int64_t words;
    int32_t *n_scanned, *n_exact;   // n_exact: range only (the marked are the survivors), zeroed by the host
    uint32_t *mask;                 // range only: the caller's survivor mask
    int64_t mask_words;
    // LDS carve-up
    uint32_t off_q, off_segp, off_segd, off_bits, off_ring;
};

// Distance tables of many queries (lut_tile_kernel).
constexpr int kLutQueries = 32;      // queries per workgroup
inline bool lut_tiled(int dsub, bool fs) { return fs ? dsub == 2 : dsub == 4 || dsub == 8 || dsub == 16; }
struct LutArgs {
    const float *queries;
    int64_t nq;
    int32_t d;
    const float *codebooks;
    int32_t nsub;
    const int32_t *order;
    int64_t slot0, nslots;
    int32_t by_slot;
    float *lut;
    uint32_t *bad;
};

// Which queries scan a list, and where: inv[start[l] .. start[l+1]) = (workspace row, scan-order number
// of the list's first vector).
struct InvertArgs {
    const int32_t *probes;
    int64_t nq;
    const int32_t *order;
    int64_t slot0, nslots;
    int32_t by_query, nseg, nlist, max_cand;
    const int64_t *list_offsets;
    int64_t n;
    int32_t *cnt;      // [nlist], zero; then the running slots
    int32_t *start;    // [nlist + 1]
    int32_t *tasks;    // [nlist + 1] prefix of the filter's tiles
    int32_t *row_tasks;   // [nlist + 1] prefix of the measure pass's
    int2 *inv;
    int32_t *seg;      // [rows][2][nseg]: the queries' segment tables (segment_table), made here once for all passes
    __device__ __forceinline__ int64_t query(int64_t slot) const {
        const int64_t q = order ? order[slot0 + slot] : slot0 + slot;
        return q >= 0 && q < nq ? q : -1;
    }
};

// ---- filter: who can pass, on the matrix cores (see filter_kernel) ----
constexpr int kFltRows = 512, kFltQ = 128, kFltThreads = 512, kFltSlice = 32;
constexpr int kMsrRows = 256, kMsrBlock = 512;        // measure: rows at a time, queries per task
// LDS of measure_kernel<wq, wr>: two buffers of rows and of queries (two and four spare per 8 columns), the rows' norms, the
// waiting queries, and the centroids' means.
constexpr size_t measure_lds(int d, int wq, int wr) {
    return 2 * 4 * ((size_t)(64 * wr + 2) + 64 * wq + 4) * 16 + 2 * 64 * wr * 4 + 5 * (size_t)(2 * 64 * wq) * 4 + 64 + (size_t)d * 4;
}
// Values per sub-vector after padding: what a 16-byte operand holds, a part or a multiple of it.
__host__ __device__ inline int filter_padded(int dsub, bool fs) {
    if (fs) return dsub == 2 ? 2 : 0;
    return dsub <= 4 ? 4 : dsub <= 8 ? 8 : dsub <= 16 ? 16 : dsub <= 32 ? 32 : 0;
}
struct FilterArgs {
    // index
    const uint8_t *codes;
    const float *dlx;
    const float *codebooks;
    int64_t n;
    int32_t d, M, dsub, nsub, ncent;   // M: code bytes; nsub subspaces of ncent centroids
    const float *queries;
    int64_t nq;
    const int32_t *order;
    int64_t slot0, nslots;
    int32_t by_query;
    const int64_t *list_offsets;
    int32_t nlist, nseg;
    const int32_t *inv_start;
    const int2 *inv;
    const int32_t *tasks, *row_tasks;
    float two_gamma;
    int32_t range;
    float radius2;
    const float *tau_of;
    int32_t tau_stride;
    int32_t lo, hi;
    const int32_t *totals;
    uint32_t *possible;
    uint32_t *certain;         // range: who passes for certain, or null
    int64_t words;
    // prepared operands (work space)
    // measure
    const float *base;
    float *d2;                 // [rows][words * 32]
    int32_t msr_block;         // queries per task
    int32_t kpad_rows;         // d rounded up to kFltSlice
    _Float16 *q16_rows;        // [rows][kpad_rows]: q16 without the padding between sub-vectors (or q16 itself)
    int32_t padded, kpad;      // values per sub-vector, per vector (a multiple of kFltSlice)
    float *mu;                 // [d] means of the centroids
    uint32_t *max_bits;        // largest |centroid - mean|
    _Float16 *books;           // [kpad / padded][ncent][padded]
    _Float16 *q16;             // [rows][kpad]: -2 (q - mu), scaled
    float *qpar;               // [rows][2]: |q - mu|^2, what rounding to 16 bits moved q by
};

struct ReplayArgs {
    const int32_t *ids;
    const float *base, *queries;
    int32_t d;
    int64_t n, nq;
    const int64_t *list_offsets;
    const int32_t *probes;
    const int32_t *seg;         // see InvertArgs (null: no lists)
    int32_t nlist, nseg, max_cand;
    int32_t k, batch;
    int32_t lo, hi;             // candidates of this pass; lo == 0: R is empty
    int32_t mid;                // the first batch's end, where it is taken with the pass after it; else 0
    int32_t picks;              // pick_kernel: vectors taken (k .. kPicks)
    const int32_t *order;       // queries that it does not name are left alone
    int64_t slot0, nslots;
    const int32_t *totals;
    const uint32_t *possible;
    const float *g, *d2;        // d2: lower bounds of the exact distances
    int64_t words;
    int32_t *out_ids;           // [nq][k]: R between passes, the results after the last
    float *out_d2;
    int32_t *n_exact;
    uint32_t *mask;
    int64_t mask_words;
    // range_exact_kernel: possible and d2 are updated, results counted per chunk
    uint32_t *bits;
    float *d2_out;
    float radius2;
    int32_t chunk, nchunk;
    int32_t *counts;
    uint32_t off_segp, off_segd, off_cl, off_g, off_d2, off_id, off_rd2, off_rid, off_q, off_key, off_todo;
};
// pick_kernel: most vectors taken; those taken, most results and least vectors of the index per query where the next pass is long; largest batch; least
// vectors of the batch per result beyond kPickMost.
constexpr int kPicks = 128, kPickLong = 64, kPickMost = 10, kPickVectors = 16, kPickBatch = 1024, kPickGroup = 4;
constexpr int kReplayThreads = 512, kReplayCap = 2048;   // (a power of two)

// ---- few queries (trim_few.h) ----
constexpr int kBoundThreads = 512;
constexpr int kSettleFirst = 4096, kSettleList = 2048;   // largest k + batch, listed candidates at a time
constexpr int settle_threads(int E) { return E <= 2 ? 1024 : 512; }   // (R's registers)
struct FewArgs {
    // index, queries, candidate structure: as in SearchArgs
    const float *base;
    const uint8_t *codes;
    const float *dlx;
    const float *codebooks;
    const int32_t *ids;
    int64_t n;
    int32_t d, M, dsub;
    const float *queries;
    int64_t nq;
    const int32_t *order;
    const float *lut;
    const int64_t *list_offsets;
    const int32_t *probes;
    int32_t nlist, nseg, max_cand;
    int32_t P, Mp;            // table phases
    float two_gamma;
    int32_t k, batch;
    // work space, by place in the query order
    int32_t *totals;          // candidates of the query
    float *g;                 // [stride] their bounds
    int64_t stride;           // (a multiple of 16)
    float *least;             // [(stride + 63) / 64] the least bound of every 64
    float *d2;                // [k + batch] exact distances of the seed and the first batch, or null: settle measures
    float *d2_all;            // [stride] exact distances of those that may be survivors (few_rows_kernel), or null: settle measures
    float *r_d2;              // [r_stride] R between launches
    int32_t *r_id;
    int32_t *r_n;             // survivors so far (by place: the order may name a query twice)
    int32_t r_stride, lo, hi; // candidates of this pass
    int32_t *out_ids;
    float *out_d2;
    int32_t *n_scanned, *n_exact;
    uint32_t *mask;
    int64_t mask_words;
    uint32_t off_q, off_segp, off_segd, off_rd2, off_rid, off_fd2, off_key, off_todo;
};

}  // namespace trim
