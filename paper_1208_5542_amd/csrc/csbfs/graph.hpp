// Internal layout of a partitioned graph (not installed).
#pragma once

#include <memory>
#include <vector>

#include "common.hpp"

namespace csbfs {

// Rows longer than kBigRow adjacency entries are expanded through the chunk
// queue, kBigChunk entries per queue item, instead of inside their frontier
// word's wavefront.
constexpr int kBigRow = 128;
constexpr int kBigChunk = 512;
// Queue items of a row of len entries; rows may have up to 2^31 - 2.
__host__ __device__ inline int32_t row_items(int32_t len) { return len > kBigRow ? (len - 1) / kBigChunk + 1 : 0; }

// Alignment of every array carved out of a caller's buffer.
constexpr int64_t kAlign = 256;
inline int64_t align_up(int64_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Upper bound on the chunk-queue items of all rows expanded at once, from
// the adjacency total alone: a row of d > kBigRow entries needs
// ceil(d / kBigChunk) < d / kBigChunk + 1 items, and there are fewer than
// nnz / kBigRow such rows.
inline int64_t big_items_bound(int64_t nnz) { return nnz / kBigChunk + nnz / kBigRow + 2; }

// Byte offsets of the arrays of a graph inside its device buffer, and of the
// build's temporaries inside the build scratch; both depend on (n, p,
// n_tuples) only, and the scratch on whether the entries are sorted as a whole
// (where `sort` allows it and there are neither few nor very many of them).
struct GraphLayout {
    int64_t n, P, R, W, B, nnz, ntile;
    // graph buffer
    int64_t row_ptr, col_base, col, dir, deg, pull_off, pull_col, head, live, qoff, small, graph_bytes;
    // build scratch
    bool sorted;  // entries sorted as a whole (radix.hip)
    int64_t radix, cnt, sums, nnzb, misc, queues, scan, scratch_bytes;
};
int graph_layout(int64_t n, int64_t n_tuples, int32_t p, GraphLayout *out, bool sort = true);

}  // namespace csbfs

struct csbfs_graph {
    int device = -1;
    int64_t n = 0;          // vertices
    int32_t P = 1;          // virtual processors
    int64_t R = 0;          // n / P
    int64_t W = 0;          // R / 64 words per piece
    int64_t n_tuples = 0;
    int64_t nnz = 0;
    int64_t max_block_nnz = 0;
    std::vector<int64_t> big_items;  // per block-row: queue items if every row were expanded at once
    int64_t device_bytes = 0;
    csbfs::DeviceBlock owned;         // the graph buffer when the library allocated it
    // block b = i * P + j: rows are sources u in R_j, columns targets in R_i
    int32_t *row_ptr = nullptr;       // [P*P][R + 1], offsets within the block
    int64_t *col_base = nullptr;      // [P*P + 1], block start in col
    std::vector<int64_t> col_base_host;
    uint32_t *col = nullptr;          // [nnz], local target ids
    uint64_t *dir = nullptr;          // [P*P][W], V_{i,j} = non-empty rows of block (i, j)
    int32_t *deg = nullptr;           // [n], adjacency entries of u over all blocks
    // Pull layout: the rows of v in blocks (j, i), j = P-1 down to 0, merged
    // into one row of global ids in decreasing order (processor i's view of
    // column v of its block-row; by symmetry the same entries as the blocks)
    int64_t *pull_off = nullptr;      // [n + 1]
    uint32_t *pull_col = nullptr;     // [nnz]
    uint32_t *head = nullptr;         // [2n]: the first two ids of v's merged row (0xFFFFFFFF: none)
    uint64_t *live = nullptr;         // [n / 64]: vertices with at least one adjacency entry
    int64_t *qoff = nullptr;          // [P + 1]: processor r's chunk-queue region
    unsigned long long *scratch = nullptr;  // small reduction scratch
};

namespace csbfs {
int graph_device_check(const csbfs_graph *g);
// Sort every block row (descending target id) in place, unless `sorted` says
// it is (the long rows are then only queued); tmp has nnz entries
// of scratch, queues and q_count come from the build scratch.
// Rows above kLongRow entries are sorted (and copied into the pull layout) by
// whole workgroups; the sort leaves their numbers b * R + u in two queues.
constexpr int kLongRow = 1024;
struct LongRows {
    const int64_t *rows[2];
    const unsigned long long *count;  // [2]
    int64_t cap[2];
};
int64_t sort_queue_cap(int64_t nnz, int which);
LongRows sort_long_rows(const int64_t *queues, const unsigned long long *q_count, int64_t nnz);
int sort_rows_desc(uint32_t *col, uint32_t *tmp, const int32_t *row_ptr, const int64_t *col_base, int64_t R,
                   int32_t P, int64_t nnz, int64_t *queues, unsigned long long *q_count, int32_t *err,
                   bool sorted, hipStream_t st);
// Every entry of the tuples to its sorted place in col (all blocks, rows in
// decreasing id order), and the place after the last entry of a non-empty row u
// of block b to row_end[b * (n / P + 1) + u]; *err is set by a tuple id outside
// [0, n). `keys` holds 8 bytes an entry and may overlap col.
int64_t radix_scratch_bytes(int64_t nnz);
int sort_entries(const int64_t *src, const int64_t *dst, int64_t n_tuples, int64_t n, int32_t P, void *scratch,
                 void *keys, uint32_t *col, int32_t *row_end, int32_t *err, hipStream_t st);
// off[v] = sum of deg[u] for u < v (off has n + 1 entries; off[n] = total);
// tile_sum holds scan_tiles(n) entries of scratch.
int64_t scan_tiles(int64_t n);
int degree_offsets(const int32_t *deg, int64_t n, int64_t *off, int64_t *tile_sum, hipStream_t st);
// A batch engine on caller memory: a device block of csbfs_batch_engine_bytes
// and a pinned two-word host buffer (each may be null: then allocated and
// owned by the engine); `st` runs its initial zeroing.
int batch_engine_make(const csbfs_graph *g, int32_t max_roots, int32_t max_levels, uint32_t flags, void *mem,
                      unsigned long long *host_ctl, hipStream_t st, csbfs_batch_engine **out);
void batch_engine_release(csbfs_batch_engine *e);
// csbfs_batch_bfs with a place of its own for each root's levels (n each, apart
// from each other).
int batch_bfs_into(csbfs_batch_engine *e, const int64_t *roots, int32_t n_roots, int32_t *const *level,
                   csbfs_level_stats *stats, int32_t stats_cap, int32_t *n_levels, void *stream);
}
