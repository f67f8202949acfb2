// Graph partitioning: the p x p sub-block grid of Sec. V.A (Eq. abc, Eq.
// sub-block), one CSR per block, and the directory vectors of Eq. dir-vec.
//
// Block b = i * P + j holds, for every source u in R_j (row u - j*R), its
// neighbours v in R_i as local ids v - i*R. Tuple {u, v} contributes u -> v
// to block (owner(v), owner(u)) and v -> u to block (owner(u), owner(v)); a
// self-loop contributes twice to one row. Rows are built by sorting the
// entries (radix.hip) or, for few or very many of them, by a counting pass and
// a scatter whose rows are sorted afterwards (sort.hip); row offsets come from
// a per-block scan (tile sums, scan of tile sums, local scans).
#include <algorithm>
#include <vector>

#include "device.hpp"
#include "graph.hpp"

namespace csbfs {
namespace {

constexpr int kThreads = 256;
constexpr int kTileItems = 4;
constexpr int kTile = kThreads * kTileItems;

// Scans of rows: of their counts (sums), or (kEnds) of the places after their
// last entries, 0 for an empty row (maxima, as places grow with the rows).
template <bool kEnds>
__device__ __forceinline__ long long scan_op(long long a, long long b) {
    return kEnds ? (a > b ? a : b) : a + b;
}

// Exclusive over the workgroup, from 0; the total in *total.
template <bool kEnds>
__device__ long long block_excl_scan_ll(long long v, long long *total) {
    __shared__ long long ws[kThreads / 64];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    long long incl = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const long long t = __shfl_up(incl, d, 64);
        if (lane >= d) incl = scan_op<kEnds>(incl, t);
    }
    if (lane == 63) ws[wid] = incl;
    const long long up = __shfl_up(incl, 1, 64);
    __syncthreads();
    long long before = 0, tot = 0;
    for (int k = 0; k < kThreads / 64; ++k) {
        if (k < wid) before = scan_op<kEnds>(before, ws[k]);
        tot = scan_op<kEnds>(tot, ws[k]);
    }
    __syncthreads();
    *total = tot;
    return lane > 0 ? scan_op<kEnds>(before, up) : before;
}

__global__ void k_count(const int64_t *src, const int64_t *dst, int64_t m, int64_t n, int64_t R,
                        int32_t P, int32_t *cnt, int32_t *err) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < m;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t u = src[t], v = dst[t];
        if (u < 0 || u >= n || v < 0 || v >= n) {
            *err = 1;
            continue;
        }
        const int64_t ou = u / R, ov = v / R;
        atomicAdd(&cnt[(ov * P + ou) * R + (u - ou * R)], 1);  // u -> v
        atomicAdd(&cnt[(ou * P + ov) * R + (v - ov * R)], 1);  // v -> u
    }
}

// tile totals of every block's rows, cnt[b * stride + u]: sums[b * ntile + t]
template <bool kEnds>
__global__ __launch_bounds__(kThreads) void k_tile_sum(const int32_t *cnt, int64_t stride, int64_t R,
                                                       int64_t ntile, long long *sums) {
    const int64_t t = blockIdx.x, b = blockIdx.y;
    long long s = 0;
    for (int64_t k = threadIdx.x; k < kTile; k += kThreads) {
        const int64_t u = t * kTile + k;
        if (u < R) s = scan_op<kEnds>(s, (uint32_t)cnt[b * stride + u]);
    }
    __shared__ long long red[kThreads / 64];
    for (int d = 32; d > 0; d >>= 1) s = scan_op<kEnds>(s, __shfl_xor(s, d, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        long long tot = 0;
        for (int k = 0; k < kThreads / 64; ++k) tot = scan_op<kEnds>(tot, red[k]);
        sums[b * ntile + t] = tot;
    }
}

// in-place exclusive scan of each block's tile totals; block totals to nnz[b]
template <bool kEnds>
__global__ __launch_bounds__(kThreads) void k_tile_scan(long long *sums, int64_t ntile,
                                                        long long *nnz) {
    const int64_t b = blockIdx.x;
    long long carry = 0;
    for (int64_t base = 0; base < ntile; base += kThreads) {
        const int64_t t = base + threadIdx.x;
        const long long v = t < ntile ? sums[b * ntile + t] : 0;
        long long tot;
        const long long ex = block_excl_scan_ll<kEnds>(v, &tot);
        if (t < ntile) sums[b * ntile + t] = scan_op<kEnds>(carry, ex);
        carry = scan_op<kEnds>(carry, tot);
    }
    if (threadIdx.x == 0) nnz[b] = carry;
}

// row_ptr[b * (R + 1) + u] = entries of block b's rows before u. Counts become
// the scatter cursors (cursor[u] = row_ptr[u]); ends lie in row_ptr itself
// (stride R + 1), and each thread replaces those it read. An end is a place
// among all blocks' entries, so the block's first place is taken off.
template <bool kEnds>
__global__ __launch_bounds__(kThreads) void k_tile_apply(int32_t *cnt, int64_t stride, int64_t R, int64_t ntile,
                                                         const long long *sums, const int64_t *col_base, int32_t *row_ptr) {
    const int64_t t = blockIdx.x, b = blockIdx.y;
    const int64_t u0 = t * kTile + threadIdx.x * kTileItems;
    const long long first = kEnds ? col_base[b] : 0;
    long long v[kTileItems];
    long long mine = 0;
    for (int k = 0; k < kTileItems; ++k) {
        const int64_t u = u0 + k;
        v[k] = u < R ? (uint32_t)cnt[b * stride + u] : 0;
        mine = scan_op<kEnds>(mine, v[k]);
    }
    long long tot;
    const long long before = block_excl_scan_ll<kEnds>(mine, &tot);
    long long x = scan_op<kEnds>(scan_op<kEnds>(sums[b * ntile + t], before), first);
    for (int k = 0; k < kTileItems; ++k) {
        const int64_t u = u0 + k;
        if (u < R) {
            row_ptr[b * (R + 1) + u] = (int32_t)(x - first);
            if (!kEnds) cnt[b * stride + u] = (int32_t)x;
            x = scan_op<kEnds>(x, v[k]);
            if (u == R - 1) row_ptr[b * (R + 1) + R] = (int32_t)(x - first);
        }
    }
}

__global__ void k_scatter(const int64_t *src, const int64_t *dst, int64_t m, int64_t R, int32_t P,
                          int32_t *cursor, const int64_t *col_base, uint32_t *col) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < m;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t u = src[t], v = dst[t];
        const int64_t ou = u / R, ov = v / R;
        const int64_t b1 = ov * P + ou, b2 = ou * P + ov;
        const int32_t p1 = atomicAdd(&cursor[b1 * R + (u - ou * R)], 1);
        col[col_base[b1] + p1] = (uint32_t)(v - ov * R);
        const int32_t p2 = atomicAdd(&cursor[b2 * R + (v - ov * R)], 1);
        col[col_base[b2] + p2] = (uint32_t)(u - ou * R);
    }
}

// V_{i,j}: bit u of block b's vector = row u of block b is non-empty.
__global__ void k_directory(const int32_t *row_ptr, int64_t R, int64_t W, int64_t nblocks,
                            uint64_t *dir) {
    const int lane = threadIdx.x & 63;
    const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t w = wave; w < nblocks * W; w += nwaves) {
        const int64_t b = w / W, q = w - b * W;
        const int32_t *rp = row_ptr + b * (R + 1) + q * 64 + lane;
        const bool nz = rp[1] > rp[0];
        const uint64_t m = __ballot(nz);
        if (lane == 0) dir[w] = m;
    }
}

// deg[u] = adjacency entries of u over all blocks of its column; big[i] +=
// the expansion-queue items that the rows of block-row i would need if every
// row were expanded at once (the capacity of processor i's chunk queue). The
// sums go to memory once per workgroup: device-scope atomics on one address
// are serialized, and one per wave was most of this kernel's time (scale 20:
// 269 us, now 46 us).
__global__ __launch_bounds__(kThreads) void k_degree(const int32_t *row_ptr, int64_t R, int32_t P, int64_t n,
                                                     int32_t *deg, unsigned long long *big_items) {
    __shared__ unsigned long long big[64];  // P <= 64
    if (threadIdx.x < 64) big[threadIdx.x] = 0;
    __syncthreads();
    for (int64_t base = blockIdx.x * (int64_t)blockDim.x; base < n;
         base += (int64_t)gridDim.x * blockDim.x) {
        const int64_t u = base + threadIdx.x;
        const bool ok = u < n;
        const int64_t j = ok ? u / R : 0, ul = ok ? u - j * R : 0;
        int32_t d = 0;
        for (int32_t i = 0; i < P; ++i) {
            if (!ok) continue;
            const int32_t *rp = row_ptr + ((int64_t)i * P + j) * (R + 1) + ul;
            const int32_t len = rp[1] - rp[0];
            d += len;
            const int32_t items = row_items(len);
            if (items) atomicAdd(&big[i], (unsigned long long)items);
        }
        if (ok) deg[u] = d;
    }
    __syncthreads();
    if (threadIdx.x < P && big[threadIdx.x]) atomicAdd(&big_items[threadIdx.x], big[threadIdx.x]);
}

// Consistency of a built graph: the largest column id (must be below R) and
// the degree total (must equal nnz). One pair of atomics per workgroup (one
// per wave took 392 us of atomics on two addresses at scale 20; now 72).
__global__ __launch_bounds__(kThreads) void k_check(const uint32_t *col, int64_t nnz, const int32_t *deg, int64_t n,
                                                    unsigned long long *out) {
    __shared__ uint32_t wmax[kThreads / 64];
    uint32_t mx = 0;
    unsigned long long ds = 0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t quads = nnz / 4;  // col starts at a multiple of 256 bytes
    for (int64_t k = t; k < quads; k += stride) {
        const uint4 c = reinterpret_cast<const uint4 *>(col)[k];
        mx = max(max(max(mx, c.x), max(c.y, c.z)), c.w);
    }
    for (int64_t k = quads * 4 + t; k < nnz; k += stride) mx = max(mx, col[k]);
    for (int64_t u = t; u < n; u += stride) ds += (unsigned long long)deg[u];
    for (int d = 32; d > 0; d >>= 1) {
        mx = max(mx, (uint32_t)__shfl_xor(mx, d, 64));
        ds += __shfl_xor(ds, d, 64);
    }
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kThreads / 64; ++w) mx = max(mx, wmax[w]);
        atomicMax(&out[0], (unsigned long long)mx);
    }
    block_add<kThreads / 64>(ds, &out[1]);
}

__global__ void k_count_m(const int32_t *level, const int32_t *deg, int64_t n,
                          unsigned long long *out) {
    unsigned long long s = 0;
    for (int64_t u = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; u < n;
         u += (int64_t)gridDim.x * blockDim.x)
        if (level[u] >= 0) s += (unsigned long long)deg[u];
    for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d, 64);
    if ((threadIdx.x & 63) == 0 && s) atomicAdd(out, s);
}

// Merge the rows of v in blocks (j, i), j = P-1 down to 0, into one row of
// global ids: each block row is already in decreasing order and block j
// holds the ids of R_j, so the merged row is in decreasing order. The row's
// first two ids are also kept beside each other per vertex (head; 0xFFFFFFFF
// where the row is shorter), so a pull can test them without the row.
//
// A plain copy of nnz ids, bound by memory as long as no lane follows a hub's
// row alone: a wavefront takes 64 vertices of one processor and, block after
// block, spreads the entries of their 64 rows evenly over its lanes; rows
// above kLongRow entries, which would hold such a wave for milliseconds, are
// copied by whole workgroups (k_pull_long) from the sort's queues. Scale 20,
// 4 x 4: one thread per vertex took 25.97 ms for the 33.5M entries (its
// time was the largest hub's row), the two kernels 0.15 ms (2.1 TB/s).
__device__ __forceinline__ void put_id(uint32_t id, int64_t pos, int64_t first, int64_t v, uint32_t *pull_col,
                                       uint32_t *head) {
    pull_col[pos] = id;
    if (pos - first < 2) head[2 * v + (pos - first)] = id;
}

__global__ __launch_bounds__(kThreads) void k_pull_fill(const int32_t *row_ptr, const int64_t *col_base,
                                                        const uint32_t *col, int64_t R, int32_t P, int64_t n,
                                                        const int64_t *pull_off, uint32_t *pull_col,
                                                        uint32_t *head) {
    constexpr int kUn = 4;  // entries in flight per lane
    const int lane = threadIdx.x & 63;
    const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t g = wave; g < n / 64; g += nwaves) {
        const int64_t v = (g << 6) + lane, i = (g << 6) / R, vl = v - i * R;  // R is a multiple of 64
        const int64_t first = pull_off[v];
        const int64_t deg = pull_off[v + 1] - first;
        for (int64_t k = deg; k < 2; ++k) head[2 * v + k] = 0xFFFFFFFFu;
        int64_t d = first;
        for (int32_t j = P - 1; j >= 0; --j) {
            const int64_t b = (int64_t)j * P + i;
            const int32_t *rp = row_ptr + b * (R + 1) + vl;
            const int32_t rs = rp[0], len = rp[1] - rs;
            const int32_t mine = len > kLongRow ? 0 : len;
            const int32_t incl = wave_incl_scan_i32(mine);
            const int32_t total = __shfl(incl, 63, 64), excl = incl - mine;
            const uint32_t *src = col + col_base[b];
            const uint32_t base = (uint32_t)(j * R);
            for (int32_t e0 = 0; e0 < total; e0 += 64 * kUn) {
                uint32_t id[kUn];
                int64_t at[kUn], f[kUn];
                int o[kUn];
#pragma unroll
                for (int k = 0; k < kUn; ++k) {
                    const int32_t e = min(e0 + 64 * k + lane, total - 1);
                    o[k] = owner_lane(excl, e);
                    const int32_t x = e - __shfl(excl, o[k], 64);
                    id[k] = base + src[__shfl(rs, o[k], 64) + x];
                    at[k] = shfl64(d, o[k]) + x;
                    f[k] = shfl64(first, o[k]);
                }
#pragma unroll
                for (int k = 0; k < kUn; ++k)
                    if (e0 + 64 * k + lane < total) put_id(id[k], at[k], f[k], (g << 6) + o[k], pull_col, head);
            }
            d += len;
        }
    }
}

// The rows above kLongRow entries (two queues of row numbers b * R + u).
__global__ __launch_bounds__(kThreads) void k_pull_long(const int32_t *row_ptr, const int64_t *col_base,
                                                        const uint32_t *col, int64_t R, int32_t P,
                                                        const int64_t *pull_off, uint32_t *pull_col, uint32_t *head,
                                                        LongRows q) {
    constexpr int kUn = 4;
    const int64_t n0 = (int64_t)q.count[0] < q.cap[0] ? (int64_t)q.count[0] : q.cap[0];
    const int64_t n1 = (int64_t)q.count[1] < q.cap[1] ? (int64_t)q.count[1] : q.cap[1];
    // the longest rows first
    for (int64_t k = blockIdx.x; k < n0 + n1; k += gridDim.x) {
        const int64_t row = k < n1 ? q.rows[1][k] : q.rows[0][k - n1];
        const int64_t b = row / R, vl = row - b * R;
        const int32_t j = (int32_t)(b / P), i = (int32_t)(b - (int64_t)j * P);
        const int64_t v = (int64_t)i * R + vl, first = pull_off[v];
        int64_t d = first;
        for (int32_t jj = P - 1; jj > j; --jj) {
            const int32_t *rp = row_ptr + ((int64_t)jj * P + i) * (R + 1) + vl;
            d += rp[1] - rp[0];
        }
        const int32_t *rp = row_ptr + b * (R + 1) + vl;
        const int32_t rs = rp[0], len = rp[1] - rs;
        const uint32_t *src = col + col_base[b] + rs;
        const uint32_t base = (uint32_t)(j * R);
        // 64-bit places: a row may end within one step of 2^31
        for (int64_t e0 = threadIdx.x; e0 < len; e0 += kUn * kThreads) {
            uint32_t id[kUn];
#pragma unroll
            for (int u = 0; u < kUn; ++u) {
                const int64_t e = e0 + u * kThreads;
                id[u] = src[e < len ? e : len - 1];
            }
#pragma unroll
            for (int u = 0; u < kUn; ++u) {
                const int64_t e = e0 + u * kThreads;
                if (e < len) put_id(base + id[u], d + e, first, v, pull_col, head);
            }
        }
    }
}

// Vertices with at least one adjacency entry, one bit each.
__global__ void k_live(const int32_t *deg, int64_t n, uint64_t *live) {
    const int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const uint64_t b = __ballot(v < n && deg[v] > 0);
    if ((threadIdx.x & 63) == 0 && v < n) live[v >> 6] = b;
}

// Builds of this many entries sort them (radix.hip) instead of counting,
// scattering and sorting rows. R-MAT, 4 x 4, in us (sort, counting), in memory
// of the caller's: 2^17 entries 313, 321; 2^18 313, 369; 2^20 358, 582; 2^25
// 1780, 6136; 2^31 (8 x 8) 148 ms, 406. (csbfs_graph_build adds its allocations:
// above the 2 GiB that are kept, about 30 ms a GiB where the memory was given back
// just before and is cleared first.) Above 2^31, the places do not fit 32 bits.
// The sort needs 8.25 bytes of scratch an entry, where counting needs 4 p n and
// a quarter byte an entry: at 2^31 entries on the 8 x 8 grid 17.0 GiB against
// 2.6. A build that cannot have the sort's scratch counts instead.
constexpr int64_t kSortMin = int64_t(1) << 18, kSortMax = int64_t(1) << 31;

constexpr int kMiscWords = 64;  // build flags and counters: err, sort queue counts, check, big items

int check_sizes(int64_t n, int64_t n_tuples, int32_t p, const char *who) {
    if (n_tuples < 0) return fail(CSBFS_EINVAL, std::string(who) + ": negative tuple count");
    if (n < 64 || n >= ((int64_t)1 << 31)) return fail(CSBFS_ERANGE, std::string(who) + ": need 64 <= n < 2^31");
    if (p < 1 || p > 64 || n % p != 0 || (n / p) % 64 != 0)
        return fail(CSBFS_ERANGE, std::string(who) + ": need 1 <= p <= 64, p | n and 64 | n/p");
    if (n_tuples > ((int64_t)1 << 40)) return fail(CSBFS_ERANGE, std::string(who) + ": too many tuples");
    return CSBFS_OK;
}

}  // namespace

int graph_layout(int64_t n, int64_t n_tuples, int32_t p, GraphLayout *L, bool sort) {
    const int rc = check_sizes(n, n_tuples, p, "graph layout");
    if (rc) return rc;
    GraphLayout g{};
    g.n = n;
    g.P = p;
    g.R = n / p;
    g.W = g.R / 64;
    g.B = (int64_t)p * p;
    g.nnz = 2 * n_tuples;
    g.ntile = (g.R + kTile - 1) / kTile;
    int64_t o = 0;
    auto take = [&o](int64_t bytes) {
        const int64_t at = o;
        o += align_up(bytes > 0 ? bytes : 1);
        return at;
    };
    g.row_ptr = take(4 * g.B * (g.R + 1));
    g.col_base = take(8 * (g.B + 1));
    g.col = take(4 * g.nnz);
    g.pull_col = take(4 * g.nnz);  // right after col: together they hold 8 bytes an entry for the build's sort
    g.dir = take(8 * g.B * g.W);
    g.deg = take(4 * n);
    g.pull_off = take(8 * (n + 1));
    g.head = take(8 * n);
    g.live = take(8 * (n / 64));
    g.qoff = take(8 * (g.P + 1));
    g.small = take(8 * 64);
    g.graph_bytes = o;
    o = 0;
    g.sorted = sort && g.nnz >= kSortMin && g.nnz <= kSortMax;
    if (g.sorted)
        g.radix = take(radix_scratch_bytes(g.nnz));  // the rows' ends lie in row_ptr
    else
        g.cnt = take(4 * g.B * g.R);
    g.sums = take(8 * g.B * g.ntile);
    g.nnzb = take(8 * g.B);
    g.misc = take(8 * (kMiscWords + g.P));
    g.queues = take(8 * (sort_queue_cap(g.nnz, 0) + sort_queue_cap(g.nnz, 1) + sort_queue_cap(g.nnz, 2)));
    g.scan = take(8 * scan_tiles(n));
    g.scratch_bytes = o;
    *L = g;
    return CSBFS_OK;
}

int graph_device_check(const csbfs_graph *g) {
    int dev = -1;
    CSBFS_HIP(hipGetDevice(&dev));
    if (dev != g->device) return fail(CSBFS_EINVAL, "graph was built on another device");
    return CSBFS_OK;
}

}  // namespace csbfs

using namespace csbfs;

extern "C" int csbfs_graph_build_into(const int64_t *src, const int64_t *dst, int64_t n_tuples, int64_t n,
                                      int32_t p, void *graph_mem, size_t graph_bytes, void *scratch,
                                      size_t scratch_bytes, void *stream, csbfs_graph **out) {
    if (!out) return fail(CSBFS_EINVAL, "csbfs_graph_build_into: out is NULL");
    *out = nullptr;
    if (n_tuples < 0 || (n_tuples > 0 && (!src || !dst)))
        return fail(CSBFS_EINVAL, "csbfs_graph_build_into: null tuple arrays or negative count");
    GraphLayout L;
    int rc = graph_layout(n, n_tuples, p, &L);
    if (rc) return rc;
    if (!graph_mem || !scratch) return fail(CSBFS_EINVAL, "csbfs_graph_build_into: null graph or scratch buffer");
    if ((uintptr_t)graph_mem % kAlign || (uintptr_t)scratch % kAlign)
        return fail(CSBFS_EINVAL, "csbfs_graph_build_into: buffers must be 256-byte aligned");
    if (L.sorted && (int64_t)scratch_bytes < L.scratch_bytes) {
        rc = graph_layout(n, n_tuples, p, &L, false);
        if (rc) return rc;
    }
    if ((int64_t)graph_bytes < L.graph_bytes || (int64_t)scratch_bytes < L.scratch_bytes)
        return fail(CSBFS_ENOSPACE, "csbfs_graph_build_into: graph or scratch buffer smaller than "
                                    "csbfs_layout_query gives");
    hipStream_t st = as_stream(stream);
    const int64_t R = L.R, W = L.W, B = L.B, ntile = L.ntile;
    char *gm = (char *)graph_mem, *sm = (char *)scratch;

    std::unique_ptr<csbfs_graph> g(new csbfs_graph());
    CSBFS_HIP(hipGetDevice(&g->device));
    g->n = n;
    g->P = p;
    g->R = R;
    g->W = W;
    g->n_tuples = n_tuples;
    g->row_ptr = (int32_t *)(gm + L.row_ptr);
    g->col_base = (int64_t *)(gm + L.col_base);
    g->col = (uint32_t *)(gm + L.col);
    g->dir = (uint64_t *)(gm + L.dir);
    g->deg = (int32_t *)(gm + L.deg);
    g->pull_off = (int64_t *)(gm + L.pull_off);
    g->pull_col = (uint32_t *)(gm + L.pull_col);
    g->head = (uint32_t *)(gm + L.head);
    g->live = (uint64_t *)(gm + L.live);
    g->qoff = (int64_t *)(gm + L.qoff);
    g->scratch = (unsigned long long *)(gm + L.small);
    // the rows' counts, or (sorted) their ends, `stride` of them per block
    int32_t *cnt = L.sorted ? g->row_ptr : (int32_t *)(sm + L.cnt);
    const int64_t stride = L.sorted ? R + 1 : R;
    long long *sums = (long long *)(sm + L.sums);
    long long *nnzb = (long long *)(sm + L.nnzb);
    unsigned long long *misc = (unsigned long long *)(sm + L.misc);
    int32_t *err = (int32_t *)misc;
    unsigned long long *qcount = misc + 8, *chk = misc + 16, *big = misc + kMiscWords;

    CSBFS_HIP(hipMemsetAsync(cnt, 0, sizeof(int32_t) * B * stride, st));
    CSBFS_HIP(hipMemsetAsync(misc, 0, sizeof(unsigned long long) * (kMiscWords + p), st));
    if (L.sorted) {
        rc = sort_entries(src, dst, n_tuples, n, p, sm + L.radix, g->col, g->col, cnt, err, st);
        if (rc) return rc;
    } else if (n_tuples > 0) {
        hipLaunchKernelGGL(k_count, dim3(grid_for(n_tuples, kThreads, 65536)), dim3(kThreads), 0, st, src,
                           dst, n_tuples, n, R, p, cnt, err);
        CSBFS_HIP(hipGetLastError());
    }
    int32_t herr = 0;
    CSBFS_HIP(hipMemcpyAsync(&herr, err, sizeof(herr), hipMemcpyDeviceToHost, st));
    hipLaunchKernelGGL(L.sorted ? k_tile_sum<true> : k_tile_sum<false>, dim3((unsigned)ntile, (unsigned)B), dim3(kThreads), 0, st,
                       (const int32_t *)cnt, stride, R, ntile, sums);
    CSBFS_HIP(hipGetLastError());
    hipLaunchKernelGGL(L.sorted ? k_tile_scan<true> : k_tile_scan<false>, dim3((unsigned)B), dim3(kThreads), 0, st, sums, ntile, nnzb);
    CSBFS_HIP(hipGetLastError());
    std::vector<long long> nnz(B);
    CSBFS_HIP(hipMemcpyAsync(nnz.data(), nnzb, sizeof(long long) * B, hipMemcpyDeviceToHost, st));
    CSBFS_HIP(hipStreamSynchronize(st));
    if (herr) return fail(CSBFS_ERANGE, "csbfs_graph_build_into: a tuple id is outside [0, n)");
    std::vector<int64_t> base(B + 1, 0);
    int64_t maxb = 0;
    for (int64_t b = 0; b < B; ++b) {
        if (L.sorted) nnz[b] = std::max<long long>(nnz[b] - base[b], 0);  // from the block's last end
        if (nnz[b] >= ((long long)1 << 31) - 1)
            return fail(CSBFS_EOVERFLOW, "csbfs_graph_build_into: a sub-block has >= 2^31 entries");
        base[b + 1] = base[b] + nnz[b];
        if (nnz[b] > maxb) maxb = nnz[b];
    }
    const int64_t total = base[B];
    if (total != L.nnz) return fail(CSBFS_ECORRUPT, "csbfs_graph_build_into: adjacency count mismatch");
    CSBFS_HIP(hipMemcpyAsync(g->col_base, base.data(), sizeof(int64_t) * (B + 1), hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(L.sorted ? k_tile_apply<true> : k_tile_apply<false>, dim3((unsigned)ntile, (unsigned)B),
                       dim3(kThreads), 0, st, cnt, stride, R, ntile, (const long long *)sums,
                       (const int64_t *)g->col_base, g->row_ptr);
    CSBFS_HIP(hipGetLastError());
    if (n_tuples > 0 && !L.sorted) {
        hipLaunchKernelGGL(k_scatter, dim3(grid_for(n_tuples, kThreads, 65536)), dim3(kThreads), 0, st,
                           src, dst, n_tuples, R, p, cnt, (const int64_t *)g->col_base, g->col);
        CSBFS_HIP(hipGetLastError());
    }
    // rows in decreasing id order, if they are not yet (pull_col serves as the
    // row sort's temp buffer; it is filled from the sorted blocks afterwards)
    rc = sort_rows_desc(g->col, g->pull_col, g->row_ptr, g->col_base, R, p, total, (int64_t *)(sm + L.queues), qcount,
                        err, L.sorted, st);
    if (rc) return rc;
    hipLaunchKernelGGL(k_directory, dim3(grid_for(B * W * 64, kThreads, 65536)), dim3(kThreads), 0, st,
                       (const int32_t *)g->row_ptr, R, W, B, g->dir);
    CSBFS_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_degree, dim3(grid_for(n, kThreads, 4096)), dim3(kThreads), 0, st,
                       (const int32_t *)g->row_ptr, R, p, n, g->deg, big);
    CSBFS_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_live, dim3(grid_for(n, 256, 1 << 30)), dim3(256), 0, st, (const int32_t *)g->deg, n,
                       g->live);
    CSBFS_HIP(hipGetLastError());
    // never hand the search a column id outside its block or a lost entry
    hipLaunchKernelGGL(k_check, dim3(2048), dim3(kThreads), 0, st, (const uint32_t *)g->col, total,
                       (const int32_t *)g->deg, n, chk);
    CSBFS_HIP(hipGetLastError());
    rc = degree_offsets(g->deg, n, g->pull_off, (int64_t *)(sm + L.scan), st);
    if (rc) return rc;
    hipLaunchKernelGGL(k_pull_fill, dim3(grid_for(n, kThreads, 65536)), dim3(kThreads), 0, st,
                       (const int32_t *)g->row_ptr, (const int64_t *)g->col_base, (const uint32_t *)g->col, R, p,
                       n, (const int64_t *)g->pull_off, g->pull_col, g->head);
    CSBFS_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_pull_long, dim3(2048), dim3(kThreads), 0, st, (const int32_t *)g->row_ptr,
                       (const int64_t *)g->col_base, (const uint32_t *)g->col, R, p, (const int64_t *)g->pull_off,
                       g->pull_col, g->head, sort_long_rows((const int64_t *)(sm + L.queues), qcount, total));
    CSBFS_HIP(hipGetLastError());
    std::vector<unsigned long long> tail(kMiscWords + p);
    int64_t pull_total = -1;
    CSBFS_HIP(hipMemcpyAsync(tail.data(), misc, sizeof(unsigned long long) * (kMiscWords + p),
                             hipMemcpyDeviceToHost, st));
    CSBFS_HIP(hipMemcpyAsync(&pull_total, g->pull_off + n, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    CSBFS_HIP(hipStreamSynchronize(st));
    if ((int32_t)tail[0] != 0)
        return fail(CSBFS_ECORRUPT, "csbfs_graph_build_into: internal row-sort queue overflow");
    if (total > 0 && (tail[16] >= (unsigned long long)R || tail[17] != (unsigned long long)total))
        return fail(CSBFS_ECORRUPT, "csbfs_graph_build_into: internal consistency check of the block "
                                    "CSR failed (column id or degree total)");
    if (pull_total != total)
        return fail(CSBFS_ECORRUPT, "csbfs_graph_build_into: pull-row offsets disagree with the blocks");
    // chunk-queue regions per processor, from the long rows each block-row has
    std::vector<int64_t> qoff(p + 1, 0);
    g->big_items.assign(p, 0);
    for (int32_t r = 0; r < p; ++r) {
        g->big_items[r] = (int64_t)tail[kMiscWords + r];
        qoff[r + 1] = qoff[r] + g->big_items[r];
    }
    if (qoff[p] > big_items_bound(total))
        return fail(CSBFS_ECORRUPT, "csbfs_graph_build_into: chunk-queue items above their bound");
    CSBFS_HIP(hipMemcpyAsync(g->qoff, qoff.data(), sizeof(int64_t) * (p + 1), hipMemcpyHostToDevice, st));
    CSBFS_HIP(hipStreamSynchronize(st));
    g->col_base_host = base;
    g->nnz = total;
    g->max_block_nnz = maxb;
    g->device_bytes = L.graph_bytes;
    *out = g.release();
    return CSBFS_OK;
}

extern "C" int csbfs_graph_build(const int64_t *src, const int64_t *dst, int64_t n_tuples,
                                 int64_t n, int32_t p, void *stream, csbfs_graph **out) {
    if (!out) return fail(CSBFS_EINVAL, "csbfs_graph_build: out is NULL");
    *out = nullptr;
    if (n_tuples < 0 || (n_tuples > 0 && (!src || !dst)))
        return fail(CSBFS_EINVAL, "csbfs_graph_build: null tuple arrays or negative count");
    GraphLayout L;
    int rc = graph_layout(n, n_tuples, p, &L);
    if (rc) return rc;
    DeviceBlock gm, sm;
    rc = device_take((size_t)L.graph_bytes, &gm);
    if (rc) return rc;
    rc = device_take((size_t)L.scratch_bytes, &sm);
    if (rc && L.sorted && graph_layout(n, n_tuples, p, &L, false) == CSBFS_OK)
        rc = device_take((size_t)L.scratch_bytes, &sm);  // no room to sort: count
    if (rc) {
        device_give(gm);
        return rc;
    }
    rc = csbfs_graph_build_into(src, dst, n_tuples, n, p, gm.p, gm.bytes, sm.p, sm.bytes, stream, out);
    // a failed build may have left work behind that still uses the blocks
    if (rc) (void)hipStreamSynchronize(as_stream(stream));
    device_give(sm);
    if (rc) {
        device_give(gm);
        return rc;
    }
    (*out)->owned = gm;
    (*out)->device_bytes = (int64_t)gm.bytes;  // a kept block may be a quarter larger than asked
    return CSBFS_OK;
}

extern "C" int csbfs_graph_free(csbfs_graph *g) {
    if (!g) return CSBFS_OK;
    // a caller-owned buffer stays the caller's; the library's own is let go
    // once the device work that may still use it is done
    if (g->owned.p) device_release(g->device, g->owned);
    delete g;
    return CSBFS_OK;
}

extern "C" int csbfs_graph_get_info(const csbfs_graph *g, csbfs_graph_info *info) {
    if (!g || !info) return fail(CSBFS_EINVAL, "csbfs_graph_get_info: null argument");
    info->n = g->n;
    info->p = g->P;
    info->reserved = 0;
    info->range = g->R;
    info->n_tuples = g->n_tuples;
    info->nnz = g->nnz;
    info->max_block_nnz = g->max_block_nnz;
    info->device_bytes = g->device_bytes;
    return CSBFS_OK;
}

extern "C" int csbfs_graph_copy_directory(const csbfs_graph *g, uint64_t *dst, int64_t cap_words,
                                          void *stream) {
    if (!g || !dst) return fail(CSBFS_EINVAL, "csbfs_graph_copy_directory: null argument");
    const int64_t words = (int64_t)g->P * g->P * g->W;
    if (cap_words < words) return fail(CSBFS_ENOSPACE, "csbfs_graph_copy_directory: dst too small");
    CSBFS_HIP(hipMemcpyAsync(dst, g->dir, sizeof(uint64_t) * words, hipMemcpyDeviceToDevice,
                             as_stream(stream)));
    return CSBFS_OK;
}

extern "C" int csbfs_graph_copy_block(const csbfs_graph *g, int32_t i, int32_t j, int32_t *row_ptr,
                                      uint32_t *col, int64_t cap, int64_t *nnz_out, void *stream) {
    if (!g || !row_ptr || !nnz_out || cap < 0)
        return fail(CSBFS_EINVAL, "csbfs_graph_copy_block: null argument");
    if (i < 0 || i >= g->P || j < 0 || j >= g->P)
        return fail(CSBFS_ERANGE, "csbfs_graph_copy_block: block index outside [0, p)");
    const int64_t b = (int64_t)i * g->P + j;
    const int64_t nnz = g->col_base_host[b + 1] - g->col_base_host[b];
    *nnz_out = nnz;
    if (cap < nnz) return fail(CSBFS_ENOSPACE, "csbfs_graph_copy_block: col capacity too small");
    if (nnz > 0 && !col) return fail(CSBFS_EINVAL, "csbfs_graph_copy_block: col is NULL");
    hipStream_t st = as_stream(stream);
    CSBFS_HIP(hipMemcpyAsync(row_ptr, g->row_ptr + b * (g->R + 1), sizeof(int32_t) * (g->R + 1),
                             hipMemcpyDeviceToDevice, st));
    if (nnz > 0)
        CSBFS_HIP(hipMemcpyAsync(col, g->col + g->col_base_host[b], sizeof(uint32_t) * nnz,
                                 hipMemcpyDeviceToDevice, st));
    CSBFS_HIP(hipStreamSynchronize(st));
    return CSBFS_OK;
}

extern "C" int csbfs_count_traversed_tuples(const csbfs_graph *g, const int32_t *level,
                                            int64_t *m_out, void *stream) {
    if (!g || !level || !m_out) return fail(CSBFS_EINVAL, "csbfs_count_traversed_tuples: null argument");
    hipStream_t st = as_stream(stream);
    CSBFS_HIP(hipMemsetAsync(g->scratch, 0, sizeof(unsigned long long), st));
    hipLaunchKernelGGL(k_count_m, dim3(grid_for(g->n, kThreads, 4096)), dim3(kThreads), 0, st,
                       level, (const int32_t *)g->deg, g->n, g->scratch);
    CSBFS_HIP(hipGetLastError());
    unsigned long long s = 0;
    CSBFS_HIP(hipMemcpyAsync(&s, g->scratch, sizeof(s), hipMemcpyDeviceToHost, st));
    CSBFS_HIP(hipStreamSynchronize(st));
    // every tuple contributes two adjacency entries (a self-loop two in one row)
    *m_out = (int64_t)(s / 2);
    return CSBFS_OK;
}
