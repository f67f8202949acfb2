// Batched searches: Algorithm 3 (Sec. V.B) for up to 64 roots at once.
//
// Vertex v carries a visit mask vis[v] (bit r: reached by root r) and, during
// a level, a mask nx[v] of the roots that discovered it; the two are stored
// side by side (vn[2v], vn[2v+1]) so that one 16-byte access serves the
// push's check of both. Each root keeps its
// own frontier bitmap: plane r of `f` holds f_r, and plane r of the views
// holds the pieces P_i received for root r. One level:
//
//   expand   top-down: every view word position (i, j, q) is read in all
//            planes at once (lane = root) and transposed with ballots into
//            the masks of its 64 sources (lane = source); a source's mask
//            travels along its row of block (i, j) once, for all its roots:
//            nx[v] |= m & ~vis[v]. Long rows go to per-processor chunk queues.
//            bottom-up: every vertex v still missing some roots whose
//            frontier is not empty reads its merged row and ORs its
//            neighbours' frontier masks fm[u] (bit r: u is in root r's
//            frontier) until every missing root is found or the row ends;
//            nx[v] = the roots found (one writer per vertex, no atomics). A
//            neighbour u of v in R_i has V_{i,j}[u] = 1 (Eq. dir-vec), so
//            u's bit in P_i's view equals its frontier bit (Lemma 1): the
//            masks stand for the views, which this level then clears.
//            Chosen per level on the device by Beamer's rule over the union
//            of the roots' frontiers, as in the single-root search.
//   update   new = nx & ~vis; vis |= new; fm[v] = new; level[r][v] = k + 1
//            for each new bit r; the new masks are transposed back into the
//            planes of f^{k+1}; per-root frontier sizes and the direction
//            rule's sums (union frontier, its adjacency entries, entries of
//            vertices still missing a root) are reduced.
//   messages plane r of f^{k+1} is sieved, WAH-64 compressed, exchanged and
//            decoded exactly as in the single-root search (wah.hip, one
//            launch for all planes), so every root's streams equal those of
//            its own search.
//
// Levels only: the (select, max) parents would need one 32-bit slot per
// (vertex, root) and a max-reduction per root and edge.
#include <memory>
#include <vector>

#include "wah_device.hpp"
#include "graph.hpp"

namespace csbfs {
namespace {

constexpr int kBThreads = 256;
constexpr int kBUnroll = 4;
constexpr int kBEvPerLevel = 5;
constexpr int kMaxRoots = 64;

struct BItem {
    uint64_t mask;  // roots whose frontier holds the source
    int32_t block;
    int32_t u_local;
    int32_t start;  // offsets within the block's col
    int32_t end;
};

// A long merged row left over by the bottom-up lanes: vertex v still misses
// some of `miss` after the row's entries before e gave `got`.
struct BPullItem {
    uint64_t miss, got;
    int64_t v, e, re;
};

struct BArgs {
    uint64_t *view;  // [B][P * P * W] planes of views
    int64_t vplane;  // words per view plane
    int32_t B;
    const int32_t *row_ptr;
    const int64_t *col_base;
    const uint32_t *col;
    uint64_t *vn;         // [n][2]: visit mask, discovery mask
    BItem *queue;
    const int64_t *qoff;     // [P + 1]
    uint32_t *queue_count;   // [P]
    int64_t R;
    int64_t W;
    int32_t P;
    unsigned long long *edges;
    int32_t *status;
    // nullable: |f^j| summed over the roots; 0 leaves nothing to expand
    const unsigned long long *fcount;
    const int32_t *dir;  // direction of this level (CSBFS_DIR_*); the push runs if top-down
};

// Push kBUnroll (target v, root mask m) pairs; loads first, then atomics.
// Every load is issued unconditionally: the callers clamp the positions of
// lanes past a row's end to its last entry (an in-bounds address), and ok
// masks those lanes' results out.
__device__ __forceinline__ void brelax(const BArgs &a, const int64_t (&v)[kBUnroll],
                                       const uint64_t (&m)[kBUnroll], const bool (&ok)[kBUnroll]) {
    // one 16-byte load per target: its visit mask and a (possibly stale)
    // view of its discovery mask, which only saves redundant atomics
    ulonglong2 w[kBUnroll];
#pragma unroll
    for (int k = 0; k < kBUnroll; ++k) w[k] = *reinterpret_cast<const ulonglong2 *>(a.vn + 2 * v[k]);
#pragma unroll
    for (int k = 0; k < kBUnroll; ++k) {
        const uint64_t add = ok[k] ? m[k] & ~w[k].x : 0ull;
        if (add & ~w[k].y) atomicOr((unsigned long long *)(a.vn + 2 * v[k] + 1), (unsigned long long)add);
    }
}

// A wave's tile: kBTile consecutive words of every root plane. Loads and
// stores of a tile move 4 roots x kBTile words (four 128-byte lines) per
// instruction; LDS turns them around so that lane r holds root r's word.
constexpr int kBTile = 16;
constexpr int kBRootsPerOp = 64 / kBTile;

__global__ __launch_bounds__(kBThreads) void bexpand_kernel(BArgs a) {
    __shared__ uint64_t tile[kBThreads / 64][kBTile][kMaxRoots];
    if (a.fcount && *a.fcount == 0) return;
    if (*a.dir != CSBFS_DIR_TOP_DOWN) return;
    const int lane = threadIdx.x & 63;
    uint64_t(*tw)[kMaxRoots] = tile[threadIdx.x >> 6];
    const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const int64_t npos = (int64_t)a.P * a.P * a.W;
    const int64_t ntiles = (npos + kBTile - 1) / kBTile;
    const int t_ld = lane % kBTile, r_ld = lane / kBTile;
    const int nsteps = (a.B + kBRootsPerOp - 1) / kBRootsPerOp;
    unsigned long long edges = 0;
    for (int64_t tl = wave; tl < ntiles; tl += nwaves) {
        const int64_t pos0 = tl * kBTile;
        uint64_t anyw = 0;
        for (int s = 0; s < nsteps; ++s) {
            const int r = r_ld + kBRootsPerOp * s;
            const int64_t p = pos0 + t_ld;
            uint64_t w = 0;
            if (r < a.B && p < npos) {
                uint64_t *src = a.view + r * a.vplane + p;
                w = *src;
                if (w) *src = 0;  // the views are empty again when the level ends
            }
            tw[t_ld][r] = w;
            anyw |= w;
        }
        wave_lds_sync();
        if (__ballot(anyw != 0)) {
            for (int t = 0; t < kBTile; ++t) {
                // lane r: root r's view word at this position
                const uint64_t w = lane < a.B ? tw[t][lane] : 0ull;
                if (!__ballot(w != 0)) continue;
                const int64_t pos = pos0 + t;
                // transpose: lane b gets the roots in whose frontier source b is
                const uint64_t any = wave_or64(w);
                uint64_t mymask = 0;
                for (uint64_t it = any; it; it &= it - 1) {
                    const int b = __ffsll((unsigned long long)it) - 1;
                    const uint64_t m = __ballot((w >> b) & 1);
                    if (lane == b) mymask = m;
                }
                const int64_t blk = pos / a.W;
                const int64_t q = pos - blk * a.W;
                const int32_t i = (int32_t)(blk / a.P);
                const int64_t ul = (q << 6) + lane;
                int32_t rs = 0, deg = 0;
                if (mymask) {
                    const int32_t *rp = a.row_ptr + blk * (a.R + 1) + ul;
                    rs = rp[0];
                    deg = rp[1] - rs;
                }
                const int32_t items = row_items(deg);
                const int32_t items_incl = wave_incl_scan_i32(items);
                const int32_t items_total = __shfl(items_incl, 63, 64);
                if (items_total) {
                    uint32_t qbase = 0;
                    if (lane == 63) qbase = atomicAdd(&a.queue_count[i], (uint32_t)items_total);
                    qbase = __shfl(qbase, 63, 64);
                    if (items) {
                        const int64_t qpos = (int64_t)qbase + items_incl - items;
                        const int64_t qcap = a.qoff[i + 1] - a.qoff[i];
                        if (qpos + items > qcap) {
                            *a.status = 2;  // a row is queued at most once per level: unreachable
                        } else {
                            for (int32_t c = 0; c < items; ++c) {
                                BItem it;
                                it.mask = mymask;
                                it.block = (int32_t)blk;
                                it.u_local = (int32_t)ul;
                                it.start = rs + c * kBigChunk;
                                it.end = it.start + min(deg - c * kBigChunk, kBigChunk);
                                a.queue[a.qoff[i] + qpos + c] = it;
                            }
                        }
                        deg = 0;
                    }
                }
                const int32_t incl = wave_incl_scan_i32(deg);
                const int32_t total = __shfl(incl, 63, 64);
                const int32_t excl = incl - deg;
                edges += (unsigned long long)total;
                const uint32_t *colb = a.col + a.col_base[blk];
                const int64_t vbase = (int64_t)i * a.R;
                for (int32_t e0 = 0; e0 < total; e0 += 64 * kBUnroll) {
                    int64_t v[kBUnroll];
                    uint64_t m[kBUnroll];
                    bool ok[kBUnroll];
#pragma unroll
                    for (int k = 0; k < kBUnroll; ++k) {
                        const int32_t e = e0 + 64 * k + lane;
                        ok[k] = e < total;
                        const int o = owner_lane(excl, ok[k] ? e : total - 1);
                        const int32_t ex = __shfl(excl, o, 64);
                        const int32_t r0 = __shfl(rs, o, 64);
                        m[k] = (uint64_t)shfl64((int64_t)mymask, o);
                        const int32_t ec = ok[k] ? e : total - 1;  // clamped: an entry of the last row
                        v[k] = vbase + colb[r0 + (ec - ex)];
                    }
                    brelax(a, v, m, ok);
                }
            }
        }
        wave_lds_sync();
    }
    block_add<kBThreads / 64>(edges, a.edges);
}

// Top-down long rows: the chunk-queue items of every processor.
__device__ __forceinline__ void push_long(const BArgs &a) {
    const int lane = threadIdx.x & 63;
    const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    unsigned long long edges = 0;
    int64_t before = 0;  // items of the processors before r, for a grid-wide stride
    for (int32_t r = 0; r < a.P; ++r) {
        const int64_t cap = a.qoff[r + 1] - a.qoff[r];
        const int64_t queued = a.queue_count[r];
        const int64_t count = queued < cap ? queued : cap;
        const BItem *queue = a.queue + a.qoff[r];
        const int64_t vbase = (int64_t)r * a.R;
        int64_t first = (wave - before) % nwaves;
        if (first < 0) first += nwaves;
        before += count;
        for (int64_t kk = first; kk < count; kk += nwaves) {
            const BItem it = queue[kk];
            const uint32_t *colb = a.col + a.col_base[it.block] + it.start;
            const int32_t len = it.end - it.start;  // places from the item's first: its end may lie near 2^31
            for (int32_t e0 = 0; e0 < len; e0 += 64 * kBUnroll) {
                int64_t v[kBUnroll];
                uint64_t m[kBUnroll];
                bool ok[kBUnroll];
#pragma unroll
                for (int k = 0; k < kBUnroll; ++k) {
                    const int32_t e = e0 + 64 * k + lane;
                    ok[k] = e < len;
                    v[k] = vbase + colb[ok[k] ? e : len - 1];  // clamped to the item's last entry
                    m[k] = it.mask;
                }
                brelax(a, v, m, ok);
            }
            edges += (unsigned long long)len;
        }
    }
    block_add<kBThreads / 64>(edges, a.edges);
}

// ---------------------------------------------------------------- pull ---

constexpr int kBPullUnroll = 2;   // entries per lane step
constexpr int kBPullWindow = 4;   // row entries a lane loads at once
constexpr int kBPullSlots = 4;    // rows the wave reads side by side
constexpr int kBPullLong = 2048;  // entries left from which a row goes to a whole workgroup
constexpr int kBLongUnroll = 8;   // 64-entry steps per wave in one pass of that workgroup
// Direction rule of batched searches (Beamer's alpha and beta over the union
// of the roots' frontiers)
constexpr float kBatchAlpha = 16.0f, kBatchBeta = 24.0f;
constexpr int kBPullRounds = 16;  // lane steps before the wave takes over slow lanes

// Direction state of a batched search, carried from level to level.
struct BDirState {
    int32_t cur;              // direction of the level expanded next
    int32_t force;            // < 0: chosen by the rule; else this direction every level
    unsigned long long prev;  // union frontier size of the level before
    unsigned long long sums[3];  // union frontier, its adjacency entries, entries still missing a root
};

// A bottom-up level whose union frontier is below n / kBSparse looks a
// neighbour up in the frontier's bitmap before it reads its mask: the bitmap
// stays in L2 where the masks (64 times its size) do not. From kBBitmapVerts
// vertices on (8 MiB of masks, twice an XCD's L2; at 2^18 vertices the extra
// step cost 2%). Scale 24, 64 roots whose first level of 9153 vertices goes
// bottom-up: the batch 36.8 -> 31.7 ms.
constexpr unsigned long long kBSparse = 16;
constexpr int64_t kBBitmapVerts = int64_t(1) << 20;

struct BPullArgs {
    uint64_t *vn;              // [n][2]: visit mask, discovery mask
    const uint64_t *fm;        // [n]: frontier masks of the level
    const uint64_t *ubits;     // [n / 64]: vertices on any root's frontier (null: not known)
    const BDirState *st;
    const int64_t *pull_off;   // merged rows (global ids) of every vertex
    const uint32_t *pull_col;
    const uint32_t *head;      // [2n]: the first two ids of each merged row
    uint64_t *view;            // every view plane, zeroed here (the decode ORs into zeroed views)
    int64_t view_words;
    int64_t n;
    const unsigned long long *rootc;  // [B]: frontier size of each root at this level
    int32_t B;
    const int32_t *dir;
    unsigned long long *edges;
    const unsigned long long *fcount;
    BPullItem *queue;          // long rows, read by whole workgroups afterwards
    int64_t queue_cap;
    uint32_t *queue_count;
    int32_t *status;
};

__device__ __forceinline__ bool sparse_level(const BPullArgs &a) {
    return a.ubits && a.st->prev * kBSparse < (unsigned long long)a.n;
}
// Frontier masks of kN neighbours.
template <int kN>
__device__ __forceinline__ void gather_masks(const BPullArgs &a, bool sparse, const uint32_t (&c)[kN],
                                             uint64_t (&m)[kN]) {
    if (sparse) {
        uint64_t w[kN];
#pragma unroll
        for (int k = 0; k < kN; ++k) w[k] = a.ubits[c[k] >> 6];
#pragma unroll
        for (int k = 0; k < kN; ++k) m[k] = (w[k] >> (c[k] & 63)) & 1 ? a.fm[c[k]] : 0ull;
    } else {
#pragma unroll
        for (int k = 0; k < kN; ++k) m[k] = a.fm[c[k]];
    }
}

// Bottom-up level. A wave takes 64 vertices (lane = vertex): the two ids of
// head, then kBPullRounds steps of kBPullUnroll entries per lane. The rows
// still being read are then taken by the whole wave, 64 entries a step,
// kBPullSlots rows side by side, and rows with kBPullLong entries or more
// left go to a queue that whole workgroups work off (pull_long).
//
// Bound by chains of dependent loads (row entry, then the neighbour's mask).
// One row at a time per wave made the longest row the level's time: scale 18,
// 8 roots 479 us, now 71 + 53 us (pull_long); scale 24, 64 roots 16.4 ms for
// a level that reads all 2^29 entries, now 4.9 + 4.0 ms (60 G masks/s).
__global__ __launch_bounds__(kBThreads) void bpull_kernel(BPullArgs a) {
    if (a.fcount && *a.fcount == 0) return;
    if (*a.dir != CSBFS_DIR_BOTTOM_UP) return;
    const int lane = threadIdx.x & 63;
    const int64_t tid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t nthreads = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k = tid; k < a.view_words; k += nthreads) a.view[k] = 0;
    // roots whose frontier is not empty: only they can find anything
    const uint64_t active = __ballot(lane < a.B && (!a.rootc || a.rootc[lane] > 0));
    const int64_t wave = tid >> 6, nwaves = nthreads >> 6;
    const bool sparse = sparse_level(a);
    unsigned long long read = 0;
    for (int64_t v0 = wave * 64; v0 < a.n; v0 += nwaves * 64) {
        const int64_t v = v0 + lane;
        uint64_t missing = 0, found = 0;
        int64_t e = 0, re = 0;
        uint2 hd = make_uint2(0u, 0u);
        if (v < a.n) {
            missing = active & ~a.vn[2 * v];
            if (missing) {
                e = a.pull_off[v];
                re = a.pull_off[v + 1];
                hd = *reinterpret_cast<const uint2 *>(a.head + 2 * v);
            }
        }
        bool busy = missing && e < re;
        // the row's first two ids come from head, without the row itself
        if (busy) {
            const int32_t nk = re - e < 2 ? (int32_t)(re - e) : 2;
            const uint32_t c[2] = {hd.x, nk > 1 ? hd.y : hd.x};
            uint64_t m[2];
            gather_masks<2>(a, sparse, c, m);
            found |= (m[0] | m[1]) & missing;
            read += (unsigned long long)nk;
            e += nk;
            if (found == missing || e >= re) busy = false;
        }
        // kBPullWindow entries are loaded at once (positions past the row end
        // clamped to its last entry and masked out) and counted kBPullUnroll at
        // a time
        for (int round = 0; round < kBPullRounds * kBPullUnroll / kBPullWindow; ++round) {
            if (busy) {
                const int32_t nw = re - e < kBPullWindow ? (int32_t)(re - e) : kBPullWindow;
                uint32_t c[kBPullWindow];
                uint64_t m[kBPullWindow];
#pragma unroll
                for (int q = 0; q < kBPullWindow; ++q) c[q] = a.pull_col[e + (q < nw ? q : nw - 1)];
                gather_masks<kBPullWindow>(a, sparse, c, m);
#pragma unroll
                for (int h = 0; h < kBPullWindow / kBPullUnroll; ++h) {
                    const int32_t nk = re - e < kBPullUnroll ? (int32_t)(re - e) : kBPullUnroll;
                    if (busy) {
#pragma unroll
                        for (int q = 0; q < kBPullUnroll; ++q)
                            if (q < nk) found |= m[h * kBPullUnroll + q] & missing;
                        read += (unsigned long long)nk;
                        e += nk;
                        if (found == missing || e >= re) busy = false;
                    }
                }
            }
            if (!__ballot(busy)) break;
        }
        uint64_t slow = __ballot(busy);
        const bool far = busy && re - e >= kBPullLong;
        const uint64_t deferred = __ballot(far);
        if (deferred) {
            slow &= ~deferred;
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(a.queue_count, (uint32_t)__popcll(deferred));
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
            if (far) {
                const int64_t pos = (int64_t)at + __popcll(deferred & ((1ull << lane) - 1));
                if (pos >= a.queue_cap) {
                    *a.status = 2;  // cannot happen: the capacity counts every such row
                } else {
                    a.queue[pos] = BPullItem{missing, found, v, e, re};
                }
                found = 0;  // pull_long writes this vertex
            }
        }
        // the wave's slots, all wave-uniform: row [se, sr) of lane sl
        int64_t se[kBPullSlots], sr[kBPullSlots];
        uint64_t smiss[kBPullSlots], sgot[kBPullSlots];
        int sl[kBPullSlots];
#pragma unroll
        for (int k = 0; k < kBPullSlots; ++k) {
            se[k] = sr[k] = 0;
            smiss[k] = sgot[k] = 0;
            sl[k] = -1;
        }
        for (;;) {
            int live = 0;
#pragma unroll
            for (int k = 0; k < kBPullSlots; ++k) {
                if (sl[k] < 0 && slow) {
                    sl[k] = __ffsll((unsigned long long)slow) - 1;
                    slow &= slow - 1;
                    se[k] = (int64_t)readlane64((uint64_t)e, sl[k]);
                    sr[k] = (int64_t)readlane64((uint64_t)re, sl[k]);
                    smiss[k] = readlane64(missing, sl[k]);
                    sgot[k] = readlane64(found, sl[k]);
                }
                live |= sl[k] >= 0;
            }
            if (!live) break;
            // an empty slot reads entry 0 (there are entries) and ignores it
            uint32_t c[kBPullSlots];
            uint64_t f[kBPullSlots];
#pragma unroll
            for (int k = 0; k < kBPullSlots; ++k) {
                const int64_t pos = se[k] + lane;
                c[k] = a.pull_col[sl[k] < 0 ? 0 : pos < sr[k] ? pos : sr[k] - 1];
            }
            gather_masks<kBPullSlots>(a, sparse, c, f);
#pragma unroll
            for (int k = 0; k < kBPullSlots; ++k) f[k] &= smiss[k];  // a repeated last entry adds nothing
#pragma unroll
            for (int k = 0; k < kBPullSlots; ++k) {
                if (sl[k] < 0) continue;
                if (__ballot((f[k] & ~sgot[k]) != 0)) sgot[k] |= wave_or64(f[k]);
                if (lane == 0) read += (unsigned long long)(sr[k] - se[k] < 64 ? sr[k] - se[k] : 64);
                se[k] += 64;
                if (sgot[k] == smiss[k] || se[k] >= sr[k]) {
                    if (lane == sl[k]) found = sgot[k];
                    sl[k] = -1;
                }
            }
        }
        if (found) a.vn[2 * v + 1] = found;  // this lane's vertex: no other writer
    }
    for (int d = 32; d > 0; d >>= 1) read += (unsigned long long)shfl64((int64_t)read, lane ^ d);
    block_add<kBThreads / 64>(read, a.edges);
}

// Bottom-up long rows: a workgroup takes one row, kBLongUnroll * 64 entries
// per wave and pass, until every missing root is found or the row ends. The
// entries read are counted to the 64-entry step that completes the mask.
__device__ __forceinline__ void pull_long(const BPullArgs &a) {
    constexpr int kWaves = kBThreads / 64;
    constexpr int kStep = 64 * kBLongUnroll, kPass = kWaves * kStep;
    __shared__ uint64_t part[2][kWaves];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int64_t count = (int64_t)*a.queue_count < a.queue_cap ? (int64_t)*a.queue_count : a.queue_cap;
    const bool sparse = sparse_level(a);
    unsigned long long read = 0;
    int par = 0;
    for (int64_t it = blockIdx.x; it < count; it += gridDim.x) {
        const BPullItem x = a.queue[it];
        uint64_t got = x.got;
        for (int64_t e = x.e; e < x.re && got != x.miss; e += kPass) {
            const int64_t e0 = e + (int64_t)wid * kStep;
            uint32_t c[kBLongUnroll];
            uint64_t f[kBLongUnroll];
#pragma unroll
            for (int k = 0; k < kBLongUnroll; ++k) {
                const int64_t pos = e0 + 64 * k + lane;
                c[k] = a.pull_col[pos < x.re ? pos : x.re - 1];
            }
            uint64_t any = 0;
            gather_masks<kBLongUnroll>(a, sparse, c, f);
#pragma unroll
            for (int k = 0; k < kBLongUnroll; ++k) {
                f[k] = e0 + 64 * k + lane < x.re ? f[k] & x.miss : 0ull;
                any |= f[k];
            }
            any = __ballot((any & ~got) != 0) ? wave_or64(any) : 0ull;
            if (lane == 0) part[par][wid] = any;
            __syncthreads();  // one barrier a pass: the parts alternate
            uint64_t before = got;
            for (int w = 0; w < wid; ++w) before |= part[par][w];
            uint64_t all = before;
            for (int w = wid; w < kWaves; ++w) all |= part[par][w];
            if (all == x.miss && before != x.miss && (before | any) == x.miss) {
                // this wave's steps complete the mask: which one
                for (int k = 0; k < kBLongUnroll && before != x.miss; ++k) {
                    before |= wave_or64(f[k]);
                    if (before == x.miss) {
                        const int64_t end = e0 + 64 * (k + 1);
                        read += (unsigned long long)((end < x.re ? end : x.re) - e);
                    }
                }
            } else if (all != x.miss && wid == 0) {
                read += (unsigned long long)(x.re - e < kPass ? x.re - e : kPass);
            }
            got = all;
            par ^= 1;
        }
        if (threadIdx.x == 0 && got) a.vn[2 * x.v + 1] = got;
    }
    block_add<kWaves>(read, a.edges);
}

// The level's long rows, in the direction it was expanded in.
__global__ __launch_bounds__(kBThreads) void blong_kernel(BArgs a, BPullArgs pa) {
    if (a.fcount && *a.fcount == 0) return;
    const int32_t d = *a.dir;
    if (d == CSBFS_DIR_TOP_DOWN)
        push_long(a);
    else if (d == CSBFS_DIR_BOTTOM_UP)
        pull_long(pa);
}

// Beamer's rule over the union of the roots' frontiers (one thread, after the
// update): top-down turns bottom-up when the frontier's entries times alpha
// exceed the entries of vertices some root has not reached and the frontier
// did not shrink; bottom-up turns top-down when the frontier is below
// n / beta and shrinking. The sums are cleared for the next update, and the
// level's frontier size is posted for the host.
struct BDirArgs {
    BDirState *st;
    int32_t *rec;  // nullable
    int64_t n;
    float alpha, beta;
    const unsigned long long *total;  // frontier size of the level
    unsigned long long *host;         // pinned word: level tag << kPostBits | size
    int64_t level;
};
constexpr int kPostBits = 40;  // sizes are at most 64 n < 2^38; the tag is the level's low 24 bits

__device__ void bdir_choose(const BDirArgs &a) {
    BDirState s = *a.st;
    const unsigned long long nf = s.sums[0], mf = s.sums[1], mu = s.sums[2];
    int32_t next = s.cur;
    if (s.force >= 0) {
        next = s.force;
    } else if (s.cur == CSBFS_DIR_TOP_DOWN) {
        if ((double)mf * a.alpha > (double)mu && nf >= s.prev) next = CSBFS_DIR_BOTTOM_UP;
    } else if ((double)nf * a.beta < (double)a.n && nf < s.prev) {
        next = CSBFS_DIR_TOP_DOWN;
    }
    s.prev = nf;
    s.cur = next;
    s.sums[0] = s.sums[1] = s.sums[2] = 0;
    *a.st = s;
    if (a.rec) *a.rec = next;
    __hip_atomic_store(a.host, ((unsigned long long)a.level << kPostBits) | *a.total, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

// Sieve + compress of a level's frontier planes; the first workgroup also
// chooses the direction of the expansion that follows (nothing else of this
// launch reads the direction state) and posts the level's size. A launch of
// one thread for that and a copy of the size cost two of eight commands per
// level.
// Eight waves per SIMD, as the large searches' encoder: four workgroups share a
// CU instead of three (64 planes at scale 24 435 -> 422 us).
__global__ __launch_bounds__(kEncThreads) __attribute__((amdgpu_waves_per_eu(8))) void bencode_kernel(WahBatch b, BDirArgs d) {
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) bdir_choose(d);
    PlainWords h;
    encode_segment<kEncGpt>(b, h, blockIdx.y, blockIdx.x == 0);
}

// Where each root's levels go.
struct BLevels {
    int32_t *p[kMaxRoots];  // [n] each
};

struct BUpdateArgs {
    uint64_t *vn;      // [n][2]
    uint64_t *f;       // [B][n / 64] planes of the new frontier
    BLevels level;
    int32_t next_level;
    int32_t B;
    int64_t n;
    unsigned long long *root_count;  // [B]
    unsigned long long *total;       // [1]
    uint32_t *queue_count;           // [P + 1], cleared for the next level
    int32_t P;
    const unsigned long long *fcount;  // as in BArgs: 0 visits nothing
    uint64_t *fm;                      // [n]: frontier mask of every vertex (written for all)
    uint64_t *ubits;                   // [n / 64]: vertices with one
    const int32_t *deg;                // [n]: adjacency entries
    unsigned long long *dsums;         // [3]: union frontier, its entries, entries still missing a root
};

__global__ __launch_bounds__(kBThreads) void bupdate_kernel(BUpdateArgs a) {
    __shared__ uint64_t tile[kBThreads / 64][kBTile][kMaxRoots];
    __shared__ unsigned long long cnt[kMaxRoots];
    __shared__ unsigned long long dsum[3];
    const int lane = threadIdx.x & 63;
    uint64_t(*tw)[kMaxRoots] = tile[threadIdx.x >> 6];
    if (a.fcount && *a.fcount == 0) return;
    if (threadIdx.x < kMaxRoots) cnt[threadIdx.x] = 0;
    if (threadIdx.x < 3) dsum[threadIdx.x] = 0;
    if (blockIdx.x == 0)
        for (int q = threadIdx.x; q <= a.P; q += blockDim.x) a.queue_count[q] = 0;
    __syncthreads();
    const int64_t words = a.n / 64;
    const int64_t ntiles = (words + kBTile - 1) / kBTile;
    const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const int t_st = lane % kBTile, r_st = lane / kBTile;
    const int nsteps = (a.B + kBRootsPerOp - 1) / kBRootsPerOp;
    unsigned long long mine = 0;  // lane r: new vertices of root r seen by this wave
    const uint64_t my_level = (uint64_t)a.level.p[lane];  // lane r: where root r's levels go
    unsigned long long u_nf = 0, u_mf = 0, u_mu = 0;  // the direction rule's sums, this lane
    for (int64_t tl = wave; tl < ntiles; tl += nwaves) {
        const int64_t q0 = tl * kBTile;
        for (int t = 0; t < kBTile; ++t) {
            const int64_t q = q0 + t;
            uint64_t plane = 0;
            if (q < words) {
                const int64_t v = (q << 6) + lane;
                ulonglong2 *pv = reinterpret_cast<ulonglong2 *>(a.vn + 2 * v);
                const ulonglong2 w = *pv;
                uint64_t nw = 0;
                if (w.y) {
                    nw = w.y & ~w.x;
                    *pv = make_ulonglong2(w.x | nw, 0ull);
                }
                a.fm[v] = nw;
                const uint64_t ub = __ballot(nw != 0);
                if (lane == 0 && a.n >= kBBitmapVerts) a.ubits[q] = ub;
                const uint64_t all = a.B == 64 ? ~0ull : ((1ull << a.B) - 1);
                if (nw || (all & ~(w.x | nw))) {
                    const unsigned long long dg = (unsigned long long)a.deg[v];
                    if (nw) {
                        u_nf += 1;
                        u_mf += dg;
                    }
                    if (all & ~(w.x | nw)) u_mu += dg;
                }
                // lane r collects root r's frontier word: bit b = vertex q*64+b is new for r
                for (uint64_t it = wave_or64(nw); it; it &= it - 1) {
                    const int r = __ffsll((unsigned long long)it) - 1;
                    const bool mine_r = (nw >> r) & 1;
                    int32_t *level = (int32_t *)readlane64(my_level, r);
                    if (mine_r) level[v] = a.next_level;
                    const uint64_t bal = __ballot(mine_r);
                    if (lane == r) plane = bal;
                }
            }
            tw[t][lane] = plane;
            mine += (unsigned long long)__popcll(plane);
        }
        wave_lds_sync();
        for (int s = 0; s < nsteps; ++s) {
            const int r = r_st + kBRootsPerOp * s;
            const int64_t q = q0 + t_st;
            if (r < a.B && q < words) a.f[r * words + q] = tw[t_st][r];
        }
        wave_lds_sync();
    }
    if (lane < a.B && mine) atomicAdd(&cnt[lane], mine);
    for (int d = 32; d > 0; d >>= 1) {
        u_nf += (unsigned long long)shfl64((int64_t)u_nf, lane ^ d);
        u_mf += (unsigned long long)shfl64((int64_t)u_mf, lane ^ d);
        u_mu += (unsigned long long)shfl64((int64_t)u_mu, lane ^ d);
    }
    if (lane == 0 && (u_nf | u_mf | u_mu)) {
        atomicAdd(&dsum[0], u_nf);
        atomicAdd(&dsum[1], u_mf);
        atomicAdd(&dsum[2], u_mu);
    }
    __syncthreads();
    if (threadIdx.x < 3 && dsum[threadIdx.x]) atomicAdd(&a.dsums[threadIdx.x], dsum[threadIdx.x]);
    if (threadIdx.x < a.B && cnt[threadIdx.x]) atomicAdd(&a.root_count[threadIdx.x], cnt[threadIdx.x]);
    if (threadIdx.x == 0) {
        unsigned long long sum = 0;
        for (int r = 0; r < a.B; ++r) sum += cnt[r];
        if (sum) atomicAdd(a.total, sum);
    }
}

struct BSeedArgs {
    uint64_t *vn;      // [n][2]
    uint64_t *fm;      // [n]
    uint64_t *view;
    int64_t view_words;  // all planes
    BLevels level;
    int64_t n;
    uint32_t *zero;       // counters, look-back words and tickets, queue counts, status
    int64_t zero_words;
};

struct BRoots {
    int64_t v[kMaxRoots];
};

// One row of workgroups per root clears its levels; all of them the rest.
__global__ void bseed_fill_kernel(BSeedArgs a) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, row = (int64_t)gridDim.x * blockDim.x;
    int32_t *level = a.level.p[blockIdx.y];
    for (int64_t k = t; k < a.n; k += row) level[k] = -1;
    const int64_t stride = row * gridDim.y;
    int64_t top = a.view_words > a.n ? a.view_words : a.n;
    top = top > a.zero_words ? top : a.zero_words;
    for (int64_t k = blockIdx.y * row + t; k < top; k += stride) {
        if (k < a.n) {
            reinterpret_cast<ulonglong2 *>(a.vn)[k] = make_ulonglong2(0ull, 0ull);
            a.fm[k] = 0;
        }
        if (k < a.zero_words) a.zero[k] = 0;
        if (k < a.view_words) a.view[k] = 0;
    }
}

// f(s) <- s for every root: known to every processor without a message.
__global__ void bseed_root_kernel(BSeedArgs a, BRoots roots, int32_t B, int64_t R, int64_t W,
                                  int32_t P, int64_t vplane, unsigned long long *root_count0,
                                  unsigned long long *total0, BDirState *ds, int32_t dir0, int32_t force,
                                  int32_t *rec0) {
    const int r = threadIdx.x;
    if (r == 0) {
        BDirState d{};
        d.cur = dir0;
        d.force = force;
        d.prev = (unsigned long long)B;
        *ds = d;
        if (rec0) *rec0 = dir0;
    }
    if (r >= B) return;
    const int64_t s = roots.v[r];
    const int64_t own = s / R, sl = s - own * R;
    atomicOr((unsigned long long *)(a.vn + 2 * s), 1ull << r);
    atomicOr((unsigned long long *)(a.fm + s), 1ull << r);
    a.level.p[r][s] = 0;
    for (int32_t i = 0; i < P; ++i)
        a.view[r * vplane + ((int64_t)i * P + own) * W + (sl >> 6)] = 1ull << (sl & 63);
    root_count0[r] = 1;
    atomicAdd(total0, 1ull);
}

}  // namespace
}  // namespace csbfs

using namespace csbfs;

struct csbfs_batch_engine {
    const csbfs_graph *g = nullptr;
    int32_t Bmax = 0, L = 0;
    uint32_t flags = 0;
    int64_t cap = 0, nseg = 0, nchunk = 0, Smax = 0;
    uint64_t *vn = nullptr, *f = nullptr, *view = nullptr, *arena = nullptr;
    uint64_t *fm = nullptr;           // [n] frontier mask of every vertex (bottom-up levels)
    uint64_t *ubits = nullptr;        // [n / 64] vertices on any frontier
    BDirState *dstate = nullptr;
    unsigned long long *look = nullptr;  // encoder look-back words [Smax * nseg]
    uint32_t *enc_ticket = nullptr;      // [kTicketStride * Smax], after look
    int64_t *chunk_groups = nullptr;
    BItem *queue = nullptr;
    int64_t *qoff = nullptr;
    uint32_t *qcount = nullptr;       // [P] top-down chunk queues, then the bottom-up long rows
    BPullItem *pqueue = nullptr;
    int64_t pqueue_cap = 0;
    int32_t *status = nullptr;
    // one block that a batch starts from zero: status and queue counts, a
    // record of `stride` words per level (slot L for levels past max_levels),
    // the look-back words and tickets. A search's status and statistics are
    // one copy from its start.
    uint32_t *zero_mem = nullptr;
    int64_t zero_words = 0, hdr = 0, stride = 0;
    unsigned long long *recs = nullptr;
    unsigned long long *ctl(int64_t k) const { return recs + k * stride; }  // total frontier
    unsigned long long *edges(int64_t k) const { return ctl(k) + 1; }
    int32_t *dir(int64_t k) const { return (int32_t *)(ctl(k) + 2); }  // direction used to expand the level
    unsigned long long *rootc(int64_t k) const { return ctl(k) + 3; }                 // [Bmax]
    unsigned long long *uwords(int64_t k) const { return rootc(k) + Bmax; }           // [Bmax * P]
    unsigned long long *sbits(int64_t k) const { return uwords(k) + Bmax * g->P; }    // [Smax]
    int64_t *words(int64_t k) const { return (int64_t *)(sbits(k) + Smax); }          // [Smax]
    unsigned long long *host_ctl = nullptr;      // pinned [2]
    unsigned long long *host_ctl_dev = nullptr;  // its device address
    std::vector<hipEvent_t> events;
    void *mem = nullptr;     // every device buffer, carved from one block
    bool owns_mem = false;   // hipMalloc'd here (else the caller's, e.g. the server's pool)
    bool owns_host = false;  // host_ctl hipHostMalloc'd here
    int32_t last_levels = 0, last_roots = 0;
};

namespace {

// Releases what the engine itself allocated (hipFree orders itself after
// work still using the block; a caller-provided block stays the caller's).
void bengine_release(csbfs_batch_engine *e) {
    if (e->owns_mem && e->mem) (void)hipFree(e->mem);
    if (e->owns_host && e->host_ctl) (void)hipHostFree(e->host_ctl);
    for (hipEvent_t ev : e->events)
        if (ev) (void)hipEventDestroy(ev);
    delete e;
}

}  // namespace

namespace {

// Device bytes of every buffer of a batch engine; total() is the size of
// the one block they are carved from (each buffer 256-byte aligned).
struct BatchSizes {
    int64_t vis, f, view, arena, chunk, queue, qoff, zero, fm, ubits, dstate, pqueue;
    int64_t hdr, stride;  // words before the first record, words per record
    int64_t total() const {
        int64_t t = 0;
        for (int64_t b : {vis, f, view, arena, chunk, queue, qoff, zero, fm, ubits, dstate, pqueue})
            t += align_up(b > 0 ? b : 1);
        return t;
    }
};

// Rows with kBPullLong entries or more: each is queued at most once a level.
int64_t pull_long_rows(int64_t nnz) { return nnz / kBPullLong + 1; }

BatchSizes batch_sizes(const csbfs_graph *g, int64_t B, int64_t L, uint32_t flags) {
    const int64_t P = g->P, n = g->n;
    const int64_t Smax = B * P * P, slots = L + 1;
    const int64_t arena_slots = (flags & CSBFS_FLAG_KEEP_STREAMS) ? slots : 1;
    int64_t items = 0;
    for (int64_t r = 0; r < P; ++r) items += g->big_items[r];
    BatchSizes z{};
    z.vis = 16 * n;
    z.f = 8 * B * (n / 64);
    z.view = 8 * B * P * (n / 64);
    z.arena = 8 * Smax * wah_cap(g->R) * arena_slots;
    z.chunk = 8 * Smax * dec_chunks(g->R);
    z.queue = (int64_t)sizeof(BItem) * (items > 0 ? items : 1);
    z.qoff = 8 * (P + 1);
    z.pqueue = (int64_t)sizeof(BPullItem) * pull_long_rows(g->nnz);
    z.hdr = 1 + (P + 2) / 2;  // status, then P + 1 queue counts
    z.stride = 3 + B + B * P + 2 * Smax;
    z.zero = 8 * (z.hdr + slots * z.stride) + 8 * Smax * enc_segments(g->R) + 4 * kTicketStride * Smax;
    z.fm = 8 * n;
    z.ubits = 8 * (n / 64);
    z.dstate = (int64_t)sizeof(BDirState);
    return z;
}

}  // namespace

extern "C" int64_t csbfs_batch_engine_bytes(const csbfs_graph *g, int32_t max_roots, int32_t max_levels,
                                            uint32_t flags) {
    if (!g || max_roots < 1 || max_roots > kMaxRoots || max_levels < 1 || max_levels > 65536) return -1;
    return batch_sizes(g, max_roots, max_levels, flags).total();
}

namespace csbfs {

// A batch engine on a device block `mem` of csbfs_batch_engine_bytes bytes
// and a pinned two-word host buffer, both owned by the caller (null: the
// engine allocates them itself). Zeroing runs on `st` and is awaited with a
// synchronization of `st` alone.
int batch_engine_make(const csbfs_graph *g, int32_t max_roots, int32_t max_levels, uint32_t flags, void *mem,
                      unsigned long long *host_ctl, hipStream_t st, csbfs_batch_engine **out) {
    if (!out) return fail(CSBFS_EINVAL, "csbfs_batch_engine_create: out is NULL");
    *out = nullptr;
    if (!g) return fail(CSBFS_EINVAL, "csbfs_batch_engine_create: graph is NULL");
    if (max_roots < 1 || max_roots > kMaxRoots)
        return fail(CSBFS_EINVAL, "csbfs_batch_engine_create: max_roots outside [1, 64]");
    if (max_levels < 1 || max_levels > 65536)
        return fail(CSBFS_EINVAL, "csbfs_batch_engine_create: max_levels outside [1, 65536]");
    if (flags & ~(CSBFS_FLAG_TIMING | CSBFS_FLAG_KEEP_STREAMS | CSBFS_FLAG_NO_SIEVE | CSBFS_FLAG_SPARSE_ONLY |
                  CSBFS_FLAG_BOTTOM_UP_ONLY))
        return fail(CSBFS_EINVAL, "csbfs_batch_engine_create: unsupported flag");
    if ((flags & CSBFS_FLAG_SPARSE_ONLY) && (flags & CSBFS_FLAG_BOTTOM_UP_ONLY))
        return fail(CSBFS_EINVAL, "csbfs_batch_engine_create: SPARSE_ONLY and BOTTOM_UP_ONLY exclude each other");
    int rc = graph_device_check(g);
    if (rc) return rc;
    std::unique_ptr<csbfs_batch_engine> e(new csbfs_batch_engine());
    e->g = g;
    e->Bmax = max_roots;
    e->L = max_levels;
    e->flags = flags;
    const int64_t P = g->P, n = g->n, B = max_roots;
    e->cap = wah_cap(g->R);
    e->nseg = enc_segments(g->R);
    e->nchunk = dec_chunks(g->R);
    e->Smax = B * P * P;
    std::vector<int64_t> qoff(P + 1, 0);
    for (int64_t r = 0; r < P; ++r) qoff[r + 1] = qoff[r] + g->big_items[r];
    const BatchSizes z = batch_sizes(g, B, max_levels, flags);
    if (!mem) {
        rc = device_malloc(&e->mem, (size_t)z.total());
        if (rc) return rc;
        e->owns_mem = true;
    } else {
        e->mem = mem;
    }
    if (!host_ctl) {
        const hipError_t herr = hipHostMalloc((void **)&e->host_ctl, 2 * sizeof(unsigned long long));
        if (herr != hipSuccess) {
            e->host_ctl = nullptr;
            bengine_release(e.release());
            return hip_fail(herr, "hipHostMalloc", __FILE__, __LINE__);
        }
        e->owns_host = true;
    } else {
        e->host_ctl = host_ctl;
    }
    char *at = (char *)e->mem;
    auto carve = [&at](int64_t bytes) {
        void *p = at;
        at += align_up(bytes > 0 ? bytes : 1);
        return p;
    };
    e->vn = (uint64_t *)carve(z.vis);
    e->f = (uint64_t *)carve(z.f);
    e->view = (uint64_t *)carve(z.view);
    e->arena = (uint64_t *)carve(z.arena);
    e->chunk_groups = (int64_t *)carve(z.chunk);
    e->queue = (BItem *)carve(z.queue);
    e->qoff = (int64_t *)carve(z.qoff);
    e->zero_mem = (uint32_t *)carve(z.zero);
    e->zero_words = z.zero / 4;
    e->hdr = z.hdr;
    e->stride = z.stride;
    e->status = (int32_t *)e->zero_mem;
    e->qcount = e->zero_mem + 2;
    e->recs = (unsigned long long *)e->zero_mem + z.hdr;
    e->look = e->recs + ((int64_t)max_levels + 1) * z.stride;
    e->enc_ticket = reinterpret_cast<uint32_t *>(e->look + e->Smax * e->nseg);
    e->fm = (uint64_t *)carve(z.fm);
    e->ubits = (uint64_t *)carve(z.ubits);
    e->dstate = (BDirState *)carve(z.dstate);
    e->pqueue = (BPullItem *)carve(z.pqueue);
    e->pqueue_cap = pull_long_rows(g->nnz);
    void *hdev = nullptr;
    hipError_t herr = hipHostGetDevicePointer(&hdev, e->host_ctl, 0);
    e->host_ctl_dev = (unsigned long long *)hdev;
    if (herr == hipSuccess)
        herr = hipMemcpyAsync(e->qoff, qoff.data(), sizeof(int64_t) * (P + 1), hipMemcpyHostToDevice, st);
    if (herr == hipSuccess) herr = hipMemsetAsync(e->view, 0, sizeof(uint64_t) * B * P * (n / 64), st);
    if (herr == hipSuccess) herr = hipStreamSynchronize(st);  // qoff is read from host memory
    if (herr == hipSuccess && (flags & CSBFS_FLAG_TIMING)) {
        e->events.assign((size_t)max_levels * kBEvPerLevel, nullptr);
        for (auto &ev : e->events)  // timestamps only: no system-scope fence at each record
            if (herr == hipSuccess) herr = hipEventCreateWithFlags(&ev, hipEventDisableSystemFence);
    }
    if (herr != hipSuccess) {
        bengine_release(e.release());
        return hip_fail(herr, "csbfs_batch_engine_create", __FILE__, __LINE__);
    }
    *out = e.release();
    return CSBFS_OK;
}

void batch_engine_release(csbfs_batch_engine *e) {
    if (e) bengine_release(e);
}

}  // namespace csbfs

extern "C" int csbfs_batch_engine_create(const csbfs_graph *g, int32_t max_roots, int32_t max_levels,
                                         uint32_t flags, csbfs_batch_engine **out) {
    return batch_engine_make(g, max_roots, max_levels, flags, nullptr, nullptr, nullptr, out);
}

extern "C" int csbfs_batch_engine_free(csbfs_batch_engine *e) {
    if (!e) return CSBFS_OK;
    bengine_release(e);
    return CSBFS_OK;
}

extern "C" int csbfs_batch_bfs(csbfs_batch_engine *e, const int64_t *roots, int32_t n_roots,
                               int32_t *level, csbfs_level_stats *stats, int32_t stats_cap,
                               int32_t *n_levels, void *stream) {
    if (!e || !level) return fail(CSBFS_EINVAL, "csbfs_batch_bfs: null argument or negative stats_cap");
    int32_t *rows[kMaxRoots];
    for (int32_t r = 0; r < n_roots && r < kMaxRoots; ++r) rows[r] = level + (int64_t)r * e->g->n;
    return batch_bfs_into(e, roots, n_roots, rows, stats, stats_cap, n_levels, stream);
}

namespace csbfs {

int batch_bfs_into(csbfs_batch_engine *e, const int64_t *roots, int32_t n_roots, int32_t *const *level,
                   csbfs_level_stats *stats, int32_t stats_cap, int32_t *n_levels, void *stream) {
    if (!e || !roots || !level || !n_levels || stats_cap < 0 || (stats_cap > 0 && !stats))
        return fail(CSBFS_EINVAL, "csbfs_batch_bfs: null argument or negative stats_cap");
    if (n_roots < 1 || n_roots > e->Bmax)
        return fail(CSBFS_EINVAL, "csbfs_batch_bfs: n_roots outside [1, max_roots]");
    const csbfs_graph *g = e->g;
    for (int32_t r = 0; r < n_roots; ++r)
        if (roots[r] < 0 || roots[r] >= g->n) return fail(CSBFS_ERANGE, "csbfs_batch_bfs: root outside [0, n)");
    int rc = graph_device_check(g);
    if (rc) return rc;
    hipStream_t st = as_stream(stream);
    const int64_t P = g->P, n = g->n, R = g->R, W = g->W, B = n_roots, Bm = e->Bmax;
    const int64_t words = n / 64, vplane = P * words;
    const bool timing = (e->flags & CSBFS_FLAG_TIMING) != 0;
    const bool keep = (e->flags & CSBFS_FLAG_KEEP_STREAMS) != 0;

    // a0: seed every root
    // (its fill also clears the counters and the encoder's tickets, which count
    // on over the batch's levels)
    BLevels lv{};
    std::copy(level, level + B, lv.p);
    BSeedArgs sa{e->vn, e->fm, e->view, B * vplane, lv, n, e->zero_mem, e->zero_words};
    BRoots rt{};
    std::copy(roots, roots + B, rt.v);
    e->host_ctl[0] = e->host_ctl[1] = 0;  // level tags start at 1
    // evaluation of each level: top-down, bottom-up, or chosen on the device
    const int32_t force = (e->flags & CSBFS_FLAG_SPARSE_ONLY)      ? CSBFS_DIR_TOP_DOWN
                          : (e->flags & CSBFS_FLAG_BOTTOM_UP_ONLY) ? CSBFS_DIR_BOTTOM_UP
                                                                   : -1;
    const int32_t dir0 = force == CSBFS_DIR_BOTTOM_UP ? CSBFS_DIR_BOTTOM_UP : CSBFS_DIR_TOP_DOWN;
    const int64_t fill = std::max(std::max(B * n, B * vplane), e->zero_words);
    hipLaunchKernelGGL(bseed_fill_kernel, dim3(grid_for(fill, 256 * B, 16384 / B), (unsigned)B), dim3(256),
                       0, st, sa);
    CSBFS_HIP(hipGetLastError());
    hipLaunchKernelGGL(bseed_root_kernel, dim3(1), dim3(64), 0, st, sa, rt, (int32_t)B, R, W, (int32_t)P,
                       vplane, e->rootc(0), e->ctl(0), e->dstate, dir0, force, e->dir(0));
    CSBFS_HIP(hipGetLastError());

    BArgs ea{};
    ea.view = e->view;
    ea.vplane = vplane;
    ea.B = (int32_t)B;
    ea.row_ptr = g->row_ptr;
    ea.col_base = g->col_base;
    ea.col = g->col;
    ea.vn = e->vn;
    ea.queue = e->queue;
    ea.qoff = e->qoff;
    ea.queue_count = e->qcount;
    ea.R = R;
    ea.W = W;
    ea.P = (int32_t)P;
    ea.status = e->status;
    ea.dir = &e->dstate->cur;
    const unsigned grid = 2048;
    BPullArgs pa{};
    pa.vn = e->vn;
    pa.fm = e->fm;
    pa.pull_off = g->pull_off;
    pa.pull_col = g->pull_col;
    pa.head = g->head;
    pa.view = e->view;
    pa.view_words = B * vplane;
    pa.n = n;
    pa.B = (int32_t)B;
    pa.dir = &e->dstate->cur;
    pa.queue = e->pqueue;
    pa.queue_cap = e->pqueue_cap;
    pa.queue_count = e->qcount + P;
    pa.status = e->status;

    WahBatch wb{};
    wb.bits_base = e->f;
    wb.mask_base = (e->flags & CSBFS_FLAG_NO_SIEVE) ? nullptr : g->dir;
    wb.nbits = R;
    wb.words_per_piece = W;
    wb.cap = e->cap;
    wb.P = (int32_t)P;
    wb.planes = (int32_t)B;
    wb.bits_plane_stride = words;
    wb.dst_plane_stride = vplane;
    wb.look = e->look;
    wb.ticket = e->enc_ticket;
    wb.nseg = e->nseg;
    wb.chunk_groups = e->chunk_groups;
    wb.nchunk = e->nchunk;
    wb.chunk_starts = 1;  // the decode reads the chunk starts the encode records
    wb.dst_base = e->view;
    wb.status = e->status;

    auto slot = [&](int64_t k) { return k < e->L ? k : (int64_t)e->L; };
    auto enqueue_iter = [&](int64_t j) -> int {
        const int64_t sj = slot(j), sn = slot(j + 1);
        hipEvent_t *evp = (timing && j >= 1 && j - 1 < e->L) ? &e->events[(size_t)(j - 1) * kBEvPerLevel] : nullptr;
        hipEvent_t *ev = (timing && j < e->L) ? &e->events[(size_t)j * kBEvPerLevel] : nullptr;
        if (j >= 1) {
            wb.out_base = e->arena + (keep ? sj : 0) * e->Smax * e->cap;
            wb.n_words = e->words(sj);
            wb.stat_sieved_bits = e->sbits(sj);
            wb.stat_unsieved_words = e->uwords(sj);
            // roots whose level-j frontier is empty send nothing (the counter
            // slot past max_levels is reset before this encode: no skipping)
            wb.plane_count = j < e->L ? e->rootc(sj) : nullptr;
            const BDirArgs bd{e->dstate, j < e->L ? e->dir(j) : nullptr, n, kBatchAlpha, kBatchBeta, e->ctl(sj),
                              e->host_ctl_dev + (j & 1), j};
            hipLaunchKernelGGL(bencode_kernel, dim3((unsigned)wb.nseg, (unsigned)batch_streams(wb)), dim3(kEncThreads), 0,
                               st, wb, bd);
            CSBFS_HIP(hipGetLastError());
            if (evp) CSBFS_HIP(hipEventRecord(evp[3], st));
            const int r2 = launch_wah_decode(wb, st);
            if (r2) return r2;
            if (evp) CSBFS_HIP(hipEventRecord(evp[4], st));
        }
        // the slot past max_levels, once this level's size has been posted
        if (j + 1 >= e->L) CSBFS_HIP(hipMemsetAsync(e->ctl(e->L), 0, 8 * e->stride, st));
        if (ev) CSBFS_HIP(hipEventRecord(ev[0], st));
        // the iteration after the last level (one of look-ahead) does nothing
        const unsigned long long *fc = j < e->L ? e->ctl(sj) : nullptr;
        ea.edges = e->edges(sj);
        ea.fcount = fc;
        hipLaunchKernelGGL(bexpand_kernel, dim3(grid), dim3(kBThreads), 0, st, ea);
        CSBFS_HIP(hipGetLastError());
        // the bottom-up evaluation (returns at once on top-down levels); past
        // the kept counters every root counts as active
        pa.rootc = j < e->L ? e->rootc(sj) : nullptr;
        pa.edges = e->edges(sj);
        pa.fcount = fc;
        pa.st = e->dstate;
        pa.ubits = j > 0 && n >= kBBitmapVerts ? e->ubits : nullptr;  // no update made f^0
        hipLaunchKernelGGL(bpull_kernel, dim3(grid), dim3(kBThreads), 0, st, pa);
        CSBFS_HIP(hipGetLastError());
        // long rows: 1024 workgroups beat 512, 2048 and 4096 (a sweep, within 2%)
        hipLaunchKernelGGL(blong_kernel, dim3(1024), dim3(kBThreads), 0, st, ea, pa);
        CSBFS_HIP(hipGetLastError());
        if (ev) CSBFS_HIP(hipEventRecord(ev[1], st));
        BUpdateArgs ua{e->vn, e->f, lv, (int32_t)(j + 1), (int32_t)B, n,
                       e->rootc(sn), e->ctl(sn), e->qcount, (int32_t)P, fc,
                       e->fm, e->ubits, g->deg, e->dstate->sums};
        hipLaunchKernelGGL(bupdate_kernel, dim3(grid_for((words + kBTile - 1) / kBTile, kBThreads / 64, 2048)), dim3(kBThreads), 0, st, ua);
        CSBFS_HIP(hipGetLastError());
        if (ev) CSBFS_HIP(hipEventRecord(ev[2], st));
        return CSBFS_OK;
    };

    // the size of level k's frontier, posted by its encode (polled)
    auto wait_count = [&](int64_t k, unsigned long long *cnt) -> int {
        const unsigned long long want = (unsigned long long)k & ((1ull << (64 - kPostBits)) - 1);
        volatile unsigned long long *word = e->host_ctl + (k & 1);
        for (uint64_t spins = 1;; ++spins) {
            hipError_t q = hipErrorNotReady;
            // a failed launch never writes the word: ask the stream now and then
            if ((spins & 0x3ff) == 0) q = hipStreamQuery(st);
            if (q != hipSuccess && q != hipErrorNotReady) return hip_fail(q, "batch stream", __FILE__, __LINE__);
            const unsigned long long v = *word;  // read after the query: a drained stream has posted
            if ((v >> kPostBits) == want) {
                *cnt = v & ((1ull << kPostBits) - 1);
                return CSBFS_OK;
            }
            if (q == hipSuccess) return fail(CSBFS_ECORRUPT, "csbfs_batch_bfs: a level's frontier size never arrived");
        }
    };
    rc = enqueue_iter(0);
    if (rc) return rc;
    int64_t k = 0;
    for (;; ++k) {
        // the size is posted by the first kernel of iteration k + 1; the rest
        // of that iteration hides the host's answer
        rc = enqueue_iter(k + 1);
        if (rc) return rc;
        unsigned long long cnt = 0;
        rc = wait_count(k + 1, &cnt);
        if (rc) {
            (void)hipStreamSynchronize(st);
            return rc;
        }
        if (cnt == 0) break;
    }
    const int64_t nl = k + 1;
    *n_levels = (int32_t)(nl < INT32_MAX ? nl : INT32_MAX);
    e->last_levels = *n_levels;
    e->last_roots = (int32_t)B;

    // status and statistics: the header and the records of the levels wanted
    const int64_t have = nl < e->L ? nl : e->L;
    const int64_t want = stats_cap < have ? stats_cap : have;
    std::vector<unsigned long long> rec((size_t)(e->hdr + want * e->stride));
    CSBFS_HIP(hipMemcpyAsync(rec.data(), e->zero_mem, 8 * rec.size(), hipMemcpyDeviceToHost, st));
    CSBFS_HIP(hipStreamSynchronize(st));
    const int32_t hstatus = (int32_t)rec[0];
    if (hstatus != 0) {
        if (hstatus == 1) return fail(CSBFS_ECORRUPT, "csbfs_batch_bfs: a stream failed validation while decoding");
        return fail(CSBFS_ECORRUPT, "csbfs_batch_bfs: internal consistency check failed");
    }
    for (int64_t lv = 0; lv < want; ++lv) {
        csbfs_level_stats &s = stats[lv];
        s = csbfs_level_stats{};
        const unsigned long long *r0 = rec.data() + e->hdr + lv * e->stride;
        const unsigned long long *rootc = r0 + 3, *uw = rootc + Bm, *sb = uw + Bm * P, *wd = sb + e->Smax;
        s.edges = (int64_t)r0[1];
        s.direction = (int32_t)r0[2];
        std::vector<int64_t> send(P, 0), recv(P, 0);
        for (int64_t r = 0; r < B; ++r) {
            const int64_t fr = (int64_t)rootc[r];
            if (fr == 0) continue;
            s.frontier += fr;
            if (lv == 0) {
                s.view_bits += P;
                continue;
            }
            s.unsieved_bits += (P - 1) * fr;
            s.raw_bytes += P * (P - 1) * 8 * W;
            for (int64_t i = 0; i < P; ++i) {
                s.wah_unsieved_bytes += 8 * (P - 1) * (int64_t)uw[r * P + i];
                for (int64_t j = 0; j < P; ++j) {
                    const int64_t sidx = (r * P + i) * P + j;
                    s.view_bits += (int64_t)sb[sidx];
                    if (i == j) {
                        s.self_bytes += 8 * (int64_t)wd[sidx];
                        continue;
                    }
                    s.sieved_bits += (int64_t)sb[sidx];
                    s.wah_sieved_bytes += 8 * (int64_t)wd[sidx];
                    send[i] += 8 * (int64_t)wd[sidx];
                    recv[j] += 8 * (int64_t)wd[sidx];
                }
            }
        }
        for (int64_t i = 0; i < P; ++i) s.max_rank_bytes = std::max(s.max_rank_bytes, send[i] + recv[i]);
    }
    if (timing) {
        for (int64_t lv = 0; lv < nl && lv < e->L; ++lv) {
            hipEvent_t *ev = &e->events[(size_t)lv * kBEvPerLevel];
            float a = 0, b = 0;
            CSBFS_HIP(hipEventElapsedTime(&a, ev[0], ev[1]));
            CSBFS_HIP(hipEventElapsedTime(&b, ev[1], ev[2]));
            if (lv < want) {
                stats[lv].ms_expand = a;
                stats[lv].ms_update = b;
            }
            if (lv + 1 < nl && lv + 1 < want) {
                float c = 0, d = 0;
                CSBFS_HIP(hipEventElapsedTime(&c, ev[2], ev[3]));
                CSBFS_HIP(hipEventElapsedTime(&d, ev[3], ev[4]));
                stats[lv + 1].ms_compress = c;
                stats[lv + 1].ms_decode = d;
            }
        }
    }
    return CSBFS_OK;
}

}  // namespace csbfs

extern "C" int csbfs_batch_stream_words(const csbfs_batch_engine *e, int32_t *words, int32_t cap_levels) {
    if (!e || !words || cap_levels < 0) return fail(CSBFS_EINVAL, "csbfs_batch_stream_words: bad argument");
    const int64_t P = e->g->P, B = e->last_roots, Bm = e->Bmax;
    const int64_t lv_have = std::min<int64_t>(e->L, e->last_levels);
    std::vector<unsigned long long> rec((size_t)(lv_have * e->stride) + 1);
    if (lv_have > 0)
        CSBFS_HIP(hipMemcpy(rec.data(), e->ctl(0), sizeof(unsigned long long) * lv_have * e->stride,
                            hipMemcpyDeviceToHost));
    const int64_t words_at = 3 + Bm + Bm * P + e->Smax;
    for (int64_t lv = 0; lv < cap_levels; ++lv)
        for (int64_t r = 0; r < B; ++r)
            for (int64_t s = 0; s < P * P; ++s) {
                const unsigned long long *r0 = rec.data() + lv * e->stride;
                const bool live = lv > 0 && lv < lv_have && r0[3 + r] > 0;
                words[(lv * B + r) * P * P + s] = live ? (int32_t)r0[words_at + r * P * P + s] : 0;
            }
    return CSBFS_OK;
}

extern "C" int csbfs_batch_copy_stream(const csbfs_batch_engine *e, int32_t k, int32_t r, int32_t i,
                                       int32_t j, uint64_t *dst, int64_t cap_words, int64_t *n_words_out,
                                       void *stream) {
    if (!e || !dst || !n_words_out) return fail(CSBFS_EINVAL, "csbfs_batch_copy_stream: null argument");
    if (!(e->flags & CSBFS_FLAG_KEEP_STREAMS))
        return fail(CSBFS_EINVAL, "csbfs_batch_copy_stream: engine lacks CSBFS_FLAG_KEEP_STREAMS");
    const int64_t P = e->g->P;
    if (k < 0 || k >= e->L || k >= e->last_levels || r < 0 || r >= e->last_roots || i < 0 || i >= P ||
        j < 0 || j >= P)
        return fail(CSBFS_EINVAL, "csbfs_batch_copy_stream: level, root or processor out of range");
    const int64_t s = ((int64_t)r * P + i) * P + j;
    hipStream_t st = as_stream(stream);
    int64_t nw = 0;
    unsigned long long fr = 0;
    CSBFS_HIP(hipMemcpyAsync(&fr, e->rootc(k) + r, sizeof(fr), hipMemcpyDeviceToHost, st));
    CSBFS_HIP(hipMemcpyAsync(&nw, e->words(k) + s, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    CSBFS_HIP(hipStreamSynchronize(st));
    if (k == 0 || fr == 0) nw = 0;  // no message carries level 0 or an empty frontier
    *n_words_out = nw;
    if (nw > cap_words) return fail(CSBFS_ENOSPACE, "csbfs_batch_copy_stream: dst too small");
    if (nw > 0)
        CSBFS_HIP(hipMemcpyAsync(dst, e->arena + ((int64_t)k * e->Smax + s) * e->cap, sizeof(uint64_t) * nw,
                                 hipMemcpyDeviceToDevice, st));
    CSBFS_HIP(hipStreamSynchronize(st));
    return CSBFS_OK;
}
