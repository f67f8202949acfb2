#pragma once
// A whole search of a small graph in one launch of one workgroup (included by
// bfs.hip). Every bitmap of Algorithm 3 (visited bits, new-vertex bits, the
// p * p views) and the parents live in LDS, so a level's steps are separated
// by workgroup barriers instead of launches, and its atomics are LDS atomics.
// Messages are the same: stream i -> j is sieved, WAH-64 encoded by one wave
// (written to the arena like any stream) and decoded by that wave into view
// (j, i). small_rule.hpp says which searches.
//
// Bound by latency, and by one CU's issue rate towards the upper limit: the
// searches this serves touch a few 10^5 adjacency entries in 6 to 8 levels,
// and four launches per level of at least 6 us each were most of their time.
// R-MAT scale 10, p 1 212 -> 48 us a search; scale 12, p 4 219 -> 65; scale
// 14, p 4 242 -> 128.
namespace csbfs {
namespace {

constexpr int kSmallLong = 256;    // longer rows are pushed by the whole workgroup
constexpr int kSmallUnroll = 4;    // adjacency entries in flight per lane

struct SmallItem {
    int32_t col, len, u, vbase;
};
static_assert(sizeof(SmallItem) == 16, "two words of the queue's LDS");

struct SmallArgs {
    SmallLds l;
    int32_t n, R, W, P, root;
    const int32_t *row_ptr;
    const int64_t *col_base;
    const uint32_t *col;
    const uint64_t *mask;  // directory, or null (no sieve)
    const int32_t *deg;
    const uint64_t *live;
    const int64_t *pull_off;
    const uint32_t *pull_col;
    const uint32_t *head;
    int32_t *level, *parent;
    uint64_t *arena;
    int64_t cap, arena_stride;  // words per stream; words per kept level (0: one slot)
    unsigned long long *hdr;    // [1] status, [2] levels
    LevelCounters lc;
    int64_t L;
    unsigned long long *host;   // pinned word (status << 32 | levels), or null
    DirArgs dir;                // st and rec unused
    int32_t dir0;
};

struct SmallShared {
    unsigned long long nf, mf, edges, pulled;
    uint32_t queued;
    int32_t bad;
    DirState dir;
};

__device__ __forceinline__ unsigned long long wave_sum64(unsigned long long v) {
    return readlane64((uint64_t)wave_incl_scan_i64((long long)v), 63);
}

// Relaxes kSmallUnroll (target v, source u) pairs.
__device__ __forceinline__ void small_relax(const uint64_t *pi, uint64_t *nb, int32_t *par,
                                            const int32_t (&v)[kSmallUnroll], const int32_t (&u)[kSmallUnroll],
                                            const bool (&ok)[kSmallUnroll]) {
#pragma unroll
    for (int k = 0; k < kSmallUnroll; ++k) {
        const uint64_t bit = 1ull << (v[k] & 63);
        if (ok[k] && !(pi[v[k] >> 6] & bit) && atomicMax(&par[v[k]], u[k]) < 0)
            atomicOr((unsigned long long *)&nb[v[k] >> 6], (unsigned long long)bit);
    }
}

// Top-down: the view words are dealt to the waves in tiles, and a tile's
// sources are taken 64 at a time with their edges spread evenly over the
// lanes, as in the large graphs' push.
__device__ void small_push(const SmallArgs &a, SmallShared &sh, const uint64_t *pi, uint64_t *nb,
                           const uint64_t *view, int32_t *par, SmallItem *queue) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int32_t total_words = a.P * (a.n / 64), PW = a.P * a.W;
    int32_t tw = (total_words + kSmallWaves - 1) / kSmallWaves;
    tw = tw > 64 ? 64 : tw;
    const int32_t ntiles = (total_words + tw - 1) / tw;
    unsigned long long edges = 0;
    for (int32_t t = wid; t < ntiles; t += kSmallWaves) {
        const int32_t wi0 = t * tw + lane;
        const uint64_t bits = lane < tw && wi0 < total_words ? view[wi0] : 0;
        const int cnt = __popcll(bits);
        const int incl_b = wave_incl_scan_i32(cnt);
        const int tot_b = __builtin_amdgcn_readlane(incl_b, 63);
        const int excl_b = incl_b - cnt;
        for (int base = 0; base < tot_b; base += 64) {
            const int rk = base + lane;
            const int ln = owner_lane(excl_b, rk < tot_b ? rk : tot_b - 1);
            const uint64_t wb = __shfl(bits, ln, 64);
            const int rr = rk - __shfl(excl_b, ln, 64);
            int32_t deg = 0, u = 0, gstart = 0, vbase = 0;
            if (rk < tot_b) {
                const int32_t wi = t * tw + ln;
                const int32_t b = wi / a.W, r = wi / PW;
                const int32_t ul = ((wi - b * a.W) << 6) + select_bit(wb, rr);
                const int32_t *rp = a.row_ptr + (int64_t)b * (a.R + 1) + ul;
                const int32_t rs = rp[0];
                deg = rp[1] - rs;
                gstart = (int32_t)a.col_base[b] + rs;
                u = (b - r * a.P) * a.R + ul;
                vbase = r * a.R;
            }
            edges += wave_sum64((unsigned long long)deg);
            const bool far = deg > kSmallLong;
            const uint64_t fars = __ballot(far);
            if (fars) {
                uint32_t at = 0;
                if (lane == 0) at = atomicAdd(&sh.queued, (uint32_t)__popcll(fars));
                at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
                const uint32_t pos = at + (uint32_t)__popcll(fars & ((1ull << lane) - 1));
                if (far && pos < kSmallQueue) {
                    queue[pos] = SmallItem{gstart, deg, u, vbase};
                    deg = 0;
                }
            }
            const int32_t incl = wave_incl_scan_i32(deg);
            const int32_t total = __builtin_amdgcn_readlane(incl, 63);
            const int32_t excl = incl - deg;
            for (int32_t e0 = 0; e0 < total; e0 += 64 * kSmallUnroll) {
                int32_t v[kSmallUnroll], uu[kSmallUnroll];
                bool ok[kSmallUnroll];
#pragma unroll
                for (int k = 0; k < kSmallUnroll; ++k) {
                    const int32_t e = e0 + 64 * k + lane;
                    ok[k] = e < total;
                    const int o = owner_lane(excl, ok[k] ? e : total - 1);
                    const int32_t gs = __shfl(gstart, o, 64), ex = __shfl(excl, o, 64);
                    uu[k] = __shfl(u, o, 64);
                    v[k] = __shfl(vbase, o, 64);
                    v[k] += (int32_t)a.col[gs + ((ok[k] ? e : total - 1) - ex)];
                }
                small_relax(pi, nb, par, v, uu, ok);
            }
        }
    }
    if (lane == 0 && edges) atomicAdd(&sh.edges, edges);
    __syncthreads();
    // long rows, in chunks dealt to the waves
    const int32_t nq = sh.queued < (uint32_t)kSmallQueue ? (int32_t)sh.queued : kSmallQueue;
    int32_t chunk = 0;
    for (int32_t q = 0; q < nq; ++q) {
        const SmallItem it = queue[q];
        for (int32_t e0 = 0; e0 < it.len; e0 += 64 * kSmallUnroll, ++chunk) {
            if (chunk % kSmallWaves != wid) continue;
            int32_t v[kSmallUnroll], uu[kSmallUnroll];
            bool ok[kSmallUnroll];
#pragma unroll
            for (int k = 0; k < kSmallUnroll; ++k) {
                const int32_t e = e0 + 64 * k + lane;
                ok[k] = e < it.len;
                uu[k] = it.u;
                v[k] = it.vbase + (int32_t)a.col[it.col + (ok[k] ? e : it.len - 1)];
            }
            small_relax(pi, nb, par, v, uu, ok);
        }
    }
}

// Bottom-up: a wave takes a bitmap word (lane = vertex; two or four words at
// once were slower: the CU's issue slots are full); each candidate tests its
// row's first two ids, then kPullWindow entries a step; lanes still searching
// after 32 entries are finished by the wave.
__device__ void small_pull(const SmallArgs &a, SmallShared &sh, const uint64_t *pi, uint64_t *nb,
                           const uint64_t *view, int32_t *par) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int32_t words = a.n / 64;
    unsigned long long pulled = 0, read = 0;
    for (int32_t w = wid; w < words; w += kSmallWaves) {
        const uint64_t t = a.live[w] & ~pi[w];
        if (!t) continue;
        pulled += (unsigned long long)__popcll(t);
        const int32_t v = (w << 6) + lane;
        const uint64_t *vw = view + w / a.W * a.P * a.W;
        bool busy = (t >> lane) & 1;
        int32_t e = 0, re = 0, found = -1;
        if (busy) {
            e = (int32_t)a.pull_off[v];
            re = (int32_t)a.pull_off[v + 1];
            const uint2 hd = *reinterpret_cast<const uint2 *>(a.head + 2 * (int64_t)v);
            const int32_t nk = re - e < 2 ? re - e : 2;
            const uint32_t c0 = hd.x, c1 = nk > 1 ? hd.y : hd.x;
            const uint32_t hm = ((uint32_t)((vw[c0 >> 6] >> (c0 & 63)) & 1) |
                                 ((uint32_t)((vw[c1 >> 6] >> (c1 & 63)) & 1) << 1)) & ((1u << nk) - 1u);
            if (hm) {
                const int hit = __builtin_ctz(hm);
                found = (int32_t)(hit ? c1 : c0);
                read += (unsigned long long)(hit + 1);
                busy = false;
            } else {
                read += (unsigned long long)nk;
                e += nk;
                busy = e < re;
            }
        }
        for (int round = 0; round < kPullRounds * kPullUnroll / kPullWindow && __ballot(busy); ++round) {
            uint32_t c[kPullWindow];
            // positions past the row end are clamped and masked out; an idle
            // lane reads entry 0 (there are entries)
#pragma unroll
            for (int k = 0; k < kPullWindow; ++k) c[k] = a.pull_col[busy ? (e + k < re ? e + k : re - 1) : 0];
            if (!busy) continue;
            const int32_t nk = re - e < kPullWindow ? re - e : kPullWindow;
            uint32_t hm = 0;
#pragma unroll
            for (int k = 0; k < kPullWindow; ++k) hm |= (uint32_t)((vw[c[k] >> 6] >> (c[k] & 63)) & 1) << k;
            hm &= (1u << nk) - 1u;
            if (hm) {
                const int hit = __builtin_ctz(hm);
#pragma unroll
                for (int k = 0; k < kPullWindow; ++k)
                    if (k == hit) found = (int32_t)c[k];
                read += (unsigned long long)(hit + 1);
                busy = false;
            } else {
                read += (unsigned long long)nk;
                e += nk;
                busy = e < re;
            }
        }
        uint64_t slow = __ballot(busy);
        while (slow) {
            const int ln = __ffsll((unsigned long long)slow) - 1;
            slow &= slow - 1;
            int32_t ee = __builtin_amdgcn_readlane(e, ln);
            const int32_t rr = __builtin_amdgcn_readlane(re, ln);
            int32_t got = -1;
            for (; ee < rr && got < 0; ee += 64 * kSmallUnroll) {
                uint32_t c[kSmallUnroll];
#pragma unroll
                for (int k = 0; k < kSmallUnroll; ++k) {
                    const int32_t pos = ee + 64 * k + lane;
                    c[k] = a.pull_col[pos < rr ? pos : rr - 1];
                }
#pragma unroll
                for (int k = 0; k < kSmallUnroll; ++k) {
                    const bool hit = ee + 64 * k + lane < rr && ((vw[c[k] >> 6] >> (c[k] & 63)) & 1);
                    const uint64_t hits = __ballot(hit);
                    if (got < 0 && hits) {
                        const int first = __ffsll((unsigned long long)hits) - 1;
                        got = __builtin_amdgcn_readlane((int)c[k], first);
                        if (lane == 0) read += (unsigned long long)(64 * k + first + 1);
                    }
                }
                if (got < 0 && lane == 0)
                    read += (unsigned long long)(rr - ee < 64 * kSmallUnroll ? rr - ee : 64 * kSmallUnroll);
            }
            if (lane == ln) found = got;
        }
        if (found >= 0) par[v] = found;
        const uint64_t fb = __ballot(found >= 0);
        if (fb && lane == 0) nb[w] = fb;  // this wave's word
    }
    read = wave_sum64(read);
    if (lane == 0) {
        if (read) atomicAdd(&sh.edges, read);
        if (pulled) atomicAdd(&sh.pulled, pulled);
    }
}

// Update of f = nb: visited bits, levels, the frontier's size and entries.
__device__ void small_update(const SmallArgs &a, SmallShared &sh, uint64_t *pi, const uint64_t *nb, int32_t lvl) {
    constexpr int U = 4;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int32_t words = a.n / 64;
    unsigned long long nf = 0, mf = 0;
    for (int32_t w0 = wid; w0 < words; w0 += kSmallWaves * U) {
        uint64_t t[U];
        int32_t d[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int32_t w = w0 + q * kSmallWaves;
            t[q] = w < words ? nb[w] : 0;
            d[q] = 0;
            if ((t[q] >> lane) & 1) {
                d[q] = a.deg[(w << 6) + lane];
                a.level[(w << 6) + lane] = lvl;
            }
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            if (!t[q]) continue;
            if (lane == 0) pi[w0 + q * kSmallWaves] |= t[q];
            nf += (unsigned long long)__popcll(t[q]);
            mf += (unsigned long long)d[q];
        }
    }
    mf = wave_sum64(mf);
    if (lane == 0 && nf) {
        atomicAdd(&sh.nf, nf);
        atomicAdd(&sh.mf, mf);
    }
}

// or_bits and fill_ones on words in LDS.
__device__ __forceinline__ void or_bits_lds(unsigned long long *buf, int64_t bit, uint64_t v, int nbits) {
    const int64_t q = bit >> 6;
    const int sh = (int)(bit & 63);
    const uint64_t lo = v << sh;
    if (lo) atomicOr(&buf[q], (unsigned long long)lo);
    if (sh + nbits > 64) {
        const uint64_t hi = v >> (64 - sh);
        if (hi) atomicOr(&buf[q + 1], (unsigned long long)hi);
    }
}

__device__ void fill_ones_lds(unsigned long long *buf, int64_t lo, int64_t hi) {
    int64_t q0 = lo >> 6, q1 = (hi - 1) >> 6;
    for (int64_t q = q0; q <= q1; ++q) {
        const int64_t a = lo > q * 64 ? lo - q * 64 : 0;
        const int64_t e = hi < q * 64 + 64 ? hi - q * 64 : 64;
        if (a == 0 && e == 64) {
            buf[q] = ~0ull;  // a whole word inside one fill has no other writer
        } else {
            const uint64_t m = (e == 64 ? ~0ull : ((1ull << e) - 1)) & ~((1ull << a) - 1);
            atomicOr(&buf[q], (unsigned long long)m);
        }
    }
}

// Stream i -> j of the frontier piece f_i by one wave: sieve, encode, store,
// decode into view (j, i). `buf` holds the sieved piece and the stream.
__device__ void small_stream(const SmallArgs &a, SmallShared &sh, int32_t i, int32_t j, const uint64_t *nb,
                             uint64_t *view, uint64_t *buf, uint64_t *out, unsigned long long *rec) {
    const int lane = threadIdx.x & 63;
    const int32_t S = a.P * a.P, s = i * a.P + j;
    const int32_t G = a.R / kGroupBits, rest = a.R % kGroupBits;
    const uint64_t *piece = nb + i * a.W;
    uint64_t *words = buf + a.W + 1;
    unsigned long long ones = 0;
    for (int32_t w = lane; w < a.W; w += 64) {
        const uint64_t f = piece[w] & (a.mask ? a.mask[(int64_t)(j * a.P + i) * a.W + w] : ~0ull);
        buf[w] = f;
        ones += (unsigned long long)__popcll(f);
    }
    if (lane == 0) buf[a.W] = 0;
    ones = wave_sum64(ones);
    wave_lds_sync();

    // 64 groups a step: the lanes whose group starts a word place it; a fill
    // that runs past the step stays open until the next start
    int32_t cnt = 0, prev_cls = -1, open_pos = 0, open_at = 0, open_cls = 2;
    for (int32_t x0 = 0; x0 < G; x0 += 64) {
        const int32_t x = x0 + lane;
        const bool in = x < G;
        const uint64_t v = in ? group_bits(buf, x, 0) : 0;
        const int c = in ? group_class(v) : 3;
        int before = __shfl_up(c, 1, 64);
        if (lane == 0) before = prev_cls;
        const bool start = in && (c == 2 || c != before);
        const uint64_t starts = __ballot(start);
        if (starts) {
            const int32_t first = x0 + __ffsll((unsigned long long)starts) - 1;
            if (open_cls != 2 && lane == 0)
                words[open_pos] = kFillFlag | (open_cls == 1 ? kFillBit : 0) | (uint64_t)(first - open_at);
            const int32_t pos = cnt + __popcll(starts & ((1ull << lane) - 1));
            const uint64_t later = lane < 63 ? starts >> (lane + 1) : 0;
            if (start && c == 2) words[pos] = __builtin_bitreverse64(v) >> 1;
            if (start && c != 2 && later)
                words[pos] = kFillFlag | (c == 1 ? kFillBit : 0) |
                             (uint64_t)__ffsll((unsigned long long)later);
            const int last = 63 - __clzll((long long)starts);
            cnt += __popcll(starts);
            open_cls = __builtin_amdgcn_readlane(c, last);
            open_pos = cnt - 1;
            open_at = x0 + last;
        }
        prev_cls = __builtin_amdgcn_readlane(c, 63);
    }
    if (open_cls != 2 && lane == 0)
        words[open_pos] = kFillFlag | (open_cls == 1 ? kFillBit : 0) | (uint64_t)(G - open_at);
    const int32_t nreg = cnt;
    if (rest > 0) {
        if (lane == 0) {
            SegGeom g{};
            g.G = G;
            g.r = rest;
            words[cnt] = active_word(buf, g);
        }
        ++cnt;
    }
    // the unsieved piece's word count (once per sender)
    if (i == j) {
        int32_t starts_n = 0, pc = -1;
        for (int32_t x0 = 0; x0 < G; x0 += 64) {
            const int32_t x = x0 + lane;
            const int c = x < G ? group_class(group_bits(piece, x, 0)) : 3;
            int before = __shfl_up(c, 1, 64);
            if (lane == 0) before = pc;
            starts_n += __popcll(__ballot(x < G && (c == 2 || c != before)));
            pc = __builtin_amdgcn_readlane(c, 63);
        }
        if (lane == 0) rec[3 * kLine + 2 * S + i] = (unsigned long long)(starts_n + (rest > 0 ? 1 : 0));
    }
    if (lane == 0) {
        rec[3 * kLine + s] = (unsigned long long)cnt;
        rec[3 * kLine + S + s] = ones;
    }
    wave_lds_sync();
    for (int32_t w = lane; w < cnt; w += 64) out[(int64_t)s * a.cap + w] = words[w];

    // decode into view (j, i), which starts zeroed
    unsigned long long *dst = (unsigned long long *)(view + (j * a.P + i) * a.W);
    int32_t base = 0;
    bool bad = false;
    for (int32_t w0 = 0; w0 < nreg; w0 += 64) {
        const int32_t w = w0 + lane;
        const uint64_t v = w < nreg ? words[w] : 0;
        const bool fill = (v & kFillFlag) != 0;
        const int32_t g = w < nreg ? (fill ? (int32_t)(v & kCountMask) : 1) : 0;
        const int32_t incl = wave_incl_scan_i32(g);
        const int32_t x = base + incl - g;
        if (w < nreg) {
            if (g <= 0 || x + g > G)
                bad = true;
            else if (!fill)
                or_bits_lds(dst, (int64_t)x * kGroupBits, __builtin_bitreverse64(v) >> 1, kGroupBits);
            else if (v & kFillBit)
                fill_ones_lds(dst, (int64_t)x * kGroupBits, (int64_t)(x + g) * kGroupBits);
        }
        base += __builtin_amdgcn_readlane(incl, 63);
    }
    if (base != G) bad = true;
    if (rest > 0 && lane == 0) {
        const uint64_t av = words[nreg];
        if (av >> rest)
            bad = true;
        else if (av)
            or_bits_lds(dst, (int64_t)G * kGroupBits, __builtin_bitreverse64(av) >> (64 - rest), rest);
    }
    if (bad) sh.bad = 1;
    wave_lds_sync();  // buf is used again by the wave's next stream
}

__global__ __launch_bounds__(kSmallThreads) void small_search_kernel(SmallArgs a) {
    extern __shared__ uint64_t small_mem[];
    __shared__ SmallShared sh;
    const int tid = threadIdx.x, wid = tid >> 6;
    const int32_t words = a.n / 64, S = a.P * a.P;
    uint64_t *pi = small_mem + a.l.pi, *view = small_mem + a.l.view;
    int32_t *par = reinterpret_cast<int32_t *>(small_mem + a.l.par);
    SmallItem *queue = reinterpret_cast<SmallItem *>(small_mem + a.l.queue);
    auto nb_of = [&](int32_t k) { return small_mem + a.l.nb + (k & 1) * words; };
    // f(s) <- s: the source is known to every processor without a message
    const int32_t rw = a.root >> 6;
    const uint64_t bit = 1ull << (a.root & 63);
    for (int32_t k = tid; k < words; k += kSmallThreads) {
        pi[k] = k == rw ? bit : 0;
        nb_of(0)[k] = nb_of(1)[k] = 0;
        for (int32_t i = 0; i < a.P; ++i) view[i * words + k] = k == rw ? bit : 0;
    }
    for (int32_t k = tid; k < a.n; k += kSmallThreads) {
        par[k] = k == a.root ? k : -1;
        a.level[k] = k == a.root ? 0 : -1;
    }
    for (int32_t k = tid; k < a.lc.stride; k += kSmallThreads) a.lc.base[k] = k == 0 ? 1u : k == 2 ? (unsigned)a.dir0 : 0u;
    if (tid == 0) {
        sh.nf = sh.mf = sh.edges = sh.pulled = 0;
        sh.queued = 0;
        sh.bad = 0;
        sh.dir = DirState{};
        sh.dir.cur = a.dir0;
        sh.dir.vdeg = (unsigned long long)a.deg[a.root];
        sh.dir.prev = 1;
    }
    __syncthreads();
    int32_t k = 0;
    for (;; ++k) {
        // expand f^k; the vertices it finds are f^(k+1)
        uint64_t *nb = nb_of(k + 1), *old = nb_of(k);
        if (sh.dir.cur == kDirBU)
            small_pull(a, sh, pi, nb, view, par);
        else
            small_push(a, sh, pi, nb, view, par, queue);
        __syncthreads();
        small_update(a, sh, pi, nb, k + 1);
        for (int32_t q = tid; q < words; q += kSmallThreads) old[q] = 0;
        for (int32_t q = tid; q < a.P * words; q += kSmallThreads) view[q] = 0;
        __syncthreads();
        const unsigned long long nf = sh.nf, mf = sh.mf;
        // levels past the kept records share the last slot
        unsigned long long *cur = a.lc.at(k < a.L ? k : a.L), *next = a.lc.at(k + 1 < a.L ? k + 1 : a.L);
        if (tid == 0) {
            cur[kLine] = sh.edges;
            cur[2 * kLine] = sh.pulled;
        }
        if (nf == 0) break;
        const int64_t slot = a.arena_stride ? (k + 1 < a.L ? k + 1 : a.L) : 0;
        if (wid < a.l.nbuf)
            for (int32_t s = wid; s < S; s += a.l.nbuf)
                small_stream(a, sh, s / a.P, s % a.P, nb, view, small_mem + a.l.buf + wid * a.l.buf_words,
                             a.arena + slot * a.arena_stride, next);
        if (tid == 0) {
            next[0] = nf;
            next[1] = mf;
            DirArgs d = a.dir;
            int32_t rec = 0;
            d.st = &sh.dir;
            d.rec = &rec;
            choose_direction(d, sh.dir, nf, mf);
            next[2] = (unsigned long long)(uint32_t)rec;
            sh.edges = sh.pulled = 0;
            sh.queued = 0;
        }
        __syncthreads();
        if (tid == 0) sh.nf = sh.mf = 0;  // every wave has read them
    }
    for (int32_t q = tid; q < a.n; q += kSmallThreads) a.parent[q] = par[q];
    if (tid == 0) {
        a.hdr[1] = (unsigned long long)(uint32_t)sh.bad;
        a.hdr[2] = (unsigned long long)(k + 1);
        if (a.host)
            __hip_atomic_store(a.host, ((unsigned long long)(uint32_t)sh.bad << 32) | (unsigned long long)(k + 1),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

}  // namespace
}  // namespace csbfs
