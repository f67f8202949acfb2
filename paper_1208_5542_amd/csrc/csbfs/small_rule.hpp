#pragma once
// Which searches one workgroup makes in one launch (bfs_small.hpp), and where
// their state lies in its LDS. Host arithmetic only.
#include "common.hpp"

namespace csbfs {

constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / 64;
constexpr int kSmallQueue = 512;  // long rows per level (a row that finds no slot stays with its wave)

// Places in LDS, in 64-bit words.
struct SmallLds {
    int32_t pi, nb, view, buf, nbuf, buf_words, par, queue, total;
};
inline SmallLds small_lds(int64_t n, int64_t P) {
    const int64_t words = n / 64, R = n / P, S = P * P;
    SmallLds l{};
    int64_t o = 0;
    auto take = [&o](int64_t w) {
        const int64_t at = o;
        o += w;
        return (int32_t)at;
    };
    l.nbuf = (int32_t)(S < kSmallWaves ? S : kSmallWaves);
    l.buf_words = (int32_t)(R / 64 + 1 + wah_cap(R));  // a sieved piece and its stream
    l.pi = take(words);
    l.nb = take(2 * words);
    l.view = take(P * words);
    l.buf = take((int64_t)l.nbuf * l.buf_words);
    l.par = take((n + 1) / 2);
    l.queue = take(2 * kSmallQueue);
    l.total = (int32_t)o;
    return l;
}

// The state fits LDS, the adjacency is short enough for one CU, and a level's
// p * p streams, which the workgroup's 16 waves encode and decode one after
// another, cost less than the level-by-level kernels, which spread them over the
// GPU.
//
// Entries: the limit lies where the level-by-level kernels' time (220 to 260 us,
// launches mostly) is reached: with 2^19 entries (R-MAT scale 14) 128 us, with
// 580k (uniform, 16128 vertices) 196 us against 251, with 2^20 222 us against
// 234 (R-MAT scale 15) and 284 against 257 (uniform, 25600 vertices).
//
// Streams: a level of almost no work takes about 6 us and another 1.9 per stream
// and wave, against 27 to 31 us of four launches, and the more vertices the
// more of that is spent without streams; one stream weighs as much as 160
// vertices. One launch / level kernels, uniform graphs with 4 entries a vertex, in
// us, on either side of the rule: 8 processors, 22528 vertices 342 / 399; 10,
// 15360 334 / 404; 12, 9216 346 / 413 and 18432 427 / 394; 13, 4992 293 / 360
// and 19968 501 / 424; 14, 896 238 / 295 and 14336 461 / 391; 16, 1024 305 /
// 283; 32, 2048 1204 / 436; 64, 4096 4474 / 848. A path of 400 levels: 14, 896
// 10.5 / 12.5 ms; 16, 1024 (a mesh of 62 levels) 2.08 / 1.71 ms.
constexpr int64_t kSmallNnz = int64_t(3) << 18;
constexpr int64_t kSmallVerts = int64_t(1) << 15, kSmallStreamVerts = 160;
constexpr int64_t kSmallLdsBytes = 160 * 1024 - 1024;  // the rest: its shared counters
inline bool small_fits(int64_t n, int64_t P, int64_t nnz) {
    return nnz <= kSmallNnz && n + kSmallStreamVerts * P * P <= kSmallVerts &&
           8 * (int64_t)small_lds(n, P).total <= kSmallLdsBytes;
}

}  // namespace csbfs
