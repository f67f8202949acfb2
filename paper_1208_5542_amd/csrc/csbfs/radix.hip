// Graph build by sorting: every adjacency entry becomes one 64-bit key, block
// row above, target id below (inverted, so that ascending keys give rows in
// decreasing id order), and a least-significant-digit radix sort puts all
// rows of all blocks in place at once, whatever their lengths.
//
// A pass moves every key once: tiles of kRadixTile keys are counted by digit
// (the first pass's counts are taken while the keys are made), the counts are
// scanned digit by digit, and each tile is ranked in LDS and written out in
// digit order, in runs of about 16 keys. Bound by memory: 24 bytes per key
// and pass (read twice, written once).
#include <utility>

#include "device.hpp"
#include "graph.hpp"

namespace csbfs {
namespace {

constexpr int kRadixThreads = 512;
constexpr int kRadixItems = 8;  // keys per thread
constexpr int kRadixTile = kRadixThreads * kRadixItems;
constexpr int kRadixWaves = kRadixThreads / 64;
constexpr int kDigitBits = 8, kDigits = 1 << kDigitBits;
constexpr int kScanUnroll = 16;  // rows of counts in flight per thread

struct KeyShape {
    uint32_t n, R;
    int32_t P, target_bits, key_bits;
};
KeyShape key_shape(int64_t n, int32_t P) {
    KeyShape s{(uint32_t)n, (uint32_t)(n / P), P, 1, 0};
    while (((int64_t)1 << s.target_bits) < n / P) ++s.target_bits;
    int rb = 1;
    while (((int64_t)1 << rb) < P * n) ++rb;
    s.key_bits = s.target_bits + rb;
    return s;
}

// Digit counts of one tile, per wave in LDS, then to hist[tile][digit].
__device__ __forceinline__ void count_digit(uint32_t *cnt, uint64_t key, int shift, int bits) {
    atomicAdd(&cnt[(key >> shift) & ((1u << bits) - 1u)], 1u);
}
__device__ __forceinline__ void store_counts(const uint32_t (*cnt)[kDigits], uint32_t *hist, int64_t tile) {
    __syncthreads();
    for (int d = threadIdx.x; d < kDigits; d += kRadixThreads) {
        uint32_t s = 0;
        for (int w = 0; w < kRadixWaves; ++w) s += cnt[w][d];
        hist[tile * kDigits + d] = s;
    }
}

// Keys 2t and 2t + 1 of tuple t, and the first digit's counts.
__global__ __launch_bounds__(kRadixThreads) void k_keys(const int64_t *src, const int64_t *dst, int64_t m, KeyShape s,
                                                        uint64_t *key, uint32_t *hist, int bits, int32_t *err) {
    __shared__ uint32_t cnt[kRadixWaves][kDigits];
    for (int k = threadIdx.x; k < kRadixWaves * kDigits; k += kRadixThreads) (&cnt[0][0])[k] = 0;
    __syncthreads();
    uint32_t *mine = cnt[threadIdx.x >> 6];
    const uint64_t top = (1ull << s.target_bits) - 1;
    const int64_t t0 = blockIdx.x * (int64_t)(kRadixTile / 2) + threadIdx.x;
    int64_t us[kRadixItems / 2], vs[kRadixItems / 2];
#pragma unroll
    for (int k = 0; k < kRadixItems / 2; ++k) {
        const int64_t t = t0 + k * kRadixThreads;
        us[k] = t < m ? src[t] : 0;
        vs[k] = t < m ? dst[t] : 0;
    }
#pragma unroll
    for (int k = 0; k < kRadixItems / 2; ++k) {
        const int64_t t = t0 + k * kRadixThreads;
        if (t >= m) continue;
        uint32_t u = (uint32_t)us[k], v = (uint32_t)vs[k];
        if (us[k] < 0 || us[k] >= (int64_t)s.n || vs[k] < 0 || vs[k] >= (int64_t)s.n) {
            *err = 1;  // the build fails; the keys stay in range
            u = v = 0;
        }
        const uint32_t ou = u / s.R, ov = v / s.R, ul = u - ou * s.R, vl = v - ov * s.R;
        const uint64_t r1 = (uint64_t)(ov * s.P + ou) * s.R + ul, r2 = (uint64_t)(ou * s.P + ov) * s.R + vl;
        const uint64_t k1 = (r1 << s.target_bits) | (top - vl), k2 = (r2 << s.target_bits) | (top - ul);
        reinterpret_cast<ulonglong2 *>(key)[t] = make_ulonglong2(k1, k2);
        count_digit(mine, k1, 0, bits);
        count_digit(mine, k2, 0, bits);
    }
    store_counts(cnt, hist, blockIdx.x);
}

__global__ __launch_bounds__(kRadixThreads) void k_radix_count(const uint64_t *key, int64_t nnz, int shift, int bits,
                                                               uint32_t *hist) {
    __shared__ uint32_t cnt[kRadixWaves][kDigits];
    for (int k = threadIdx.x; k < kRadixWaves * kDigits; k += kRadixThreads) (&cnt[0][0])[k] = 0;
    __syncthreads();
    uint32_t *mine = cnt[threadIdx.x >> 6];
    const int64_t e0 = blockIdx.x * (int64_t)kRadixTile + threadIdx.x;
    uint64_t v[kRadixItems];
#pragma unroll
    for (int k = 0; k < kRadixItems; ++k) v[k] = e0 + k * kRadixThreads < nnz ? key[e0 + k * kRadixThreads] : 0;
#pragma unroll
    for (int k = 0; k < kRadixItems; ++k)
        if (e0 + k * kRadixThreads < nnz) count_digit(mine, v[k], shift, bits);
    store_counts(cnt, hist, blockIdx.x);
}

// The counts become the tiles' first places, digit-major: the sums of `per`
// tiles at a time, their scan (with the digits' totals), and the tiles again.
// Thread = digit, so every access is a whole row of counts.
__global__ __launch_bounds__(kDigits) void k_radix_sum(const uint32_t *hist, int64_t ntiles, int64_t per,
                                                       uint32_t *part) {
    const int64_t t0 = blockIdx.x * per, t1 = t0 + per < ntiles ? t0 + per : ntiles;
    uint32_t s = 0;
    for (int64_t t = t0; t < t1; t += kScanUnroll) {
        uint32_t x[kScanUnroll];
#pragma unroll
        for (int k = 0; k < kScanUnroll; ++k) x[k] = t + k < t1 ? hist[(t + k) * kDigits + threadIdx.x] : 0;
#pragma unroll
        for (int k = 0; k < kScanUnroll; ++k) s += x[k];
    }
    part[blockIdx.x * kDigits + threadIdx.x] = s;
}

__global__ __launch_bounds__(kDigits) void k_radix_scan(uint32_t *part, int64_t nchunks) {
    __shared__ uint32_t wtot[kDigits / 64];
    uint32_t s = 0;
    for (int64_t c = 0; c < nchunks; c += kScanUnroll) {
        uint32_t x[kScanUnroll];
#pragma unroll
        for (int k = 0; k < kScanUnroll; ++k) x[k] = c + k < nchunks ? part[(c + k) * kDigits + threadIdx.x] : 0;
#pragma unroll
        for (int k = 0; k < kScanUnroll; ++k) {
            if (c + k < nchunks) part[(c + k) * kDigits + threadIdx.x] = s;
            s += x[k];
        }
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const uint32_t incl = (uint32_t)wave_incl_scan_i32((int)s);
    if (lane == 63) wtot[wid] = incl;
    __syncthreads();
    uint32_t base = incl - s;
    for (int w = 0; w < wid; ++w) base += wtot[w];
    part[nchunks * kDigits + threadIdx.x] = base;  // keys of smaller digits
}

__global__ __launch_bounds__(kDigits) void k_radix_apply(uint32_t *hist, int64_t ntiles, int64_t per,
                                                         const uint32_t *part, int64_t nchunks) {
    const int64_t t0 = blockIdx.x * per, t1 = t0 + per < ntiles ? t0 + per : ntiles;
    uint32_t at = part[blockIdx.x * kDigits + threadIdx.x] + part[nchunks * kDigits + threadIdx.x];
    for (int64_t t = t0; t < t1; t += kScanUnroll) {
        uint32_t x[kScanUnroll];
#pragma unroll
        for (int k = 0; k < kScanUnroll; ++k) x[k] = t + k < t1 ? hist[(t + k) * kDigits + threadIdx.x] : 0;
#pragma unroll
        for (int k = 0; k < kScanUnroll; ++k) {
            if (t + k < t1) hist[(t + k) * kDigits + threadIdx.x] = at;
            at += x[k];
        }
    }
}

// One tile to its places. A wave ranks its kRadixItems runs of 64 keys in
// order (ballots find the lanes with the same digit, LDS holds the wave's
// counts), which keeps the pass stable.
__global__ __launch_bounds__(kRadixThreads) void k_radix_move(const uint64_t *key, int64_t nnz, int shift, int bits,
                                                              const uint32_t *hist, uint64_t *out) {
    __shared__ uint64_t sorted[kRadixTile];
    __shared__ uint16_t cnt[kRadixWaves][kDigits];
    __shared__ uint16_t local[kDigits];
    __shared__ uint32_t place[kDigits];
    __shared__ uint32_t wtot[kDigits / 64];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    for (int k = tid; k < kRadixWaves * kDigits; k += kRadixThreads) (&cnt[0][0])[k] = 0;
    const int64_t tile0 = blockIdx.x * (int64_t)kRadixTile;
    const int64_t e0 = tile0 + wid * 64 * kRadixItems + lane;
    const uint32_t mask = (1u << bits) - 1u;
    uint64_t v[kRadixItems];
    uint16_t rank[kRadixItems];
#pragma unroll
    for (int k = 0; k < kRadixItems; ++k) v[k] = e0 + 64 * k < nnz ? key[e0 + 64 * k] : 0;
    const uint32_t first = tid < kDigits ? hist[blockIdx.x * (int64_t)kDigits + tid] : 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kRadixItems; ++k) {
        const uint32_t d = (uint32_t)(v[k] >> shift) & mask;
        const bool ok = e0 + 64 * k < nnz;
        uint64_t peers = __ballot(ok);
#pragma unroll
        for (int b = 0; b < kDigitBits; ++b) {
            const uint64_t bal = __ballot((d >> b) & 1);
            peers &= (d >> b) & 1 ? bal : ~bal;
        }
        const int before = __popcll(peers & ((1ull << lane) - 1));
        const uint16_t base = cnt[wid][d];
        rank[k] = (uint16_t)(base + before);
        wave_lds_sync();
        if (ok && before == 0) cnt[wid][d] = (uint16_t)(base + __popcll(peers));
        wave_lds_sync();
    }
    __syncthreads();
    uint32_t total = 0, incl = 0;
    if (tid < kDigits) {
        for (int w = 0; w < kRadixWaves; ++w) {
            const uint16_t x = cnt[w][tid];
            cnt[w][tid] = (uint16_t)total;
            total += x;
        }
        incl = (uint32_t)wave_incl_scan_i32((int)total);
        if (lane == 63) wtot[wid] = incl;
    }
    __syncthreads();
    if (tid < kDigits) {
        uint32_t at = incl - total;
        for (int w = 0; w < wid; ++w) at += wtot[w];
        local[tid] = (uint16_t)at;
        place[tid] = first - at;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kRadixItems; ++k) {
        const uint32_t d = (uint32_t)(v[k] >> shift) & mask;
        if (e0 + 64 * k < nnz) sorted[local[d] + cnt[wid][d] + rank[k]] = v[k];
    }
    __syncthreads();
    const int count = nnz - tile0 < kRadixTile ? (int)(nnz - tile0) : kRadixTile;
    for (int i = tid; i < count; i += kRadixThreads) {
        const uint64_t x = sorted[i];
        out[place[(uint32_t)(x >> shift) & mask] + (uint32_t)i] = x;
    }
}

// Targets of the sorted keys, and the place after the last entry of every
// non-empty row (the others keep zeros); a scan of these ends gives the row
// offsets. With the rows' first places beside them a build took another 8 bytes
// of scratch per row: 192 GiB of 2^28 tuples over 3 * 2^27 vertices and 64 x 64
// blocks. Row r of the keys lies r / R (its block) slots past r; `inv` is 2^64 / R
// rounded up, which gives that quotient exactly as r * R < 2^64.
__global__ __launch_bounds__(kRadixThreads) void k_rows(const uint64_t *key, int64_t nnz, int target_bits, uint64_t inv,
                                                        uint32_t *col, int32_t *row_end) {
    const uint64_t top = (1ull << target_bits) - 1;
    for (int64_t i = blockIdx.x * (int64_t)kRadixThreads + threadIdx.x; i < nnz;
         i += (int64_t)gridDim.x * kRadixThreads) {
        const uint64_t k = key[i], row = k >> target_bits;
        col[i] = (uint32_t)(top - (k & top));
        if (i == nnz - 1 || (key[i + 1] >> target_bits) != row)
            row_end[row + __umul64hi(row, inv)] = (int32_t)(uint32_t)(i + 1);
    }
}

// Tiles per workgroup of the counts' scan: about 128 workgroups, of 16 to 512
// tiles.
int64_t radix_chunks(int64_t ntiles, int64_t *per) {
    const int64_t p = (ntiles + 127) / 128;
    *per = p < 16 ? 16 : p > 512 ? 512 : p;
    return (ntiles + *per - 1) / *per;
}

}  // namespace

int64_t radix_scratch_bytes(int64_t nnz) {
    const int64_t ntiles = (nnz + kRadixTile - 1) / kRadixTile;
    int64_t per;
    const int64_t nchunks = radix_chunks(ntiles, &per);
    return align_up(8 * nnz) + align_up(4 * kDigits * ntiles) + align_up(4 * kDigits * (nchunks + 1));
}

int sort_entries(const int64_t *src, const int64_t *dst, int64_t n_tuples, int64_t n, int32_t P, void *scratch,
                 void *keys, uint32_t *col, int32_t *row_end, int32_t *err, hipStream_t st) {
    const int64_t nnz = 2 * n_tuples;
    if (nnz == 0) return CSBFS_OK;
    const KeyShape s = key_shape(n, P);
    const int64_t ntiles = (nnz + kRadixTile - 1) / kRadixTile;
    int64_t per;
    const int64_t nchunks = radix_chunks(ntiles, &per);
    char *at = (char *)scratch;
    uint32_t *hist = (uint32_t *)(at + align_up(8 * nnz));
    uint32_t *part = (uint32_t *)((char *)hist + align_up(4 * kDigits * ntiles));
    const int passes = (s.key_bits + kDigitBits - 1) / kDigitBits;
    // the last pass ends in the scratch, as col may lie where `keys` does
    uint64_t *from = (uint64_t *)(passes & 1 ? keys : scratch), *to = (uint64_t *)(passes & 1 ? scratch : keys);
    for (int q = 0; q < passes; ++q) {
        const int shift = q * kDigitBits;
        const int bits = s.key_bits - shift < kDigitBits ? s.key_bits - shift : kDigitBits;
        if (q == 0)
            hipLaunchKernelGGL(k_keys, dim3((unsigned)ntiles), dim3(kRadixThreads), 0, st, src, dst, n_tuples, s, from,
                               hist, bits, err);
        else
            hipLaunchKernelGGL(k_radix_count, dim3((unsigned)ntiles), dim3(kRadixThreads), 0, st,
                               (const uint64_t *)from, nnz, shift, bits, hist);
        CSBFS_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_radix_sum, dim3((unsigned)nchunks), dim3(kDigits), 0, st, (const uint32_t *)hist, ntiles,
                           per, part);
        CSBFS_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_radix_scan, dim3(1), dim3(kDigits), 0, st, part, nchunks);
        CSBFS_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_radix_apply, dim3((unsigned)nchunks), dim3(kDigits), 0, st, hist, ntiles, per,
                           (const uint32_t *)part, nchunks);
        CSBFS_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_radix_move, dim3((unsigned)ntiles), dim3(kRadixThreads), 0, st, (const uint64_t *)from,
                           nnz, shift, bits, (const uint32_t *)hist, to);
        CSBFS_HIP(hipGetLastError());
        std::swap(from, to);
    }
    hipLaunchKernelGGL(k_rows, dim3(grid_for(nnz, kRadixThreads, 65536)), dim3(kRadixThreads), 0, st,
                       (const uint64_t *)from, nnz, s.target_bits, ~0ull / s.R + 1, col, row_end);
    CSBFS_HIP(hipGetLastError());
    return CSBFS_OK;
}

}  // namespace csbfs
