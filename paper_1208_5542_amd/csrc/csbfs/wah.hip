// WAH-64 sieve + compress and decompress kernels (Sec. IV, Table 3; Alg. 3
// sieve, Compress and Uncompress), batched over the p * p streams of a level;
// the device code is in wah_device.hpp.
#include <algorithm>
#include <mutex>

#include "wah_device.hpp"

namespace csbfs {
namespace {

__global__ __launch_bounds__(kEncThreads) void wah_encode_kernel(WahBatch b) {
    PlainWords h;
    encode_segment<kEncGpt>(b, h, blockIdx.y, blockIdx.x == 0);
}

// A stream from elsewhere, in one pass over it (a pass that summed every
// chunk's groups first, two clears and a copy of the length from the host made
// it 50 us for the smallest streams, now 30 with the caller's read of the
// status; 2^28 bits 90 us, now 75). Chunks are taken in ticket order, so every awaited
// one runs; a chunk publishes its group total (state 1), then the total
// through it (state 2), each in one 64-bit word whose top two bits are the
// state. Totals above G (an invalid stream) are cut off at G + 1.
struct DecodeArgs {
    const uint64_t *words;
    int64_t nw, nbits, nchunk;
    uint64_t *dst;
    int32_t *status;
    unsigned long long *look;  // [nchunk], zero (unused with one chunk)
    uint32_t *ticket;          // zero
};
constexpr int kDecWide = 2;
constexpr int64_t kDecWideWords = 512 * kDecChunk;
constexpr uint64_t kDlAgg = 1ull << 62, kDlInc = 2ull << 62, kDlValue = kDlAgg - 1;

__device__ long long dec_prefix(const DecodeArgs &a, int64_t c) {
    const int lane = threadIdx.x & 63;
    long long sum = 0;
    for (int64_t k0 = c - 1;; k0 -= 64) {
        const int64_t k = k0 - lane;
        uint64_t v = k >= 0 ? __hip_atomic_load(&a.look[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : kDlInc;
        uint32_t polls = 0;
        while (__ballot((v >> 62) == 0)) {
            if (++polls == kLbSpinLimit) {  // a lost publication: flag the stream, stop waiting
                if (lane == 0) *a.status = 1;
                if ((v >> 62) == 0) v = kDlInc;
                break;
            }
            if ((v >> 62) == 0) v = __hip_atomic_load(&a.look[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        const uint64_t inc = __ballot((v >> 62) == 2);
        const int stop = inc ? __ffsll((unsigned long long)inc) - 1 : 63;
        sum += (long long)readlane64((uint64_t)wave_incl_scan_i64(lane <= stop ? (long long)(v & kDlValue) : 0), 63);
        if (inc) return sum;
    }
}

template <int kT>
__global__ __launch_bounds__(kDecThreads) void wah_decode_kernel(DecodeArgs a) {
    __shared__ int64_t sh_c;
    __shared__ long long sh_before;
    const int64_t G = a.nbits / kGroupBits, r = a.nbits - G * kGroupBits;
    if (threadIdx.x == 0) {
        sh_c = a.nchunk > 1 ? (int64_t)atomicAdd(a.ticket, 1u) : 0;
        if (a.nchunk <= 1) *a.status = 0;  // else cleared by the launch before
    }
    __syncthreads();
    const int64_t c = sh_c;
    if (c == 0 && threadIdx.x == 0) dec_tail(a.words, a.nw, a.nw, a.nbits, G, r, a.dst, a.status);
    if (c * kT * kDecChunk >= a.nw - (r > 0 ? 1 : 0)) return;
    dec_chunk<kT, false>(a.words, a.nw, G, r, c, a.dst, a.status, [&](long long total) -> long long {
        if (a.nchunk <= 1) return 0;
        const long long cut = G + 1;
        if (threadIdx.x < 64) {
            const long long mine = total < cut ? total : cut;
            if (threadIdx.x == 0 && c > 0)
                __hip_atomic_store(&a.look[c], (uint64_t)mine | kDlAgg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const long long before = c > 0 ? dec_prefix(a, c) : 0;
            if (threadIdx.x == 0) {
                const long long all = before + mine < cut ? before + mine : cut;
                __hip_atomic_store(&a.look[c], (uint64_t)all | kDlInc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                sh_before = before;
            }
        }
        __syncthreads();
        return sh_before;
    });
}

__global__ __launch_bounds__(kDecThreads) void wah_dec_scatter(WahBatch b) { dec_scatter_body(b); }

// Zero `words` 32-bit words (a kernel rather than a memset node, so that the
// allocation-free entry point can be captured into a HIP graph).
__global__ void zero_words_kernel(uint32_t *p, int64_t words) {
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < words;
         k += (int64_t)gridDim.x * blockDim.x)
        p[k] = 0;
}

__global__ void store_i64_kernel(int64_t *p, int64_t v) { *p = v; }
__global__ void store_i32_kernel(int32_t *p, int32_t v) { *p = v; }

__global__ void clear_decode_kernel(DecodeArgs a) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    for (int64_t k = t; k < a.nchunk; k += (int64_t)gridDim.x * blockDim.x) a.look[k] = 0;
    if (t == 0) {
        *a.ticket = 0;
        *a.status = 0;
    }
}

}  // namespace

int launch_wah_encode(const WahBatch &b, hipStream_t stream) {
    const int64_t S = batch_streams(b);
    if (b.nbits / kGroupBits > kLbField) return fail(CSBFS_EINVAL, "WAH encode: more than 2^29 - 1 groups");
    dim3 grid((unsigned)b.nseg, (unsigned)S);
    hipLaunchKernelGGL(wah_encode_kernel, grid, dim3(kEncThreads), 0, stream, b);
    CSBFS_HIP(hipGetLastError());
    return CSBFS_OK;
}

int launch_wah_decode(const WahBatch &b, hipStream_t stream) {
    const int64_t S = batch_streams(b);
    dim3 grid((unsigned)b.nchunk, (unsigned)S);
    hipLaunchKernelGGL(wah_dec_scatter, grid, dim3(kDecThreads), 0, stream, b);
    CSBFS_HIP(hipGetLastError());
    return CSBFS_OK;
}

}  // namespace csbfs

// ------------------------------------------------------------ C ABI ---

using namespace csbfs;

namespace {
constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
struct WsLayout {
    size_t look, ticket, dec_look, dec_ticket, total;  // encoder's, then decoder's look-back words and tickets
};
WsLayout ws_layout(int64_t nbits) {
    WsLayout l;
    const int64_t nseg = enc_segments(nbits);
    const int64_t nchunk = dec_chunks(nbits);
    l.look = 0;
    l.ticket = l.look + align_up(sizeof(unsigned long long) * nseg);
    l.dec_look = l.ticket + align_up(sizeof(uint32_t) * kTicketStride);
    l.dec_ticket = l.dec_look + align_up(sizeof(unsigned long long) * nchunk);
    l.total = l.dec_ticket + align_up(sizeof(uint32_t));
    return l;
}
}  // namespace

extern "C" int64_t csbfs_wah_capacity(int64_t nbits) { return nbits < 0 ? -1 : wah_cap(nbits); }

extern "C" size_t csbfs_wah_workspace_bytes(int64_t nbits) {
    return nbits < 0 ? 0 : ws_layout(nbits).total;
}

extern "C" int csbfs_wah_encode(const uint64_t *bits, const uint64_t *mask, int64_t nbits,
                                uint64_t *out, int64_t cap_words, int64_t *n_words,
                                void *workspace, size_t ws_bytes, void *stream) {
    if (nbits < 0 || !out || !n_words || !workspace || (nbits > 0 && !bits))
        return fail(CSBFS_EINVAL, "csbfs_wah_encode: null pointer or negative size");
    if (nbits / kGroupBits > (int64_t)kLbField)
        return fail(CSBFS_EINVAL, "csbfs_wah_encode: nbits above 63 * (2^29 - 1)");
    if (cap_words < wah_cap(nbits))
        return fail(CSBFS_ENOSPACE, "csbfs_wah_encode: output capacity below floor(nbits/63)+1");
    const WsLayout l = ws_layout(nbits);
    if (ws_bytes < l.total) return fail(CSBFS_ENOSPACE, "csbfs_wah_encode: workspace too small");
    char *ws = (char *)workspace;
    WahBatch b{};
    b.bits_base = bits;
    b.mask_base = mask;
    b.out_base = out;
    b.n_words = n_words;
    b.nbits = nbits;
    b.words_per_piece = (nbits + 63) / 64;
    b.cap = cap_words;
    b.P = 1;
    b.look = (unsigned long long *)(ws + l.look);
    b.ticket = (uint32_t *)(ws + l.ticket);
    b.nseg = enc_segments(nbits);
    if (nbits == 0) {
        CSBFS_HIP(hipMemsetAsync(n_words, 0, sizeof(int64_t), as_stream(stream)));
        return CSBFS_OK;
    }
    // the look-back words and tickets start at zero (the caller's workspace
    // may hold anything); one segment uses neither (up to 129024 bits: 10.5 ->
    // 8.8 us a call)
    if (b.nseg > 1) CSBFS_HIP(hipMemsetAsync(ws + l.look, 0, l.dec_look - l.look, as_stream(stream)));
    return launch_wah_encode(b, as_stream(stream));
}

// ------------------------------------------- allocation-free encoder ---
//
// Scratch of csbfs_wah_encode_noalloc: the encoder's look-back words and
// segment tickets, in a file-scope device array. Each GPU the library runs
// on holds its own copy until the process ends. Host code never passes the
// array's name to a kernel (on the host it is only a stand-in symbol): the
// device address is looked up once per device with hipGetSymbolAddress and
// that pointer is used everywhere.
namespace {
constexpr size_t kNoAllocScratchBytes = 256 * 1024;
__device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

int scratch_ptr(void **out) {
    int dev = -1;
    CSBFS_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(CSBFS_EINVAL, "csbfs_wah_encode_noalloc: device id out of range");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return hip_fail(e, "hipGetSymbolAddress(scratch)", __FILE__, __LINE__);
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return CSBFS_OK;
}
}  // namespace

extern "C" int64_t csbfs_wah_noalloc_max_bits(void) {
    // the largest nbits whose look-back words and tickets fit the scratch
    int64_t lo = 0, hi = 63 * (int64_t)kLbField;
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo + 1) / 2;
        const WsLayout l = ws_layout(mid);
        if (l.dec_look <= kNoAllocScratchBytes)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

extern "C" int csbfs_wah_encode_noalloc(const uint64_t *bits, const uint64_t *mask, int64_t nbits, uint64_t *out,
                                        int64_t cap_words, int64_t *n_words, void *stream) {
    if (nbits < 0 || !out || !n_words || (nbits > 0 && !bits))
        return fail(CSBFS_EINVAL, "csbfs_wah_encode_noalloc: null pointer or negative size");
    if (nbits > csbfs_wah_noalloc_max_bits())
        return fail(CSBFS_EINVAL, "csbfs_wah_encode_noalloc: nbits above csbfs_wah_noalloc_max_bits() (the "
                                  "encoder's scratch is a fixed 256 KiB device array)");
    if (cap_words < wah_cap(nbits))
        return fail(CSBFS_ENOSPACE, "csbfs_wah_encode_noalloc: output capacity below floor(nbits/63)+1");
    void *ptr = nullptr;
    int rc = scratch_ptr(&ptr);
    if (rc) return rc;
    hipStream_t st = as_stream(stream);
    if (nbits == 0) {
        hipLaunchKernelGGL(store_i64_kernel, dim3(1), dim3(1), 0, st, n_words, (int64_t)0);
        CSBFS_HIP(hipGetLastError());
        return CSBFS_OK;
    }
    const WsLayout l = ws_layout(nbits);
    char *ws = (char *)ptr;
    // look-back words and tickets start at zero; the previous call on this
    // device left its own there. A stream of one segment reads neither.
    const int64_t words = (int64_t)((l.dec_look - l.look) / 4);
    if (enc_segments(nbits) > 1) {
        hipLaunchKernelGGL(zero_words_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, st,
                           (uint32_t *)(ws + l.look), words);
        CSBFS_HIP(hipGetLastError());
    }
    WahBatch b{};
    b.bits_base = bits;
    b.mask_base = mask;
    b.out_base = out;
    b.n_words = n_words;
    b.nbits = nbits;
    b.words_per_piece = (nbits + 63) / 64;
    b.cap = cap_words;
    b.P = 1;
    b.look = (unsigned long long *)(ws + l.look);
    b.ticket = (uint32_t *)(ws + l.ticket);
    b.nseg = enc_segments(nbits);
    return launch_wah_encode(b, st);
}

extern "C" int csbfs_wah_decode_or(const uint64_t *words, int64_t n_words, int64_t nbits,
                                   uint64_t *dst, int32_t *status, void *workspace,
                                   size_t ws_bytes, void *stream) {
    if (nbits < 0 || n_words < 0 || !status || !workspace || (nbits > 0 && !dst) ||
        (n_words > 0 && !words))
        return fail(CSBFS_EINVAL, "csbfs_wah_decode_or: null pointer or negative size");
    if (nbits >= ((int64_t)1 << 37))
        return fail(CSBFS_EINVAL, "csbfs_wah_decode_or: nbits too large");
    const WsLayout l = ws_layout(nbits);
    if (ws_bytes < l.total) return fail(CSBFS_ENOSPACE, "csbfs_wah_decode_or: workspace too small");
    hipStream_t st = as_stream(stream);
    // a length no stream of nbits bits has (and an empty stream of none, which
    // is valid)
    if (n_words > wah_cap(nbits) || nbits == 0) {
        hipLaunchKernelGGL(store_i32_kernel, dim3(1), dim3(1), 0, st, status, n_words != 0 ? 1 : 0);
        CSBFS_HIP(hipGetLastError());
        return CSBFS_OK;
    }
    char *ws = (char *)workspace;
    // kDecChunk words per workgroup while that many workgroups fit the GPU, else
    // twice that (a ticket costs 5 ns, in sequence: 2^28 bits took 67 us with
    // 4158 of them and 47 with half; four or eight times were no faster)
    const int64_t per = n_words <= kDecWideWords ? kDecChunk : kDecWide * kDecChunk;
    DecodeArgs a{words, n_words, nbits, std::max<int64_t>((n_words + per - 1) / per, 1), dst, status,
                 (unsigned long long *)(ws + l.dec_look), (uint32_t *)(ws + l.dec_ticket)};
    if (a.nchunk > 1) {
        hipLaunchKernelGGL(clear_decode_kernel, dim3(grid_for(a.nchunk, 256, 1024)), dim3(256), 0, st, a);
        CSBFS_HIP(hipGetLastError());
    }
    if (per == kDecChunk)
        hipLaunchKernelGGL(wah_decode_kernel<1>, dim3((unsigned)a.nchunk), dim3(kDecThreads), 0, st, a);
    else
        hipLaunchKernelGGL(wah_decode_kernel<kDecWide>, dim3((unsigned)a.nchunk), dim3(kDecThreads), 0, st, a);
    CSBFS_HIP(hipGetLastError());
    return CSBFS_OK;
}
