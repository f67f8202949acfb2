// Version, status strings, the thread-local last-error message, and the device
// blocks of graphs and builds.
#include <algorithm>
#include <mutex>
#include <string>

#include "common.hpp"

namespace csbfs {

namespace {
thread_local std::string g_last_error;
}

void set_error(const std::string &msg) { g_last_error = msg; }

int fail(int status, const std::string &msg) {
    g_last_error = msg;
    return status;
}

int hip_fail(hipError_t err, const char *what, const char *file, int line) {
    g_last_error = std::string(what) + " failed: " + hipGetErrorString(err) + " (" + file + ":" +
                   std::to_string(line) + ")";
    return CSBFS_EHIP;
}

namespace {

// Kept blocks, oldest first. A fixed array: giving a block back must not
// allocate, as no exception may leave csbfs_graph_free.
struct Kept {
    int device;
    DeviceBlock b;
};
constexpr int kKeptMax = 64;
std::mutex g_kept_mu;
Kept g_kept[kKeptMax];
int g_kept_count = 0;
size_t g_kept_bytes = 0;

// Takes entry k out (the lock is held).
DeviceBlock take_out(int k) {
    const DeviceBlock b = g_kept[k].b;
    g_kept_bytes -= b.bytes;
    std::copy(g_kept + k + 1, g_kept + g_kept_count, g_kept + k);
    --g_kept_count;
    return b;
}

// Gives back the oldest kept blocks until at most `limit` bytes in `count`
// blocks are kept (the lock is held).
void trim(size_t limit, int count) {
    while (g_kept_bytes > limit || g_kept_count > count) (void)hipFree(take_out(0).p);
}

}  // namespace

void device_trim() {
    std::lock_guard<std::mutex> lk(g_kept_mu);
    trim(0, 0);
}

int device_malloc(void **p, size_t bytes) {
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        device_trim();
        e = hipMalloc(p, bytes);
    }
    if (e != hipSuccess) {
        *p = nullptr;
        (void)hipGetLastError();
        return hip_fail(e, "hipMalloc", __FILE__, __LINE__);
    }
    return CSBFS_OK;
}

int device_take(size_t bytes, DeviceBlock *out) {
    int dev = -1;
    CSBFS_HIP(hipGetDevice(&dev));
    {
        std::lock_guard<std::mutex> lk(g_kept_mu);
        int best = -1;
        for (int k = 0; k < g_kept_count; ++k) {
            const Kept &x = g_kept[k];
            if (x.device == dev && x.b.bytes >= bytes && x.b.bytes <= bytes + bytes / 4 &&
                (best < 0 || x.b.bytes < g_kept[best].b.bytes))
                best = k;
        }
        if (best >= 0) {
            *out = take_out(best);
            return CSBFS_OK;
        }
    }
    const int rc = device_malloc(&out->p, bytes);
    out->bytes = rc == CSBFS_OK ? bytes : 0;
    return rc;
}

void device_give(const DeviceBlock &b) {
    int dev = -1;
    if (b.bytes > kKeptBytes || hipGetDevice(&dev) != hipSuccess) {
        (void)hipFree(b.p);
        return;
    }
    std::lock_guard<std::mutex> lk(g_kept_mu);
    trim(kKeptBytes - b.bytes, kKeptMax - 1);
    g_kept[g_kept_count++] = Kept{dev, b};
    g_kept_bytes += b.bytes;
}

void device_release(int device, const DeviceBlock &b) {
    int dev = -1;
    const bool other = hipGetDevice(&dev) == hipSuccess && dev != device;
    if (other) (void)hipSetDevice(device);
    // a failed wait leaves the block to hipFree, which waits by itself
    if (hipDeviceSynchronize() == hipSuccess)
        device_give(b);
    else
        (void)hipFree(b.p);
    if (other) (void)hipSetDevice(dev);
}

}  // namespace csbfs

extern "C" int csbfs_version(void) { return CSBFS_VERSION; }

extern "C" int csbfs_trim(void) {
    csbfs::device_trim();
    return CSBFS_OK;
}

extern "C" const char *csbfs_strerror(int status) {
    switch (status) {
        case CSBFS_OK: return "ok";
        case CSBFS_EINVAL: return "invalid argument";
        case CSBFS_ERANGE: return "value out of range";
        case CSBFS_ENOSPACE: return "buffer or workspace too small";
        case CSBFS_EHIP: return "HIP runtime error";
        case CSBFS_EOVERFLOW: return "sub-block too large";
        case CSBFS_ECORRUPT: return "corrupt compressed stream";
        default: return "unknown status";
    }
}

extern "C" const char *csbfs_last_error(void) { return csbfs::g_last_error.c_str(); }
