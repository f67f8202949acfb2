// Version, status strings, the thread-local last-error message, and the device
// blocks of graphs and builds.
#include <mutex>
#include <string>
#include <vector>

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

struct Kept {
    int device;
    DeviceBlock b;
};
std::mutex g_kept_mu;
std::vector<Kept> g_kept;  // oldest first
size_t g_kept_bytes = 0;

// Gives back the oldest kept blocks until at most `limit` bytes are kept (the
// lock is held).
void trim(size_t limit) {
    size_t k = 0;
    while (k < g_kept.size() && g_kept_bytes > limit) {
        (void)hipFree(g_kept[k].b.p);
        g_kept_bytes -= g_kept[k].b.bytes;
        ++k;
    }
    g_kept.erase(g_kept.begin(), g_kept.begin() + (long)k);
}

}  // namespace

void device_trim() {
    std::lock_guard<std::mutex> lk(g_kept_mu);
    trim(0);
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
        size_t best = g_kept.size();
        for (size_t k = 0; k < g_kept.size(); ++k) {
            const Kept &x = g_kept[k];
            if (x.device == dev && x.b.bytes >= bytes && x.b.bytes <= bytes + bytes / 4 &&
                (best == g_kept.size() || x.b.bytes < g_kept[best].b.bytes))
                best = k;
        }
        if (best < g_kept.size()) {
            *out = g_kept[best].b;
            g_kept_bytes -= out->bytes;
            g_kept.erase(g_kept.begin() + (long)best);
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
    trim(kKeptBytes - b.bytes);
    g_kept.push_back(Kept{dev, b});
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
