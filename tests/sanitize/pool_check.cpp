// The pool of device blocks (api.hip) on the CPU: what is kept and what is given
// back, memory that runs out, blocks of two devices, a host allocator that
// fails, and threads. Blocks are stub memory whose size is counted, not held.
#include <atomic>
#include <cstdio>
#include <map>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

#include "api.hip"

size_t stub_capacity = size_t(8) << 30, stub_used = 0, stub_calls = 0;
thread_local int stub_device = 0;

static std::mutex mu;
static std::map<void *, size_t> *live = new std::map<void *, size_t>;
static std::atomic<bool> no_memory{false};

void *operator new(size_t n) {
    void *p = no_memory ? nullptr : std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

hipError_t hipMalloc(void **p, size_t bytes) {
    std::lock_guard<std::mutex> lk(mu);
    ++stub_calls;
    if (bytes > stub_capacity - stub_used) return hipErrorOutOfMemory;
    *p = std::malloc(1);
    (*live)[*p] = bytes;
    stub_used += bytes;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    std::lock_guard<std::mutex> lk(mu);
    auto it = live->find(p);
    if (it == live->end()) std::abort();  // freed twice, or never allocated
    stub_used -= it->second;
    live->erase(it);
    std::free(p);
    return hipSuccess;
}

using csbfs::DeviceBlock;
#define CHECK(x)                                                \
    do {                                                        \
        if (!(x)) {                                             \
            std::printf("line %d: %s\n", __LINE__, #x);         \
            return 1;                                           \
        }                                                       \
    } while (0)

static DeviceBlock take(size_t bytes) {
    DeviceBlock b;
    return csbfs::device_take(bytes, &b) == CSBFS_OK ? b : DeviceBlock{};
}

int main() {
    const size_t G = size_t(1) << 30;
    // a block serves a taker of its size or up to a fifth less, and no other
    DeviceBlock a = take(1000);
    csbfs::device_give(a);
    CHECK(stub_used == 1000);
    DeviceBlock b = take(800), c = take(800);
    CHECK(b.p == a.p && b.bytes == 1000 && c.p != a.p && c.bytes == 800);
    csbfs::device_give(b);
    CHECK(take(799).p != a.p && take(1001).p != a.p);
    // nor one of another device; a release comes back to the block's own
    stub_device = 1;
    CHECK(take(1000).p != a.p);
    csbfs::device_release(0, c);
    CHECK(stub_device == 1);
    stub_device = 0;
    CHECK(take(800).p == c.p);
    csbfs::device_trim();
    CHECK(stub_used == 799 + 1001 + 1000 + 800);
    const size_t used = stub_used;
    // at most kKeptBytes are kept, the oldest go first; larger ones never are
    DeviceBlock x = take(G), y = take(G), z = take(G), w = take(3 * G);
    for (const DeviceBlock &q : {x, y, z, w}) csbfs::device_give(q);
    CHECK(stub_used == used + 2 * G);
    CHECK(take(G).p == y.p);
    // memory that runs out brings the kept ones back
    CHECK(take(stub_capacity - used - G).p != nullptr && stub_used == stub_capacity);
    CHECK(take(1).p == nullptr);
    stub_capacity += 16 * G;
    // many small blocks: the number kept is bounded too
    const size_t base = stub_used;
    std::vector<DeviceBlock> many;
    for (int k = 0; k < 500; ++k) many.push_back(take(1000 * (k + 1)));
    // and none of it may throw where the host has no memory
    no_memory = true;
    bool threw = false;
    try {
        for (const DeviceBlock &q : many) csbfs::device_release(0, q);
    } catch (...) {
        threw = true;
    }
    no_memory = false;
    CHECK(!threw);
    CHECK(stub_used > base && stub_used - base <= size_t(64) * 500000);
    csbfs::device_trim();
    CHECK(stub_used == base);
    // threads
    std::vector<std::thread> ts;
    for (int t = 0; t < 4; ++t)
        ts.emplace_back([t] {
            stub_device = t & 1;
            for (int k = 0; k < 2000; ++k) {
                DeviceBlock q = take(100 + 10 * ((k * 7 + t) % 9)), r = take(100);
                csbfs::device_give(q);
                if (k % 64 == 0) csbfs::device_trim();
                csbfs::device_release(t & 1, r);
            }
        });
    for (auto &t : ts) t.join();
    csbfs::device_trim();
    CHECK(stub_used == base);
    for (auto &q : *live) std::free(q.first);
    delete live;
    std::printf("ok\n");
    return 0;
}
