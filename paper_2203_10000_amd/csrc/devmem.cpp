// Device allocations.  dev_malloc is hipMalloc with the tests' fault injection and
// the kept blocks as a reserve; pool_malloc / pool_free keep blocks that a mesh or a call has finished with for
// the next one: hipMalloc and hipFree cost 0.1 to 0.2 ms each, hipFree waits for
// the device, and a mesh with its post-processing makes some hundred of each
// (24 of the 45 ms of conforming, smoothing and inflating 1.5 million leaves).
#include <atomic>
#include <map>
#include <mutex>
#include <unordered_map>

#include "runtime.h"

namespace sal {
namespace {

std::atomic<int64_t> g_fail_countdown{0};   // allocations left before the one that fails; 0 = off

bool injected_failure() {
    int64_t c = g_fail_countdown.load();
    while (c > 0 && !g_fail_countdown.compare_exchange_weak(c, c - 1)) {
    }
    return c == 1;
}

// Kept per device at most, and no block above the second bound: under 1 % of the
// card, and what is larger costs more to fill than to allocate.
constexpr size_t kKeepBytes = (size_t)2 << 30, kKeepBlock = (size_t)512 << 20;

struct Block {
    void *ptr;
    size_t bytes;
    uint64_t token;   // where its last work was enqueued; 0: none is pending
};

// One device's blocks.  Held while a context lives on the device; with the last
// one gone the kept blocks are freed and later ones are not kept.
struct Pool {
    std::mutex mu;
    int contexts = 0;
    size_t kept = 0;
    std::multimap<size_t, Block> idle;
    std::unordered_map<void *, size_t> live;   // blocks handed out
};

constexpr int kMaxDevices = 64;
Pool g_pool[kMaxDevices];

Pool *current_pool() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    return &g_pool[dev];
}

// Sizes in steps of an eighth of a power of two, so that blocks fit again.
size_t rounded(size_t bytes) {
    size_t step = 512;
    while (step * 8 < bytes) step *= 2;
    return (bytes + step - 1) / step * step;
}

void drop_idle(Pool &p) {
    for (auto &b : p.idle) (void)hipFree(b.second.ptr);
    p.idle.clear();
    p.kept = 0;
}

}  // namespace

void fail_allocation(int64_t n) { g_fail_countdown.store(n > 0 ? n : 0); }

hipError_t dev_malloc(void **ptr, size_t bytes) {
    if (injected_failure()) {
        if (ptr) *ptr = nullptr;
        return hipErrorOutOfMemory;
    }
    const hipError_t e = hipMalloc(ptr, bytes);
    Pool *p = e == hipErrorOutOfMemory ? current_pool() : nullptr;
    if (!p) return e;
    std::lock_guard<std::mutex> lk(p->mu);
    if (p->idle.empty()) return e;
    (void)hipGetLastError();
    drop_idle(*p);
    return hipMalloc(ptr, bytes);
}

uint64_t new_stream_token() {
    static std::atomic<uint64_t> next{1};
    return next++;
}

void pool_add_context() {
    Pool *p = current_pool();
    if (!p) return;
    std::lock_guard<std::mutex> lk(p->mu);
    ++p->contexts;
}

void pool_remove_context() {
    Pool *p = current_pool();
    if (!p) return;
    std::lock_guard<std::mutex> lk(p->mu);
    if (--p->contexts == 0) drop_idle(*p);
}

hipError_t pool_malloc(void **ptr, size_t bytes, uint64_t token) {
    *ptr = nullptr;
    if (injected_failure()) return hipErrorOutOfMemory;
    Pool *p = current_pool();
    if (!p) return hipMalloc(ptr, bytes);
    const size_t size = rounded(bytes);
    std::lock_guard<std::mutex> lk(p->mu);
    // the smallest kept block that fits with at most a quarter to spare; of
    // those of its size, one whose last work precedes the caller's in its stream
    auto best = p->idle.end();
    for (auto it = p->idle.lower_bound(size); it != p->idle.end() && it->first <= size + size / 4; ++it) {
        if (best != p->idle.end() && it->first != best->first) break;
        best = it;
        if (it->second.token == token || it->second.token == 0) break;
    }
    if (best != p->idle.end()) {
        const Block b = best->second;
        if (b.token != token && b.token != 0) {
            const hipError_t e = hipDeviceSynchronize();
            if (e != hipSuccess) return e;
            for (auto &i : p->idle) i.second.token = 0;
        }
        p->idle.erase(best);
        p->kept -= b.bytes;
        p->live[b.ptr] = b.bytes;
        *ptr = b.ptr;
        return hipSuccess;
    }
    hipError_t e = hipMalloc(ptr, size);
    if (e == hipErrorOutOfMemory && !p->idle.empty()) {
        (void)hipGetLastError();
        drop_idle(*p);
        e = hipMalloc(ptr, size);
    }
    if (e == hipSuccess) p->live[*ptr] = size;
    return e;
}

void pool_free(void *ptr, uint64_t token) {
    if (!ptr) return;
    Pool *p = current_pool();
    if (!p) {
        (void)hipFree(ptr);
        return;
    }
    std::lock_guard<std::mutex> lk(p->mu);
    auto it = p->live.find(ptr);
    const size_t bytes = it == p->live.end() ? 0 : it->second;
    if (it != p->live.end()) p->live.erase(it);
    if (bytes == 0 || bytes > kKeepBlock || p->contexts == 0 || p->kept + bytes > kKeepBytes) {
        (void)hipFree(ptr);
        return;
    }
    p->idle.insert({bytes, Block{ptr, bytes, token}});
    p->kept += bytes;
}

}  // namespace sal
