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
    uint64_t token;    // where its last work was enqueued; 0: none is pending
    uint64_t serial;   // of its release
};

// One device's blocks.  Held while a context lives on the device; with the last
// one gone the kept blocks are freed and later ones are not kept.  The lock is
// never held through a call that may wait for the device.
struct Pool {
    std::mutex mu;
    int contexts = 0;
    size_t kept = 0;
    uint64_t releases = 0;
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

// Frees the idle blocks; false: there were none.
bool drop_idle(Pool &p) {
    std::multimap<size_t, Block> gone;
    {
        std::lock_guard<std::mutex> lk(p.mu);
        gone.swap(p.idle);
        p.kept = 0;
    }
    for (auto &b : gone) (void)hipFree(b.second.ptr);
    return !gone.empty();
}

// hipMalloc with the idle blocks as a reserve.
hipError_t card_malloc(Pool *p, void **ptr, size_t bytes) {
    hipError_t e = hipMalloc(ptr, bytes);
    if (e == hipErrorOutOfMemory && p && drop_idle(*p)) {
        (void)hipGetLastError();
        e = hipMalloc(ptr, bytes);
    }
    // (the caller reports it; the next launch is checked by the last error)
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}

}  // namespace

void fail_allocation(int64_t n) { g_fail_countdown.store(n > 0 ? n : 0); }

hipError_t dev_malloc(void **ptr, size_t bytes) {
    if (injected_failure()) {
        if (ptr) *ptr = nullptr;
        return hipErrorOutOfMemory;
    }
    return card_malloc(current_pool(), ptr, bytes);
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

// token: of the context that goes, whose stream is idle (0: that is not known).
void pool_remove_context(uint64_t token) {
    Pool *p = current_pool();
    if (!p) return;
    bool last;
    {
        std::lock_guard<std::mutex> lk(p->mu);
        last = --p->contexts == 0;
        for (auto &b : p->idle)
            if (b.second.token == token) b.second.token = 0;
    }
    if (last) (void)drop_idle(*p);
}

hipError_t pool_device_synchronize() {
    Pool *p = current_pool();
    uint64_t before = 0;
    if (p) {
        std::lock_guard<std::mutex> lk(p->mu);
        before = p->releases;
    }
    const hipError_t e = hipDeviceSynchronize();
    if (p && e == hipSuccess) {
        std::lock_guard<std::mutex> lk(p->mu);
        for (auto &b : p->idle)
            if (b.second.serial <= before) b.second.token = 0;
    }
    return e;
}

hipError_t pool_malloc(void **ptr, size_t bytes, uint64_t token) {
    *ptr = nullptr;
    if (injected_failure()) return hipErrorOutOfMemory;
    Pool *p = current_pool();
    if (!p) return hipMalloc(ptr, bytes);
    const size_t size = rounded(bytes);
    {
        // the smallest kept block that fits with at most a quarter to spare and has
        // no work pending in another stream (a fresh one costs less than waiting)
        std::lock_guard<std::mutex> lk(p->mu);
        for (auto it = p->idle.lower_bound(size); it != p->idle.end() && it->first <= size + size / 4; ++it) {
            const Block b = it->second;
            if (b.token != token && b.token != 0) continue;
            p->idle.erase(it);
            p->kept -= b.bytes;
            p->live[b.ptr] = b.bytes;
            *ptr = b.ptr;
            return hipSuccess;
        }
    }
    const hipError_t e = card_malloc(p, ptr, size);
    if (e == hipSuccess) {
        std::lock_guard<std::mutex> lk(p->mu);
        p->live[*ptr] = size;
    }
    return e;
}

void pool_free(void *ptr, uint64_t token) {
    if (!ptr) return;
    Pool *p = current_pool();
    if (p) {
        std::lock_guard<std::mutex> lk(p->mu);
        auto it = p->live.find(ptr);
        const size_t bytes = it == p->live.end() ? 0 : it->second;
        if (it != p->live.end()) p->live.erase(it);
        if (bytes != 0 && bytes <= kKeepBlock && p->contexts > 0 && p->kept + bytes <= kKeepBytes) {
            p->idle.insert({bytes, Block{ptr, bytes, token, ++p->releases}});
            p->kept += bytes;
            return;
        }
    }
    (void)hipFree(ptr);
}

}  // namespace sal
