// Runs host parts of libsal's runtime under AddressSanitizer and
// UndefinedBehaviorSanitizer.  argv[1] names the check (argv[2]: a file to write); exit status 0 when it
// holds, a message and 1 when it does not.
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <future>
#include <map>
#include <mutex>
#include <thread>
#include <vector>

#include "runtime.h"
#include "tune_cache.h"

// A card of kCard bytes in place of the device.
namespace {
constexpr size_t kCard = (size_t)1 << 30;
std::mutex card_mu;
std::map<void *, size_t> card;
size_t card_used = 0;
constexpr size_t kSlow = 12288;          // an allocation of this size waits for `go`
std::promise<void> slow_started, go;
std::function<void()> during_sync;
int syncs = 0;
hipError_t last_error = hipSuccess;
}  // namespace

extern "C" {
hipError_t hipMalloc(void **ptr, size_t bytes) {
    if (bytes == kSlow) {
        slow_started.set_value();
        go.get_future().wait();
    }
    std::lock_guard<std::mutex> lk(card_mu);
    *ptr = nullptr;
    if (card_used + bytes > kCard) return last_error = hipErrorOutOfMemory;
    *ptr = std::malloc(1);
    card[*ptr] = bytes;
    card_used += bytes;
    return hipSuccess;
}
hipError_t hipFree(void *ptr) {
    std::lock_guard<std::mutex> lk(card_mu);
    card_used -= card.at(ptr);
    card.erase(ptr);
    std::free(ptr);
    return hipSuccess;
}
hipError_t hipGetDevice(int *dev) { *dev = 0; return hipSuccess; }
hipError_t hipDeviceSynchronize() {
    ++syncs;
    if (during_sync) during_sync();
    return hipSuccess;
}
hipError_t hipGetLastError() {
    const hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}
}

namespace {

#define CHECK(what)                                              \
    do {                                                         \
        if (!(what)) {                                           \
            std::printf("line %d: %s\n", __LINE__, #what);       \
            return 1;                                            \
        }                                                        \
    } while (0)

// Idle blocks are given back when an allocation of either kind needs the memory; one
// that fails all the same leaves no error behind.
int reserve() {
    sal::pool_add_context();
    const uint64_t t = sal::new_stream_token();
    void *a = nullptr, *b = nullptr;
    CHECK(sal::pool_malloc(&a, kCard * 3 / 8, t) == hipSuccess);
    sal::pool_free(a, t);
    CHECK(card_used >= kCard * 3 / 8);   // kept
    CHECK(sal::dev_malloc(&b, kCard * 3 / 4) == hipSuccess);
    CHECK(sal::dev_malloc(&a, kCard / 2) == hipErrorOutOfMemory);   // nothing left to give
    CHECK(sal::pool_malloc(&a, kCard / 2, t) == hipErrorOutOfMemory);
    CHECK(last_error == hipSuccess);
    CHECK(hipFree(b) == hipSuccess);
    CHECK(sal::pool_malloc(&a, kCard * 3 / 8, t) == hipSuccess);
    sal::pool_free(a, t);
    CHECK(sal::pool_malloc(&b, kCard * 3 / 4, t) == hipSuccess);
    sal::pool_free(b, t);
    sal::pool_remove_context(t);
    CHECK(card_used == 0);
    return 0;
}

// A block with work pending in one stream is not waited for by another, and is that
// stream's or anyone's again once the device or its own stream is idle.
int streams() {
    for (int k = 0; k < 3; ++k) sal::pool_add_context();
    const uint64_t t = sal::new_stream_token(), u = sal::new_stream_token();
    void *a = nullptr, *b = nullptr, *c = nullptr;
    CHECK(sal::pool_malloc(&a, 4096, t) == hipSuccess && sal::pool_malloc(&c, 4096, t) == hipSuccess);
    void *const a0 = a, *const c0 = c;
    sal::pool_free(a, t);
    sal::pool_remove_context(0);   // a context goes whose stream may be at work
    CHECK(sal::pool_malloc(&b, 4096, u) == hipSuccess && b != a0 && syncs == 0);
    CHECK(sal::pool_malloc(&a, 4096, t) == hipSuccess && a == a0);
    sal::pool_free(a, t);
    // freed while the device is waited for: work may have come after the wait began
    during_sync = [&] { sal::pool_free(c0, t); };
    CHECK(sal::pool_device_synchronize() == hipSuccess);
    void *d = nullptr, *e = nullptr;
    CHECK(sal::pool_malloc(&d, 4096, u) == hipSuccess && d == a0);
    CHECK(sal::pool_malloc(&e, 4096, u) == hipSuccess && e != c0);
    sal::pool_remove_context(t);
    CHECK(sal::pool_malloc(&c, 4096, u) == hipSuccess && c == c0);
    for (void *p : {b, c, d, e}) sal::pool_free(p, u);
    sal::pool_remove_context(u);
    CHECK(card_used == 0 && syncs == 1);
    return 0;
}

// While one thread's allocation waits, another's goes on.
int threads() {
    sal::pool_add_context();
    const uint64_t t = sal::new_stream_token(), u = sal::new_stream_token();
    void *a = nullptr;
    CHECK(sal::pool_malloc(&a, 4096, t) == hipSuccess);
    sal::pool_free(a, t);
    void *slow = nullptr;
    std::thread waits([&] { (void)sal::pool_malloc(&slow, kSlow, u); });
    slow_started.get_future().wait();
    std::promise<void> done;
    std::future<void> other = done.get_future();
    std::thread goes([&] {
        void *p = nullptr;
        (void)sal::pool_malloc(&p, 4096, t);
        sal::pool_free(p, t);
        done.set_value();
    });
    const bool went = other.wait_for(std::chrono::seconds(5)) == std::future_status::ready;
    go.set_value();
    waits.join();
    goes.join();
    CHECK(went);
    sal::pool_free(slow, u);
    sal::pool_remove_context(u);
    CHECK(card_used == 0);
    return 0;
}

// Scratch sized for n points holds what a call on any m <= n of them uses.
int scratch() {
    std::vector<int64_t> sizes;
    for (int64_t step = 1; step <= ((int64_t)1 << 30); step *= 2)
        for (const int64_t d : {-1, 0, 1})
            for (const int64_t k : {1, 3})
                if (k * step + d > 0) sizes.push_back(k * step + d);
    for (const int64_t n : {(int64_t)257250, (int64_t)282048, (int64_t)300000}) sizes.push_back(n);
    for (const int64_t n : sizes)
        for (const int64_t m : sizes) {
            if (m > n) continue;
            const sal::ScratchSize z = sal::label_scratch_size(n, 5), y = sal::label_scratch_size(m, 5);
            const int64_t c = m < sal::kChunkPoints ? m : sal::kChunkPoints;
            const int64_t tiles = m > sal::kPointFormMax ? sal::order_tiles(c) : 0;   // written by the order
            if (y.points > z.points || y.tiles > z.tiles || y.insts > z.insts || y.spans > z.spans ||
                y.pairs > z.pairs || tiles > z.tiles) {
                std::printf("scratch for %lld points has %lld tiles, %lld points use %lld\n", (long long)n,
                            (long long)z.tiles, (long long)m, (long long)tiles);
                return 1;
            }
        }
    return 0;
}

// Many instances of a batch between the bounds leave the point form together.
int batch() {
    using sal::batch_point_max;
    CHECK(batch_point_max({}) == sal::kBatchPointMax);
    CHECK(batch_point_max({8192, 8192, 400000}) == sal::kBatchPointMax);
    CHECK(batch_point_max(std::vector<int64_t>(256, 8000)) == sal::kBatchCrowdMin);
    CHECK(batch_point_max(std::vector<int64_t>(4096, 2048)) == sal::kBatchPointMax);
    CHECK(batch_point_max(std::vector<int64_t>(8, 8192)) == sal::kBatchCrowdMin);
    CHECK(batch_point_max({8192, 8192, 8192, 8192, 8192, 8192, 8192, 8191}) == sal::kBatchPointMax);
    return 0;
}

// The tuner tells apart what runs other kernels or another number of surfaces, and
// takes no entry of a file from before it did.
int tuner(const char *file) {
    const std::string arch = "gfx950";
    const auto key = [&](int64_t n, int n_surf) { return sal::tune_key(0, 1, 5000, n, n_surf, arch); };
    CHECK(key(sal::kPointFormMax, 1) != key(sal::kPointFormMax + 1, 1));
    CHECK(key(sal::kPointFormMax - 1, 1) != key(sal::kPointFormMax + 1, 1));
    CHECK(key(1000, 1) != key(1000, 20) && key(100000, 1) != key(100000, 20));
    CHECK(key(100000, 5) == key(120000, 6));
    CHECK(key((int64_t)1 << 19, 1) == key((int64_t)1 << 24, 1));
    FILE *f = std::fopen(file, "w");
    CHECK(f);
    for (int points = 0; points <= 19; ++points)
        for (const int rp : {0, 1, 2, 4})
            for (const int rb : {0, 1, 2, 4, 8})
                std::fprintf(f, "%s 0 1 12 %d %d %d 1 1\n", arch.c_str(), points, rp, rb);
    std::fclose(f);
    sal::TuneMap m;
    CHECK(sal::tune_cache_read(file, &m) && m.size() == 400);
    for (int64_t n = 1; n <= ((int64_t)1 << 20); n *= 2)
        for (const int n_surf : {1, 2, 4, 16}) CHECK(m.count(key(n, n_surf)) == 0);
    m = {{key(1000, 20), {1, 8}}};
    CHECK(sal::tune_cache_write(file, m) && sal::tune_cache_read(file, &m) && m.size() == 1);
    CHECK(m.at(key(1000, 20)) == std::make_pair(1, 8));
    return 0;
}

}  // namespace

int main(int argc, char **argv) {
    if (argc == 3 && !std::strcmp(argv[1], "tuner")) return tuner(argv[2]);
    if (argc != 2) return 2;
    if (!std::strcmp(argv[1], "scratch")) return scratch();
    if (!std::strcmp(argv[1], "batch")) return batch();
    if (!std::strcmp(argv[1], "reserve")) return reserve();
    if (!std::strcmp(argv[1], "streams")) return streams();
    if (!std::strcmp(argv[1], "threads")) return threads();
    return 2;
}
