// Runs host parts of libsal's runtime under AddressSanitizer and
// UndefinedBehaviorSanitizer.  argv[1] names the check; exit status 0 when it
// holds, a message and 1 when it does not.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <vector>

#include "runtime.h"

// A card of kCard bytes in place of the device.
namespace {
constexpr size_t kCard = (size_t)1 << 30;
std::mutex card_mu;
std::map<void *, size_t> card;
size_t card_used = 0;
}  // namespace

extern "C" {
hipError_t hipMalloc(void **ptr, size_t bytes) {
    std::lock_guard<std::mutex> lk(card_mu);
    *ptr = nullptr;
    if (card_used + bytes > kCard) return hipErrorOutOfMemory;
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
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
}

namespace {

#define CHECK(what)                                              \
    do {                                                         \
        if (!(what)) {                                           \
            std::printf("line %d: %s\n", __LINE__, #what);       \
            return 1;                                            \
        }                                                        \
    } while (0)

// Idle blocks are given back when an allocation of either kind needs the memory.
int reserve() {
    sal::pool_add_context();
    const uint64_t t = sal::new_stream_token();
    void *a = nullptr, *b = nullptr;
    CHECK(sal::pool_malloc(&a, kCard * 3 / 8, t) == hipSuccess);
    sal::pool_free(a, t);
    CHECK(card_used >= kCard * 3 / 8);   // kept
    CHECK(sal::dev_malloc(&b, kCard * 3 / 4) == hipSuccess);
    CHECK(sal::dev_malloc(&a, kCard / 2) == hipErrorOutOfMemory);   // nothing left to give
    CHECK(hipFree(b) == hipSuccess);
    CHECK(sal::pool_malloc(&a, kCard * 3 / 8, t) == hipSuccess);
    sal::pool_free(a, t);
    CHECK(sal::pool_malloc(&b, kCard * 3 / 4, t) == hipSuccess);
    sal::pool_free(b, t);
    sal::pool_remove_context();
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

}  // namespace

int main(int argc, char **argv) {
    if (argc != 2) return 2;
    if (!std::strcmp(argv[1], "scratch")) return scratch();
    if (!std::strcmp(argv[1], "reserve")) return reserve();
    return 2;
}
