// Runs host parts of libsal's runtime under AddressSanitizer and
// UndefinedBehaviorSanitizer.  argv[1] names the check; exit status 0 when it
// holds, a message and 1 when it does not.
#include <cstdio>
#include <cstring>
#include <vector>

#include "runtime.h"

namespace {

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
    return 2;
}
