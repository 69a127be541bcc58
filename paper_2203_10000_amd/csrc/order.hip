// Spatial order of the points to be labeled, so that the 64 points of a
// wavefront lie close together: a stable counting sort by the place of the
// point's cell (128 per axis of the surface set's box; points outside it go to
// the border cells) on a Hilbert curve, 11 low bits, then 10 high bits.  Along a
// Hilbert curve consecutive cells are neighbours.  In Morton order one run of 64
// in a hundred jumps across a quarter of the box (on 1.3M lattice points: extent
// 13.6 mm on average, 46.7 mm at the 99th percentile, 198 mm at most, against
// 11.2, 17.5 and 20.0 mm), its surfaces meet far more boxes (0.69 of them
// against 0.52 over four shells), and such wavefronts are the launch's tail.
// Stable, so that the wavefronts, and with them every rounding, are the same
// in every run.
//
// Per pass: a histogram per tile, a scan over the tiles of each bin, and a
// scatter that ranks the keys of a tile in input order (wave by wave, 64 at a
// time, equal digits found by one ballot per bit).  Up to some 200,000 points it is
// bound by its six launches and the chains in them (51 us), at 6M by the ranking's
// instructions and the places on the curve, which three of the launches compute (276
// us for 46 bytes a point read and 10 written).  One pass over
// 2048 cells takes 20 us off below 2^18 points, but points along a surface fill few
// cells: 60,001 of them near two surfaces 280 -> 490 us.  All instances of a batch are sorted by the same three
// launches (their tiles are separate).  No memsets, no allocations: the
// launches can be captured.
#include <hip/hip_runtime.h>

#include "sal_internal.h"
#include "wave.h"

namespace sal {
namespace {

constexpr int kThreads = 256, kWaves = kThreads / 64;
constexpr int kAxisBits = 7;
static_assert(3 * kAxisBits == kOrderBits1 + kOrderBits2, "two digits hold a place on the curve");

__device__ __forceinline__ int find_tile(const LabelInst *insts, int n_inst, int64_t t) {
    int lo = 0, hi = n_inst - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (insts[mid].tile_base <= t) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Three bits apart: the low seven bits of v.
__device__ __forceinline__ uint32_t spread3(uint32_t v) {
    v = (v | (v << 8)) & 0x0000f00fu;
    v = (v | (v << 4)) & 0x000c30c3u;
    v = (v | (v << 2)) & 0x00249249u;
    return v;
}

// Place of cell q (kAxisBits bits an axis) on the Hilbert curve: J. Skilling,
// "Programming the Hilbert curve", AIP Conf. Proc. 707 (2004) -- from the top bit
// down, each axis' bit either reflects the lower bits of axis 0 or exchanges them
// with its own; a Gray decode across the axes follows.
__device__ __forceinline__ uint32_t hilbert(uint32_t (&q)[3]) {
#pragma unroll
    for (int b = kAxisBits - 1; b > 0; --b) {
        const uint32_t low = (1u << b) - 1u;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const uint32_t set = 0u - ((q[c] >> b) & 1u);           // all ones where the bit is set
            const uint32_t flip = low & set, swap = (q[0] ^ q[c]) & low & ~set;
            q[0] ^= flip | swap;
            q[c] ^= swap;                                           // (axis 0 exchanges with itself: 0)
        }
    }
    q[1] ^= q[0];
    q[2] ^= q[1];
    uint32_t t = 0;
#pragma unroll
    for (int b = kAxisBits - 1; b > 0; --b) t ^= ((1u << b) - 1u) & (0u - ((q[2] >> b) & 1u));
    return (spread3(q[0] ^ t) << 2) | (spread3(q[1] ^ t) << 1) | spread3(q[2] ^ t);
}

__device__ __forceinline__ uint32_t cell_code(const LabelInst &in, int64_t i) {
    uint32_t q[3];
    const float p[3] = {in.x[i], in.y[i], in.z[i]};
    for (int c = 0; c < 3; ++c) {
        // (a NaN becomes 0: fmaxf and fminf return the other operand)
        const float f = fminf(fmaxf((p[c] - in.lo[c]) * in.scale[c], 0.0f), 127.0f);
        q[c] = (uint32_t)f;
    }
    return hilbert(q);
}

template <int PASS>
__device__ __forceinline__ uint32_t digit(const LabelArgs &a, const LabelInst &in, int64_t i, uint32_t &code) {
    if (PASS == 1) {
        code = cell_code(in, i);
        return code & (kOrderBins - 1);
    }
    code = a.ord.key1[in.order_base + i];
    return code;
}

template <int PASS>
constexpr int bins() { return PASS == 1 ? kOrderBins : 1 << kOrderBits2; }

template <int PASS>
__global__ __launch_bounds__(kThreads) void k_order_hist(LabelArgs a) {
    __shared__ uint32_t h[bins<PASS>()];
    const int ii = a.insts ? find_tile(a.insts, a.n_inst, blockIdx.x) : 0;
    const LabelInst &in = a.insts ? a.insts[ii] : a.one;
    const int64_t n = label_count(a, in), t = (int64_t)blockIdx.x - in.tile_base;
    if (PASS == 1 && blockIdx.x == 0 && threadIdx.x < kNumWork) a.work[threadIdx.x] = 0ull;
    // The whole workgroup.  Grids of a device-side count are as large as its bound:
    // with empty tiles counted and scanned, two captured rounds of a small head took
    // 905 us instead of 805.
    if (t * in.tile >= n) return;
    for (int b = threadIdx.x; b < bins<PASS>(); b += kThreads) h[b] = 0u;
    __syncthreads();
    const int64_t i0 = t * in.tile, i1 = i0 + in.tile < n ? i0 + in.tile : n;
    for (int64_t i = i0 + threadIdx.x; i < i1; i += kThreads) {
        uint32_t code;
        atomicAdd(&h[digit<PASS>(a, in, i, code)], 1u);
    }
    __syncthreads();
    uint32_t *out = a.ord.hist + kOrderBins * in.tile_base + t;
    for (int b = threadIdx.x; b < bins<PASS>(); b += kThreads) out[(int64_t)b * in.n_tiles] = h[b];
}

// One wavefront per (bin, instance): exclusive scan over the tiles that have
// points, in place.
template <int PASS>
__global__ __launch_bounds__(64) void k_order_scan(LabelArgs a) {
    const int ii = (int)(blockIdx.x / bins<PASS>()), bin = (int)(blockIdx.x % bins<PASS>());
    const int lane = lane_id();
    const LabelInst &in = a.insts ? a.insts[ii] : a.one;
    uint32_t *h = a.ord.hist + kOrderBins * in.tile_base + (int64_t)bin * in.n_tiles;
    const int used = (int)((label_count(a, in) + in.tile - 1) / in.tile);
    uint32_t run = 0;
    for (int b = 0; b < used; b += 64) {
        const uint32_t v = b + lane < used ? h[b + lane] : 0u;
        uint32_t s = v;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t u = (uint32_t)__shfl_up((int)s, d);
            if (lane >= d) s += u;
        }
        if (b + lane < used) h[b + lane] = run + s - v;
        run += (uint32_t)__shfl((int)s, 63);
    }
    if (lane == 0) a.ord.tot[(int64_t)ii * kOrderBins + bin] = run;
}

template <int PASS>
__global__ __launch_bounds__(kThreads) void k_order_scatter(LabelArgs a) {
    constexpr int B = bins<PASS>(), PER = B / kThreads, BITS = PASS == 1 ? kOrderBits1 : kOrderBits2;
    __shared__ uint32_t cnt[kWaves][B];
    __shared__ uint32_t base[B];
    __shared__ uint32_t part[kThreads];
    const int ii = a.insts ? find_tile(a.insts, a.n_inst, blockIdx.x) : 0;
    const LabelInst &in = a.insts ? a.insts[ii] : a.one;
    const int64_t n = label_count(a, in), t = (int64_t)blockIdx.x - in.tile_base;
    const int64_t i0 = t * in.tile, i1 = i0 + in.tile < n ? i0 + in.tile : n;
    if (i0 >= i1) return;   // (the whole workgroup)
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    // where each bin of this tile starts: all smaller bins, then this bin's
    // earlier tiles
    const uint32_t *tot = a.ord.tot + (int64_t)ii * kOrderBins;
    uint32_t sum = 0;
    for (int q = 0; q < PER; ++q) sum += tot[tid * PER + q];
    part[tid] = sum;
    __syncthreads();
    for (int d = 1; d < kThreads; d <<= 1) {
        const uint32_t u = tid >= d ? part[tid - d] : 0u;
        __syncthreads();
        part[tid] += u;
        __syncthreads();
    }
    uint32_t run = part[tid] - sum;
    const uint32_t *h = a.ord.hist + kOrderBins * in.tile_base + t;
    for (int q = 0; q < PER; ++q) {
        const int b = tid * PER + q;
        base[b] = run + h[(int64_t)b * in.n_tiles];
        run += tot[b];
    }
    for (int w = 0; w < kWaves; ++w)
        for (int b = tid; b < B; b += kThreads) cnt[w][b] = 0u;
    __syncthreads();
    // each wavefront owns a quarter of the tile, in order
    const int64_t quarter = in.tile / kWaves;
    const int64_t w0 = i0 + wave * quarter, w1 = w0 + quarter < i1 ? w0 + quarter : i1;
    for (int64_t i = w0 + lane; i < w1; i += 64) {
        uint32_t code;
        atomicAdd(&cnt[wave][digit<PASS>(a, in, i, code)], 1u);
    }
    __syncthreads();
    for (int b = tid; b < B; b += kThreads) {
        uint32_t at = base[b];
        for (int w = 0; w < kWaves; ++w) {
            const uint32_t c = cnt[w][b];
            cnt[w][b] = at;
            at += c;
        }
    }
    __syncthreads();
    for (int64_t b = w0; b < w1; b += 64) {
        const int64_t i = b + lane;
        const bool have = i < w1;
        uint32_t code = 0;
        const uint32_t d = have ? digit<PASS>(a, in, i, code) : 0u;
        uint64_t same = ballot(have);
#pragma unroll
        for (int q = 0; q < BITS; ++q) {
            const uint64_t m = ballot((d >> q) & 1u);
            same &= ((d >> q) & 1u) ? m : ~m;
        }
        const uint32_t at = cnt[wave][d] + (uint32_t)lanes_below(same);
        wave_sync();
        if (have) {
            if (lanes_below(same) == 0) cnt[wave][d] = at + (uint32_t)__popcll(same);
            if (PASS == 1) {
                a.ord.idx1[in.order_base + at] = (uint32_t)i;
                a.ord.key1[in.order_base + at] = (uint16_t)(code >> kOrderBits1);
            } else {
                a.ord.perm[in.order_base + at] = a.ord.idx1[in.order_base + i];
            }
        }
        wave_sync();
    }
}

}  // namespace

hipError_t launch_order(const LabelArgs &a, int64_t tiles, hipStream_t s) {
    if (tiles <= 0) return hipSuccess;
    if (tiles > 0x7fffffff || (a.insts && a.n_inst > 0x7fffffff / kOrderBins)) return hipErrorInvalidValue;
    const unsigned ni = (unsigned)(a.insts ? a.n_inst : 1);
    const dim3 g((unsigned)tiles), b(kThreads);
    k_order_hist<1><<<g, b, 0, s>>>(a);
    k_order_scan<1><<<dim3(ni << kOrderBits1), dim3(64), 0, s>>>(a);
    k_order_scatter<1><<<g, b, 0, s>>>(a);
    k_order_hist<2><<<g, b, 0, s>>>(a);
    k_order_scan<2><<<dim3(ni << kOrderBits2), dim3(64), 0, s>>>(a);
    k_order_scatter<2><<<g, b, 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace sal
