// Conforming transition refinement of the leaf set (paper section 2.1.2,
// Fig. 2c-e) and the conforming mesh it gives: explicit tetrahedra over
// numbered nodes.
//
// A leaf edge is *hanging* when its midpoint is a vertex of another leaf; a
// node at a quarter point means a neighbour two or more levels finer.  The
// patterns the paper splits are one hanging edge (2 tetrahedra), two hanging
// edges of one face (3) and the three edges of one face (4); a leaf with any
// other pattern is split into its 8 children (labels kept) and the patterns
// are found again (closure, driven from mesh.cpp).  Nodes are points of the
// finest grid (level kMaxLevels), keyed by 21-bit coordinates.
#include <hip/hip_runtime.h>
#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include "kuhn_dev.h"
#include "mesh_internal.h"

namespace sal {
namespace {

constexpr uint64_t kEmpty = ~0ull;
constexpr unsigned kDeep = 1u << 6;   // an edge has a node at a quarter point
constexpr unsigned kRed = 1u << 7;    // pattern not split by the paper: split 1 -> 8

// The four vertices of leaf (l, i) on the finest grid.
__device__ __forceinline__ void leaf_fine_vertices(const LevelPtrs &L, const LatticeGeom &g, int l,
                                                   int64_t i, int64_t F[4][3]) {
    int lk, q;
    int64_t c[3];
    split_key(entry_key(L, g, l, i), lk, q, c);
    kuhn_vertices(q, c, F);
    const int sh = kMaxLevels - l;
    for (int v = 0; v < 4; ++v)
        for (int a = 0; a < 3; ++a) F[v][a] <<= sh;
}

__device__ __forceinline__ uint64_t fine_key(const int64_t f[3]) {
    return ((uint64_t)f[0] << 42) | ((uint64_t)f[1] << 21) | (uint64_t)f[2];
}

__device__ __forceinline__ uint64_t set_hash(uint64_t k) {
    k ^= k >> 33;
    k *= 0xff51afd7ed558ccdull;
    k ^= k >> 33;
    k *= 0xc4ceb9fe1a85ec53ull;
    k ^= k >> 33;
    return k;
}

__device__ __forceinline__ bool set_find(const unsigned long long *tkeys, int64_t cap, uint64_t key) {
    uint64_t h = set_hash(key) & (uint64_t)(cap - 1);
    for (int64_t probe = 0; probe < cap; ++probe) {
        const uint64_t k = tkeys[h];
        if (k == key) return true;
        if (k == kEmpty) return false;
        h = (h + 1) & (uint64_t)(cap - 1);
    }
    return false;
}

// Inserts key; *added tells whether it was new.  False when the table is full.
// A slot only ever changes from empty to a key, so a key read with a plain
// (cached) load is final: most inserts find their key already there (a vertex is
// shared by many leaves) and need no atomic; an empty slot is claimed with a
// compare-and-swap.
__device__ __forceinline__ bool set_insert(unsigned long long *tkeys, int64_t cap, uint64_t key,
                                           bool *added) {
    uint64_t h = set_hash(key) & (uint64_t)(cap - 1);
    for (int64_t probe = 0; probe < cap; ++probe) {
        unsigned long long cur = __hip_atomic_load(&tkeys[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (cur == kEmpty) cur = atomicCAS(&tkeys[h], kEmpty, key);
        if (cur == kEmpty || cur == key) {
            if (added) *added = cur == kEmpty;
            return true;
        }
        h = (h + 1) & (uint64_t)(cap - 1);
    }
    return false;
}

// Sets the bit of every level-0 cell whose closure holds the finest-grid
// point f (up to 8 cells for a point on cell corners).
__device__ __forceinline__ void mark_cells(uint32_t *__restrict__ bits, const LatticeGeom &g,
                                           const int64_t f[3]) {
    int64_t lo[3], hi[3];
    for (int a = 0; a < 3; ++a) {
        const int64_t c = f[a] >> kMaxLevels, last = g.cells[a] - 1;
        const bool on_face = (f[a] & ((1 << kMaxLevels) - 1)) == 0;
        hi[a] = c < last ? c : last;
        lo[a] = on_face && c > 0 ? c - 1 : c;
        if (lo[a] > last) lo[a] = last;
    }
    for (int64_t z = lo[2]; z <= hi[2]; ++z)
        for (int64_t y = lo[1]; y <= hi[1]; ++y)
            for (int64_t x = lo[0]; x <= hi[0]; ++x) {
                const int64_t cell = (z * g.cells[1] + y) * g.cells[0] + x;
                atomicOr(&bits[cell >> 5], 1u << (cell & 31));
            }
}

// Empties the vertices new in a round and their cells' bits.
__global__ void k_closure_clear(unsigned long long *__restrict__ fresh, int64_t fcap,
                                uint32_t *__restrict__ cells_new, int64_t cell_words) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < fcap) fresh[i] = kEmpty;
    else if (i - fcap < cell_words) cells_new[i - fcap] = 0u;
}

// Inserts the vertices of the spans' entries (leaves or not: an inner entry's
// vertices are those of its corner children).  Keys that were not in the set are
// counted in *n_new and, when `fresh` is given, also put in that second set (the
// vertices new in this closure round), with the bits of the level-0 cells they
// touch set in `cells_new`.
__global__ void k_insert_levels(LevelPtrs L, LatticeGeom g, LevelSpans r,
                                unsigned long long *__restrict__ set, int64_t cap,
                                unsigned long long *__restrict__ fresh, int64_t fcap,
                                uint32_t *__restrict__ cells_new,
                                unsigned long long *__restrict__ n_new,
                                unsigned long long *__restrict__ overflow) {
    int64_t jj;
    const int l = span_level(r, jj);
    unsigned n_added = 0;   // the wavefront's
    for (int u = 0; u < r.turns; ++u, jj += 256) {
        bool added = false;
        if (jj < 4 * (r.n[l] - r.first[l])) {
            int64_t F[4][3];
            leaf_fine_vertices(L, g, l, r.first[l] + (jj >> 2), F);
            const uint64_t key = fine_key(F[jj & 3]);
            if (set_insert(set, cap, key, &added)) {
                if (added && fresh) {
                    if (set_insert(fresh, fcap, key, nullptr))
                        mark_cells(cells_new, g, F[jj & 3]);
                    else
                        atomicAdd(overflow, 1ull);
                }
            } else {
                atomicAdd(overflow, 1ull);
            }
        }
        n_added += (unsigned)__popcll(__ballot(added));
    }
    // one counter update per block
    __shared__ unsigned int block_new;
    if (threadIdx.x == 0) block_new = 0;
    __syncthreads();
    if ((threadIdx.x & 63) == 0 && n_added) atomicAdd(&block_new, n_added);
    __syncthreads();
    if (threadIdx.x == 0 && block_new) atomicAdd(n_new, (unsigned long long)block_new);
}

constexpr int kEdgeA[6] = {0, 0, 0, 1, 1, 2};
constexpr int kEdgeB[6] = {1, 2, 3, 2, 3, 3};

__device__ __forceinline__ bool allowed_pattern(unsigned bits) {
    const int n = __popc(bits);
    if (n <= 1) return true;
    if (n > 3) return false;
    unsigned verts = 0;
    for (int e = 0; e < 6; ++e)
        if (bits >> e & 1u) verts |= (1u << kEdgeA[e]) | (1u << kEdgeB[e]);
    return __popc(verts) == 3;   // two edges sharing a vertex, or the edges of one face
}

// Hanging-edge bits (0-5) and the quarter-point flag (bit 6) of a level-l
// leaf against a vertex set.
__device__ __forceinline__ unsigned leaf_hits(const int64_t F[4][3], int l,
                                              const unsigned long long *set, int64_t cap) {
    unsigned bits = 0;
    for (int e = 0; e < 6; ++e) {
        const int a = kEdgeA[e], b = kEdgeB[e];
        if (l < kMaxLevels) {
            int64_t m[3];
            for (int x = 0; x < 3; ++x) m[x] = (F[a][x] + F[b][x]) >> 1;
            if (set_find(set, cap, fine_key(m))) bits |= 1u << e;
        }
        if (l + 2 <= kMaxLevels && !(bits & kDeep)) {
            int64_t q1[3], q2[3];
            for (int x = 0; x < 3; ++x) {
                q1[x] = (3 * F[a][x] + F[b][x]) >> 2;
                q2[x] = (F[a][x] + 3 * F[b][x]) >> 2;
            }
            if (set_find(set, cap, fine_key(q1)) || set_find(set, cap, fine_key(q2))) bits |= kDeep;
        }
    }
    return bits;
}

__device__ __forceinline__ uint8_t with_red(unsigned f) {
    return (uint8_t)(((f & kDeep) || !allowed_pattern(f & 63u)) ? f | kRed : f);
}

// Patterns after a closure round: flag = hanging bits | deep | red for a leaf, 0
// for an inner entry.  Entries from first on are new and get theirs from the whole
// vertex set.  For an older leaf the set has only grown, so its pattern is the old
// one plus what the vertices of this round (the `fresh` set) hit; every point it
// tests lies in the closure of its level-0 cell, so a leaf whose cell got no new
// vertex keeps its pattern without probing the set.
__global__ void k_pattern_levels(LevelPtrs L, LatticeGeom g, LevelSpans r,
                                 const unsigned long long *__restrict__ set, int64_t cap,
                                 const unsigned long long *__restrict__ fresh, int64_t fcap,
                                 const uint32_t *__restrict__ cells_new) {
    int64_t i;
    const int l = span_level(r, i);
    if (i >= r.n[l]) return;
    const bool is_new = i >= r.first[l];
    const uint8_t old = is_new ? 0 : L.flag[l][i];
    if (L.child[l][i] >= 0) {
        if (is_new || old) L.flag[l][i] = 0;
        return;
    }
    if (!is_new) {
        int64_t cell;
        if (l == 0) {
            cell = i / 6;
        } else {
            int lk, q;
            int64_t c[3];
            split_key(L.key[l][i], lk, q, c);
            cell = ((c[2] >> l) * g.cells[1] + (c[1] >> l)) * g.cells[0] + (c[0] >> l);
        }
        if (!((cells_new[cell >> 5] >> (cell & 31)) & 1u)) return;
    }
    int64_t F[4][3];
    leaf_fine_vertices(L, g, l, i, F);
    const unsigned f = old | leaf_hits(F, l, is_new ? set : fresh, is_new ? cap : fcap);
    if (is_new || f != old) L.flag[l][i] = with_red(f);
}

// Tetrahedra per listed leaf: one plus its number of hanging edges; hist[k]
// counts the leaves cut into k + 1 pieces (one atomic per block and bin).
__global__ void k_tet_counts(LevelPtrs L, LevelSpans r, const int32_t *__restrict__ list,
                             int32_t *__restrict__ counts, unsigned long long *__restrict__ hist) {
    __shared__ unsigned int bins[4];
    if (threadIdx.x < 4) bins[threadIdx.x] = 0;
    __syncthreads();
    int64_t j;
    const int l = span_level(r, j);
    unsigned n[4] = {0, 0, 0, 0};   // the wavefront's
    for (int u = 0; u < r.turns; ++u, j += 256) {
        int c = 0;
        if (j < r.n[l]) {
            c = 1 + __popc((unsigned)L.flag[l][list[r.first[l] + j]] & 63u);
            counts[r.first[l] + j] = c;
        }
        for (int k = 0; k < 4; ++k) n[k] += (unsigned)__popcll(__ballot(k < 3 ? c == k + 1 : c >= 4));
    }
    for (int k = 0; k < 4; ++k)
        if ((threadIdx.x & 63) == 0 && n[k]) atomicAdd(&bins[k], n[k]);
    __syncthreads();
    if (threadIdx.x < 4 && bins[threadIdx.x]) atomicAdd(&hist[threadIdx.x], (unsigned long long)bins[threadIdx.x]);
}

// ------------------------------------------------------------------ numbering
// The nodes of the conforming mesh are the vertex set: every key in it is a vertex
// of some leaf, and a leaf's tetrahedra use its vertices and vertices of others.
// (Sorting the corners' keys instead, four for each tetrahedron, dropping the
// repeated ones and finding every corner again by bisection took 2.4 ms for 5.2M
// tetrahedra with 0.88M nodes; this takes 0.7.)
__device__ __forceinline__ uint64_t pack_key(uint64_t k, const NodeBits &nb) {
    return ((k >> 42) << (nb.y + nb.z)) | (((k >> 21) & 0x1fffffu) << nb.z) | (k & 0x1fffffu);
}

__device__ __forceinline__ uint64_t unpack_key(uint64_t p, const NodeBits &nb) {
    return ((p >> (nb.y + nb.z)) << 42) | (((p >> nb.z) & ((1ull << nb.y) - 1ull)) << 21) |
           (p & ((1ull << nb.z) - 1ull));
}

constexpr int kKeysPerThread = 16;

__global__ __launch_bounds__(256) void k_set_keys(const unsigned long long *__restrict__ set, int64_t cap,
                                                  NodeBits nb, uint64_t *__restrict__ out, int64_t out_cap,
                                                  unsigned long long *__restrict__ n_out) {
    __shared__ unsigned wave_n[4];
    __shared__ unsigned long long base;
    const int64_t first = (int64_t)blockIdx.x * 256 * kKeysPerThread + threadIdx.x;
    const int wave = threadIdx.x >> 6;
    unsigned long long k[kKeysPerThread];
    unsigned before[kKeysPerThread], n = 0;
    for (int j = 0; j < kKeysPerThread; ++j) {
        const int64_t i = first + 256 * j;
        k[j] = i < cap ? set[i] : kEmpty;
        const unsigned long long m = __ballot(k[j] != kEmpty);
        before[j] = n + __popcll(m & ((1ull << (threadIdx.x & 63)) - 1ull));
        n += (unsigned)__popcll(m);
    }
    if ((threadIdx.x & 63) == 0) wave_n[wave] = n;
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned all = wave_n[0] + wave_n[1] + wave_n[2] + wave_n[3];
        base = all ? atomicAdd(n_out, (unsigned long long)all) : 0ull;
    }
    __syncthreads();
    unsigned long long at = base;
    for (int w = 0; w < wave; ++w) at += wave_n[w];
    for (int j = 0; j < kKeysPerThread; ++j)
        if (k[j] != kEmpty && (int64_t)(at + before[j]) < out_cap) out[at + before[j]] = pack_key(k[j], nb);
}

// Where the table holds a key; the key is there, or a place for it is.
__device__ __forceinline__ int64_t node_slot(const NodeEntry *__restrict__ table, int64_t cap, uint64_t key) {
    uint64_t h = set_hash(key) & (uint64_t)(cap - 1);
    for (int64_t probe = 0; probe < cap; ++probe) {
        const uint64_t k = table[h].key;
        if (k == key) return (int64_t)h;
        if (k == kEmpty) break;
        h = (h + 1) & (uint64_t)(cap - 1);
    }
    return 0;
}

__global__ void k_clear_nodes(NodeEntry *__restrict__ table, int64_t cap) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < cap) table[i] = NodeEntry{kEmpty, 0, 0};
}

__global__ void k_number_nodes(LatticeGeom g, const uint64_t *__restrict__ packed, int64_t n, NodeBits nb,
                               NodeEntry *__restrict__ table, int64_t cap, int64_t *__restrict__ keys,
                               float *__restrict__ xyz) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t p = packed[i], k = unpack_key(p, nb);
    keys[i] = (int64_t)k;
    const int64_t f[3] = {(int64_t)(k >> 42), (int64_t)((k >> 21) & 0x1fffffu), (int64_t)(k & 0x1fffffu)};
    const double hf = ldexp(g.h, -kMaxLevels);
    for (int a = 0; a < 3; ++a) xyz[3 * i + a] = lattice_coord(g.origin[a], hf, (double)f[a]);
    uint64_t h = set_hash(p) & (uint64_t)(cap - 1);
    for (int64_t probe = 0; probe < cap; ++probe) {
        if (atomicCAS(&table[h].key, kEmpty, (unsigned long long)p) == kEmpty) {
            table[h].id = (int32_t)i;
            return;
        }
        h = (h + 1) & (uint64_t)(cap - 1);
    }
}

// Writes tetrahedra as node numbers.
struct TetSink {
    const NodeEntry *table;
    int64_t cap;
    NodeBits nb;
    int32_t *ids;

    __device__ __forceinline__ int32_t id(const int64_t f[3]) const {
        return table[node_slot(table, cap, pack_key(fine_key(f), nb))].id;
    }
    __device__ __forceinline__ void put(int64_t slot, const int64_t a[3], const int64_t b[3], const int64_t c[3],
                                        const int64_t d[3]) const {
        // positive orientation: det(b - a, c - a, d - a) > 0, else swap a and b
        const int64_t u[3] = {b[0] - a[0], b[1] - a[1], b[2] - a[2]};
        const int64_t v[3] = {c[0] - a[0], c[1] - a[1], c[2] - a[2]};
        const int64_t w[3] = {d[0] - a[0], d[1] - a[1], d[2] - a[2]};
        const int64_t det = u[0] * (v[1] * w[2] - v[2] * w[1]) - u[1] * (v[0] * w[2] - v[2] * w[0]) +
                            u[2] * (v[0] * w[1] - v[1] * w[0]);
        const int32_t ia = id(a), ib = id(b), ic = id(c), ie = id(d);
        *(int4 *)(ids + 4 * slot) = det > 0 ? make_int4(ia, ib, ic, ie) : make_int4(ib, ia, ic, ie);
    }
};

// The tetrahedra of every listed leaf at offsets[j] (first output slot).
__global__ void k_emit(LevelPtrs L, LatticeGeom g, LevelSpans r, const int32_t *__restrict__ list,
                       const int64_t *__restrict__ offsets, TetSink out, int32_t *__restrict__ labels) {
    int64_t j;
    const int l = span_level(r, j);
    if (j >= r.n[l]) return;
    j += r.first[l];
    const int64_t i = list[j];
    int64_t F[4][3];
    leaf_fine_vertices(L, g, l, i, F);
    const unsigned b = L.flag[l][i] & 63u;
    const int n = __popc(b);
    const int64_t o = offsets[j];
    const int32_t lab = L.label[l][i];
    for (int t = 0; t <= n; ++t) labels[o + t] = lab;
    if (n == 0) {
        out.put(o, F[0], F[1], F[2], F[3]);
        return;
    }
    int ed[3], k = 0;
    for (int e = 0; e < 6; ++e)
        if (b >> e & 1u) ed[k++] = e;
    if (n == 1) {
        const int x = kEdgeA[ed[0]], y = kEdgeB[ed[0]];
        int o2[2], m = 0;
        for (int v = 0; v < 4; ++v)
            if (v != x && v != y) o2[m++] = v;
        int64_t mid[3];
        for (int a = 0; a < 3; ++a) mid[a] = (F[x][a] + F[y][a]) >> 1;
        out.put(o, F[x], mid, F[o2[0]], F[o2[1]]);
        out.put(o + 1, mid, F[y], F[o2[0]], F[o2[1]]);
        return;
    }
    if (n == 2) {
        const int e0a = kEdgeA[ed[0]], e0b = kEdgeB[ed[0]];
        const int e1a = kEdgeA[ed[1]], e1b = kEdgeB[ed[1]];
        const int a = (e0a == e1a || e0a == e1b) ? e0a : e0b;   // the shared vertex
        const int bv = e0a + e0b - a, cv = e1a + e1b - a;
        const int d = 6 - a - bv - cv;
        int64_t m1[3], m2[3];
        for (int x = 0; x < 3; ++x) {
            m1[x] = (F[a][x] + F[bv][x]) >> 1;
            m2[x] = (F[a][x] + F[cv][x]) >> 1;
        }
        out.put(o, F[a], m1, m2, F[d]);
        // the quadrilateral (m1, b, c, m2) is cut along the diagonal through
        // its smallest node key, a property of the face alone
        const uint64_t km1 = fine_key(m1), kb = fine_key(F[bv]), kc = fine_key(F[cv]),
                       km2 = fine_key(m2);
        const uint64_t low = min(min(km1, kb), min(kc, km2));
        if (low == km1 || low == kc) {
            out.put(o + 1, m1, F[bv], F[cv], F[d]);
            out.put(o + 2, m1, F[cv], m2, F[d]);
        } else {
            out.put(o + 1, m1, F[bv], m2, F[d]);
            out.put(o + 2, F[bv], F[cv], m2, F[d]);
        }
        return;
    }
    // three edges of one face (a < b < c), apex d
    unsigned vm = 0;
    for (int q = 0; q < 3; ++q) vm |= (1u << kEdgeA[ed[q]]) | (1u << kEdgeB[ed[q]]);
    int fv[3], m = 0, d = 0;
    for (int v = 0; v < 4; ++v) {
        if (vm >> v & 1u) fv[m++] = v;
        else d = v;
    }
    int64_t mab[3], mbc[3], mca[3];
    for (int x = 0; x < 3; ++x) {
        mab[x] = (F[fv[0]][x] + F[fv[1]][x]) >> 1;
        mbc[x] = (F[fv[1]][x] + F[fv[2]][x]) >> 1;
        mca[x] = (F[fv[2]][x] + F[fv[0]][x]) >> 1;
    }
    out.put(o, F[fv[0]], mab, mca, F[d]);
    out.put(o + 1, mab, F[fv[1]], mbc, F[d]);
    out.put(o + 2, mca, mbc, F[fv[2]], F[d]);
    out.put(o + 3, mab, mbc, mca, F[d]);
}

inline unsigned grid_of(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

// In a launch that counts, a large one gives a thread 16 items: a counter takes some
// 5 ns for each workgroup's update (11M vertices inserted: 580 us with 45,000 of
// them, 190 now).
static int count_turns(const int64_t (&per)[kMaxLevels + 1]) {
    int64_t all = 0;
    for (const int64_t n : per) all += n;
    return all >= (int64_t)1 << 21 ? 16 : 1;
}

hipError_t launch_closure_clear(unsigned long long *fresh, int64_t fcap, uint32_t *cells_new, int64_t cell_words,
                                hipStream_t s) {
    k_closure_clear<<<grid_of(fcap + cell_words), 256, 0, s>>>(fresh, fcap, cells_new, cell_words);
    return hipGetLastError();
}

hipError_t launch_insert_levels(const LevelPtrs &L, const LatticeGeom &g, const LevelSpans &r,
                                unsigned long long *set, int64_t cap, unsigned long long *fresh, int64_t fcap,
                                uint32_t *cells_new, unsigned long long *n_new, unsigned long long *overflow,
                                hipStream_t s) {
    int64_t per[kMaxLevels + 1] = {}, nb;
    for (int l = 0; l <= r.top; ++l) per[l] = 4 * (r.n[l] - r.first[l]);
    const LevelSpans q = with_blocks(r, per, count_turns(per), &nb);
    if (nb == 0) return hipSuccess;
    if (nb > 0x7fffffff) return hipErrorInvalidValue;
    k_insert_levels<<<(unsigned)nb, 256, 0, s>>>(L, g, q, set, cap, fresh, fcap, cells_new, n_new, overflow);
    return hipGetLastError();
}

hipError_t launch_pattern_levels(const LevelPtrs &L, const LatticeGeom &g, const LevelSpans &r,
                                 const unsigned long long *set, int64_t cap, const unsigned long long *fresh,
                                 int64_t fcap, const uint32_t *cells_new, hipStream_t s) {
    int64_t per[kMaxLevels + 1] = {}, nb;
    for (int l = 0; l <= r.top; ++l) per[l] = r.n[l];
    const LevelSpans q = with_blocks(r, per, 1, &nb);
    if (nb == 0) return hipSuccess;
    if (nb > 0x7fffffff) return hipErrorInvalidValue;
    k_pattern_levels<<<(unsigned)nb, 256, 0, s>>>(L, g, q, set, cap, fresh, fcap, cells_new);
    return hipGetLastError();
}

hipError_t launch_tet_counts(const LevelPtrs &L, const LevelSpans &r, const int32_t *list, int32_t *counts,
                             unsigned long long *hist, hipStream_t s) {
    int64_t per[kMaxLevels + 1] = {}, nb;
    for (int l = 0; l <= r.top; ++l) per[l] = r.n[l];
    const LevelSpans q = with_blocks(r, per, count_turns(per), &nb);
    if (nb == 0) return hipSuccess;
    if (nb > 0x7fffffff) return hipErrorInvalidValue;
    k_tet_counts<<<(unsigned)nb, 256, 0, s>>>(L, q, list, counts, hist);
    return hipGetLastError();
}

hipError_t exclusive_sum_i32(const int32_t *in, int64_t *out, int64_t n, void *tmp,
                             size_t *tmp_bytes, hipStream_t s) {
    return rocprim::exclusive_scan(tmp, *tmp_bytes, in, out, (int64_t)0, (size_t)n,
                                   rocprim::plus<int64_t>(), s);
}

hipError_t launch_set_keys(const unsigned long long *set, int64_t cap, const NodeBits &nb, uint64_t *out,
                           int64_t out_cap, unsigned long long *n_out, hipStream_t s) {
    const int64_t per = 256 * kKeysPerThread;
    k_set_keys<<<(unsigned)((cap + per - 1) / per), 256, 0, s>>>(set, cap, nb, out, out_cap, n_out);
    return hipGetLastError();
}

hipError_t sort_packed(const uint64_t *in, uint64_t *out, int64_t n, int bits, void *tmp, size_t *tmp_bytes,
                       hipStream_t s) {
    return rocprim::radix_sort_keys(tmp, *tmp_bytes, in, out, (size_t)n, 0u, (unsigned)bits, s);
}

hipError_t launch_number_nodes(const LatticeGeom &g, const uint64_t *packed, int64_t n, const NodeBits &nb,
                               NodeEntry *table, int64_t cap, int64_t *keys, float *xyz, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    k_clear_nodes<<<grid_of(cap), 256, 0, s>>>(table, cap);
    k_number_nodes<<<grid_of(n), 256, 0, s>>>(g, packed, n, nb, table, cap, keys, xyz);
    return hipGetLastError();
}

hipError_t launch_emit(const LevelPtrs &L, const LatticeGeom &g, const LevelSpans &r, const int32_t *list,
                       const int64_t *offsets, const NodeBits &nb, const NodeEntry *table, int64_t cap,
                       int32_t *ids, int32_t *labels, hipStream_t s) {
    int64_t per[kMaxLevels + 1] = {}, blocks;
    for (int l = 0; l <= r.top; ++l) per[l] = r.n[l];
    const LevelSpans q = with_blocks(r, per, 1, &blocks);
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    k_emit<<<(unsigned)blocks, 256, 0, s>>>(L, g, q, list, offsets, TetSink{table, cap, nb, ids}, labels);
    return hipGetLastError();
}

}  // namespace sal
