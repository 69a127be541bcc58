// Rebuilding a refined mesh from its leaves (sal_tet_mesh_import): the leaves go
// into a hash table, their ancestors into a set, and the levels are laid out from
// the lattice down, each tetrahedron a leaf or refined and never both.
//
// Bound by latency and HBM (a few random probes per leaf).  The host form this
// replaces copied the leaves back, sorted them and searched per child: 0.46 s for
// 1.5 million leaves, against under a millisecond here.
#include <hip/hip_runtime.h>

#include "kuhn_dev.h"

namespace sal {
namespace {

constexpr unsigned long long kNoKey = ~0ull;
// The tables are at most a quarter full for a valid leaf set; a longer probe
// means that they hold far more (the set is invalid) and ends the search.
constexpr int kMaxProbe = 4096;

__device__ __forceinline__ uint64_t key_hash(uint64_t k) {
    k ^= k >> 33;
    k *= 0x9e3779b97f4a7c15ull;
    k ^= k >> 29;
    k *= 0xbf58476d1ce4e5b9ull;
    return k ^ (k >> 32);
}

// Slot of `key` after inserting it (*fresh: it was not there), -1: no room.
__device__ __forceinline__ int64_t insert(unsigned long long *t, int64_t cap, unsigned long long key, bool *fresh) {
    uint64_t h = key_hash(key) & (uint64_t)(cap - 1);
    for (int p = 0; p < kMaxProbe; ++p, h = (h + 1) & (uint64_t)(cap - 1)) {
        unsigned long long v = t[h];
        if (v == kNoKey) v = atomicCAS(&t[h], kNoKey, key);
        if (v == kNoKey || v == key) {
            *fresh = v == kNoKey;
            return (int64_t)h;
        }
    }
    return -1;
}

__device__ __forceinline__ int64_t find(const unsigned long long *t, int64_t cap, unsigned long long key) {
    uint64_t h = key_hash(key) & (uint64_t)(cap - 1);
    for (int p = 0; p < kMaxProbe; ++p, h = (h + 1) & (uint64_t)(cap - 1)) {
        const unsigned long long v = t[h];
        if (v == key) return (int64_t)h;
        if (v == kNoKey) return -1;
    }
    return -1;
}

// The parent of the tetrahedron (level l >= 1, q, cell c).
__device__ __forceinline__ uint64_t parent_key(const ChildTables &T, int l, int q, const int64_t c[3]) {
    const int code = (int)(c[0] & 1) | (int)((c[1] & 1) << 1) | (int)((c[2] & 1) << 2);
    int pq = 0;
    for (int k = 0; k < 6; ++k)
        if (T.rank[k][code][q] >= 0) pq = k;
    return make_key(l - 1, pq, c[0] >> 1, c[1] >> 1, c[2] >> 1);
}

__device__ __forceinline__ void fault(ImportFaults *f, int bit) { atomicOr(&f->bits, 1u << bit); }

__global__ void k_import_insert(const uint64_t *__restrict__ keys, const int32_t *__restrict__ labels, int64_t n,
                                LatticeGeom g, ChildTables T, ImportTables t, ImportFaults *f) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t key = keys[i];
    int l, q;
    int64_t c[3];
    split_key(key, l, q, c);
    int why = -1;
    if (l > kMaxLevels || q > 5) why = 0;
    else
        for (int a = 0; a < 3; ++a)
            if (c[a] >= ((int64_t)g.cells[a] << l)) why = 1;
    if (why < 0 && labels[i] < 0) why = 2;
    if (why >= 0) {   // the first such leaf is the one reported
        atomicMin(&f->first, ((unsigned long long)i << 2) | (unsigned)why);
        return;
    }
    bool fresh = false;
    const int64_t at = insert(t.leaf, t.leaf_cap, key, &fresh);
    if (at < 0) return fault(f, kFaultChildren);
    if (!fresh) return fault(f, kFaultTwice);
    t.label[at] = labels[i];
    // ancestors, up to one that another leaf has entered
    for (; l > 0; --l) {
        const uint64_t p = parent_key(T, l, q, c);
        if (insert(t.inner, t.inner_cap, p, &fresh) < 0) return fault(f, kFaultChildren);
        if (!fresh) return;
        int pl;
        split_key(p, pl, q, c);
    }
}

// What the tables say of `key`: its label for a leaf, -2 and *refined for an
// inner tetrahedron; `missing` is the fault where it is neither.
__device__ __forceinline__ int32_t look_up(const ImportTables &t, uint64_t key, int missing, bool *refined,
                                           ImportFaults *f) {
    const int64_t at = find(t.leaf, t.leaf_cap, key);
    *refined = find(t.inner, t.inner_cap, key) >= 0;
    if (at >= 0 && *refined) fault(f, kFaultBoth);
    if (at < 0 && !*refined) fault(f, missing);
    return at >= 0 ? t.label[at] : -2;
}

__global__ void k_import_lattice(LevelPtrs L, LatticeGeom g, int64_t n0, ImportTables t, ImportFaults *f) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n0) return;
    bool refined;
    L.label[0][i] = look_up(t, entry_key(L, g, 0, i), kFaultCover, &refined, f);
    L.child[0][i] = -1;
    L.flag[0][i] = refined ? 1 : 0;
}

// The children of the refined level-l entries list[0 .. count): block b of the
// next level for the b-th.
__global__ void k_import_children(LevelPtrs L, LatticeGeom g, ChildTables T, int l, const int32_t *__restrict__ list,
                                  int64_t count, ImportTables t, ImportFaults *f) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 8 * count) return;
    const int64_t b = i >> 3;
    const int r = (int)(i & 7), e = list[b];
    int pl, q;
    int64_t c[3];
    split_key(entry_key(L, g, l, e), pl, q, c);
    const int code = T.list[q][r][0], cq = T.list[q][r][1];
    const uint64_t key = make_key(l + 1, cq, 2 * c[0] + (code & 1), 2 * c[1] + ((code >> 1) & 1),
                                  2 * c[2] + ((code >> 2) & 1));
    bool refined;
    L.key[l + 1][i] = key;
    L.label[l + 1][i] = look_up(t, key, kFaultChildren, &refined, f);
    L.child[l + 1][i] = -1;
    L.flag[l + 1][i] = refined ? 1 : 0;
    if (r == 0) L.child[l][e] = (int32_t)b;
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

hipError_t launch_import_insert(const uint64_t *keys, const int32_t *labels, int64_t n, const LatticeGeom &g,
                                const ChildTables &T, const ImportTables &t, ImportFaults *f, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    k_import_insert<<<blocks_for(n), 256, 0, s>>>(keys, labels, n, g, T, t, f);
    return hipGetLastError();
}

hipError_t launch_import_lattice(const LevelPtrs &L, const LatticeGeom &g, int64_t n0, const ImportTables &t,
                                 ImportFaults *f, hipStream_t s) {
    k_import_lattice<<<blocks_for(n0), 256, 0, s>>>(L, g, n0, t, f);
    return hipGetLastError();
}

hipError_t launch_import_children(const LevelPtrs &L, const LatticeGeom &g, const ChildTables &T, int l,
                                  const int32_t *list, int64_t count, const ImportTables &t, ImportFaults *f,
                                  hipStream_t s) {
    if (count <= 0) return hipSuccess;
    k_import_children<<<blocks_for(8 * count), 256, 0, s>>>(L, g, T, l, list, count, t, f);
    return hipGetLastError();
}

}  // namespace sal
