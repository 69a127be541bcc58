// Tetrahedral-mesh data shared by the mesh kernels (mesh.hip) and the host
// orchestration (mesh.cpp).
#pragma once

#include "sal_internal.h"

namespace sal {

constexpr int kMaxLevels = 3;   // refinement levels 1..3 above the lattice

// Per-level arrays.  Level 0 is the lattice (keys implicit from the index);
// level l >= 1 holds blocks of 8 children appended in split order.
//   child[l][i] = -1 for a leaf, else b: its children are level l+1 entries
//   8b .. 8b+7 (in the order of ChildTables::list).
struct LevelPtrs {
    uint64_t *key[kMaxLevels + 1];
    int32_t *label[kMaxLevels + 1];
    int32_t *child[kMaxLevels + 1];
    uint8_t *flag[kMaxLevels + 1];
    int64_t n[kMaxLevels + 1];
    const int64_t *n_dev;   // device copy of the level sizes; when set it replaces n
    int inherit;            // splits give the children their parent's label
};

// Per-round figures kept on the device by the captured refine round.
struct RoundStat {
    int64_t n_leaves, n_boundary, n_labeled, n_recheck_pairs;
};

// Device-resident state of the captured refine round: every size the round
// needs lives here, so one captured graph serves every round.  The plan step
// turns `status` nonzero (sticky) instead of writing past a capacity; the
// steps that change the mesh then do nothing.
struct RoundState {
    int64_t n[kMaxLevels + 1];           // entries per level
    int64_t cap[kMaxLevels + 1];         // capacity per level
    int64_t base_block[kMaxLevels + 1];  // first child block of each level's splits
    int64_t kid_off[kMaxLevels + 1];     // each level's children in the labeling scratch
    int64_t n_kids;                      // children made this round
    int64_t kid_cap;                     // labeling scratch capacity
    int64_t n_leaves;
    int32_t status;                      // 0 ok, 1 out of capacity, 2 beyond the deepest level
    int32_t round;                       // rounds completed
    RoundStat stat[kMaxLevels + 1];
};

// A launch over levels 0..top, usually of the entries [first[l], n[l]) of level l.
struct LevelSpans {
    int top;
    int64_t first[kMaxLevels + 1], n[kMaxLevels + 1];
    uint32_t block0[kMaxLevels + 2];   // first workgroup (this and `turns` set by with_blocks)
    int turns;                         // items of a thread
};

// Workgroups of 256 for per[l] items of level l, a level's first one its own.
inline LevelSpans with_blocks(LevelSpans r, const int64_t (&per)[kMaxLevels + 1], int turns, int64_t *blocks) {
    int64_t nb = 0;
    r.turns = turns;
    for (int l = 0; l <= kMaxLevels; ++l) {
        r.block0[l] = (uint32_t)nb;
        if (l <= r.top) nb += (per[l] + 256 * turns - 1) / (256 * turns);
    }
    r.block0[kMaxLevels + 1] = (uint32_t)nb;
    *blocks = nb;
    return r;
}

struct LatticeGeom {
    double origin[3];
    double h;
    int32_t cells[3];
};

// Children of a tetrahedron with permutation index q: list[q][r] = (sub-cell
// code dx + 2 dy + 4 dz, child q') for r = 0..7; rank[q][code][q'] = r or -1.
struct ChildTables {
    int8_t list[6][8][2];
    int8_t rank[6][8][6];
};

// Source of a compaction: nonzero flags, or leaves (child < 0).
struct CompactSrc {
    const uint8_t *flag;    // entries with flag & mask != 0 (mask 0: any bit) ...
    const int32_t *child;   // ... or, without flag, the leaves (child < 0)
    uint8_t mask;
};

hipError_t launch_lattice_centroids(const LatticeGeom &g, int64_t n0, float *cx, float *cy,
                                    float *cz, hipStream_t s);
// Clears the flags of levels 0..top (size[l] entries, or L.n_dev[l] of them), the
// label counters, the new nodes' counters (n_new, may be null) and the kids' count
// (rs, may be null); then marks.
hipError_t launch_round_clear(const LevelPtrs &L, int top, const int64_t *size, unsigned long long *counters,
                              unsigned long long *n_new, RoundState *rs, hipStream_t s);
hipError_t launch_mark(const LevelPtrs &L, const LatticeGeom &g, const ChildTables &T, int top,
                       const int64_t *size, hipStream_t s);
int64_t compact_blocks(int64_t n);
hipError_t launch_compact(const CompactSrc &src, int64_t n, int64_t *block_scratch,
                          int64_t *total, int32_t *out, hipStream_t s);
// One compaction over levels 0..top, a level's list behind the one before it in
// `out`: the leaves, or (mask != 0) the entries with a flag bit of mask.  Writes
// the levels' totals and the *extra word to totals[0..kMaxLevels + 1] and, once the
// stream has got there, to the same places of host_words (pinned memory).
// (Device-sized, with L.n_dev: size[l] bounds a level's entries, host_words is null.)
int64_t compact_level_blocks(const int64_t *size, int top);
hipError_t launch_compact_levels(const LevelPtrs &L, int top, const int64_t *size, uint8_t mask,
                                 int64_t *block_scratch,
                                 int64_t *totals, const unsigned long long *extra, int64_t *host_words,
                                 int32_t *out, hipStream_t s);
hipError_t launch_split(const LevelPtrs &L, const LatticeGeom &g, const ChildTables &T, int l,
                        const int32_t *list, int64_t count, int64_t base_block, float *cx,
                        float *cy, float *cz, hipStream_t s);
hipError_t launch_export(const LevelPtrs &L, const LatticeGeom &g, int l, const int32_t *list,
                         int64_t count, int64_t out_base, uint64_t *keys, int32_t *labels,
                         float *cx, float *cy, float *cz, hipStream_t s);
// Device-sized forms for the captured refine round (sizes read from
// RoundState / compaction totals; fixed grids stride over them).
hipError_t launch_round_state(RoundState *rs, const RoundState &first, hipStream_t s);
hipError_t launch_plan(RoundState *rs, const int64_t *totals, hipStream_t s);
hipError_t launch_split_dev(const LevelPtrs &L, const LatticeGeom &g, const ChildTables &T, const int32_t *list,
                            const int64_t *totals, const RoundState *rs, float *cx, float *cy, float *cz,
                            hipStream_t s);
hipError_t launch_commit(const LevelPtrs &L, const RoundState *rs, const int64_t *totals,
                         const int32_t *scratch_labels, hipStream_t s);
hipError_t launch_round_end(RoundState *rs, const unsigned long long *counters, hipStream_t s);

// Four-node rule (node enclosure masks).
hipError_t launch_lattice_nodes(const LatticeGeom &g, int64_t n_nodes, float *x, float *y, float *z,
                               hipStream_t s);
hipError_t launch_elem_from_nodes0(const LatticeGeom &g, int64_t n0,
                                   const unsigned long long *node0, const SurfaceDev *surf,
                                   int32_t *label0, hipStream_t s);
// Node table (open addressing; keys ~0 = empty; the host keeps it at most half
// full).  The midpoints of the listed leaves' edges: slot[6 j + e] is the table's
// place of leaf j's edge e; those not in it before are listed with their
// coordinates (new_slot, x, y, z; *n_new of them).
hipError_t launch_midpoints(const LevelPtrs &L, const LatticeGeom &g, int l, const int32_t *list,
                            int64_t count, unsigned long long *tkeys, int64_t cap, int64_t *slot,
                            int64_t *new_slot, unsigned long long *n_new, float *x, float *y, float *z,
                            hipStream_t s);
hipError_t launch_node_store(const int64_t *new_slot, const unsigned long long *n_new, int64_t n_cap,
                             const unsigned long long *masks, unsigned long long *tmasks, hipStream_t s);
hipError_t launch_node_rehash(const unsigned long long *okeys, const unsigned long long *omasks,
                              int64_t ocap, unsigned long long *tkeys, unsigned long long *tmasks,
                              int64_t cap, hipStream_t s);
hipError_t launch_child_masks(const LevelPtrs &L, const LatticeGeom &g, int l,
                              const int32_t *list, int64_t count, int64_t base_block,
                              const unsigned long long *node0,
                              const unsigned long long *vmask_parent,
                              const int64_t *slot, const unsigned long long *tmasks,
                              unsigned long long *vmask_child, const SurfaceDev *surf,
                              hipStream_t s);

// Conforming transition refinement (conform.hip).
// Flags of a leaf during the closure (in LevelPtrs::flag): bits 0-5 the
// hanging edges, bit 6 a node at a quarter point, bit 7 split 1 -> 8.
// cells_new: one bit per level-0 cell, set for the cells a vertex added to
// `fresh` touches (both null: the first pass).
hipError_t launch_closure_clear(unsigned long long *fresh, int64_t fcap, uint32_t *cells_new, int64_t cell_words,
                                hipStream_t s);
// n_new: accumulated, not cleared.  *overflow counts the keys that found no place.
hipError_t launch_insert_levels(const LevelPtrs &L, const LatticeGeom &g, const LevelSpans &r,
                                unsigned long long *set, int64_t cap, unsigned long long *fresh, int64_t fcap,
                                uint32_t *cells_new, unsigned long long *n_new, unsigned long long *overflow,
                                hipStream_t s);
// New patterns after a closure round: entries [0, first) of a level from the
// round's new vertices, entries [first, n) in full.
hipError_t launch_pattern_levels(const LevelPtrs &L, const LatticeGeom &g, const LevelSpans &r,
                                 const unsigned long long *set, int64_t cap, const unsigned long long *fresh,
                                 int64_t fcap, const uint32_t *cells_new, hipStream_t s);
// The conforming mesh: `list` holds the leaves level by level, n[l] of each.
// hist: 4 counters (leaves cut into 1, 2, 3, 4 tetrahedra), accumulated.
hipError_t launch_tet_counts(const LevelPtrs &L, const LevelSpans &r, const int32_t *list, int32_t *counts,
                             unsigned long long *hist, hipStream_t s);
// rocPRIM device-wide primitives: with tmp == nullptr they only set *tmp_bytes.
hipError_t exclusive_sum_i32(const int32_t *in, int64_t *out, int64_t n, void *tmp,
                             size_t *tmp_bytes, hipStream_t s);
// Nodes: the vertex set's keys with their 21-bit fields packed (`bits` per axis), in
// no order; sorted; numbered (keys, coordinates, and a table from packed key to
// number, cap a power of two).
struct NodeEntry {
    unsigned long long key;   // ~0: empty
    int32_t id, pad;
};
struct NodeBits {
    int y, z;   // of the two lower fields
};
hipError_t launch_set_keys(const unsigned long long *set, int64_t cap, const NodeBits &nb, uint64_t *out,
                           int64_t out_cap, unsigned long long *n_out, hipStream_t s);
hipError_t sort_packed(const uint64_t *in, uint64_t *out, int64_t n, int bits, void *tmp, size_t *tmp_bytes,
                       hipStream_t s);
hipError_t launch_number_nodes(const LatticeGeom &g, const uint64_t *packed, int64_t n, const NodeBits &nb,
                               NodeEntry *table, int64_t cap, int64_t *keys, float *xyz, hipStream_t s);
hipError_t launch_emit(const LevelPtrs &L, const LatticeGeom &g, const LevelSpans &r, const int32_t *list,
                       const int64_t *offsets, const NodeBits &nb, const NodeEntry *table, int64_t cap,
                       int32_t *ids, int32_t *labels, hipStream_t s);

// Checkpoint import (import.hip).
struct ImportTables {
    unsigned long long *leaf;    // [leaf_cap] keys of the leaves (open addressing, ~0 empty)
    int32_t *label;              // [leaf_cap]
    int64_t leaf_cap;
    unsigned long long *inner;   // [inner_cap] keys of the refined tetrahedra
    int64_t inner_cap;
};
// What is wrong with a leaf set.  first: (index << 2) | reason of the first leaf
// that is no leaf of the lattice (0: level or permutation, 1: outside, 2: no
// label), ~0 when there is none; bits: faults of the set as a whole.
struct ImportFaults {
    unsigned long long first;
    unsigned int bits, pad;
};
enum { kFaultTwice = 0, kFaultChildren = 1, kFaultBoth = 2, kFaultCover = 3 };
hipError_t launch_import_insert(const uint64_t *keys, const int32_t *labels, int64_t n, const LatticeGeom &g,
                                const ChildTables &T, const ImportTables &t, ImportFaults *f, hipStream_t s);
hipError_t launch_import_lattice(const LevelPtrs &L, const LatticeGeom &g, int64_t n0, const ImportTables &t,
                                 ImportFaults *f, hipStream_t s);
hipError_t launch_import_children(const LevelPtrs &L, const LatticeGeom &g, const ChildTables &T, int l,
                                  const int32_t *list, int64_t count, const ImportTables &t, ImportFaults *f,
                                  hipStream_t s);

// counters[kCntRecheck] and n_new[0..kMaxLevels) into pinned host memory.
hipError_t launch_report(const unsigned long long *counters, const unsigned long long *n_new,
                         int64_t *host_words, hipStream_t s);
hipError_t launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t s);
hipError_t launch_fill_u8(uint8_t *p, uint8_t v, int64_t n, hipStream_t s);

}  // namespace sal
