// Host-only surface-set construction (no device calls).
#pragma once

#include <cstdint>
#include <vector>

#include "sal_internal.h"

namespace sal {

// Everything a surface set uploads: triangle records (each surface's
// triangles, then its caps), the patch trees and the per-surface table.
struct SurfaceRecords {
    std::vector<TriRec> recs;
    std::vector<SurfaceDev> table;
    std::vector<PatchEntry> entries;   // four per node
    std::vector<LeafBox> leaves;       // and their groups, surface by surface
    int64_t total_tri = 0, n_leaves = 0;
};

// Validates the surfaces (section 2.1.3: closed, consistently oriented
// boundaries; SAL_SURF_AUTO_ORIENT reverses inward ones) and builds their
// records.  Errors as sal_surface_set_create's, with nothing built.
sal_status build_surface_records(const sal_surface_desc *desc, int32_t n, uint32_t flags,
                                 SurfaceRecords *rec);

}  // namespace sal
