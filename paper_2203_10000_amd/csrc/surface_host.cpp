// Host side of surface-set construction, with no device call: validation
// of closed oriented manifolds, the patch tree with its caps, the triangle
// records and the per-surface table.  Kept apart from the
// upload so that validation runs (and is tested) without a GPU.
#include <algorithm>
#include <array>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "surface_host.h"

namespace sal {

namespace {

struct HostSurface {
    const float *xyz;
    int64_t nv, nt;
    std::vector<int32_t> tri;  // possibly reoriented copy
    int32_t label;
    // Half-edge 3 t + c runs from corner c of triangle t to the next corner;
    // twin[h] is the opposite half-edge.
    std::vector<uint32_t> twin;

    int32_t from(uint32_t h) const { return tri[h]; }
    int32_t to(uint32_t h) const { return tri[h % 3 == 2 ? h - 2 : h + 1]; }
};

// A directed edge used twice among the first n_tri triangles?
bool repeated_edge(const HostSurface &s, int64_t n_tri) {
    std::vector<uint64_t> e;
    e.reserve((size_t)(3 * n_tri));
    for (uint32_t h = 0; h < (uint32_t)(3 * n_tri); ++h)
        e.push_back(((uint64_t)(uint32_t)s.from(h) << 32) | (uint32_t)s.to(h));
    std::sort(e.begin(), e.end());
    return std::adjacent_find(e.begin(), e.end()) != e.end();
}

enum class Pairing { ok, repeated, open };

// Fills s.twin: the half-edges leaving each vertex, sorted by their other
// end (a counting sort by vertex, then short sorts), hold each directed edge
// once exactly when neighbours in a list differ.
Pairing pair_half_edges(HostSurface &s) {
    const uint32_t nh = (uint32_t)(3 * s.nt);
    std::vector<uint32_t> start((size_t)s.nv + 1, 0);
    for (uint32_t h = 0; h < nh; ++h) ++start[(size_t)s.from(h) + 1];
    for (int64_t v = 0; v < s.nv; ++v) start[(size_t)v + 1] += start[(size_t)v];
    struct Out {
        int32_t to;
        uint32_t h;
    };
    std::vector<Out> out((size_t)nh);
    {
        std::vector<uint32_t> at(start.begin(), start.end() - 1);
        for (uint32_t h = 0; h < nh; ++h) out[at[(size_t)s.from(h)]++] = Out{s.to(h), h};
    }
    for (int64_t v = 0; v < s.nv; ++v) {
        Out *b = out.data() + start[(size_t)v], *e = out.data() + start[(size_t)v + 1];
        if (e - b <= 16) {
            for (Out *i = b + 1; i < e; ++i) {
                const Out x = *i;
                Out *j = i;
                for (; j > b && x.to < (j - 1)->to; --j) *j = *(j - 1);
                *j = x;
            }
        } else {
            std::sort(b, e, [](const Out &x, const Out &y) { return x.to < y.to; });
        }
        for (Out *i = b + 1; i < e; ++i)
            if (i->to == (i - 1)->to) return Pairing::repeated;
    }
    s.twin.assign((size_t)nh, 0);
    for (int64_t v = 0; v < s.nv; ++v)
        for (uint32_t i = start[(size_t)v]; i < start[(size_t)v + 1]; ++i) {
            const int32_t w = out[i].to;
            const Out *b = out.data() + start[(size_t)w], *e = out.data() + start[(size_t)w + 1];
            if (e - b > 16) {
                b = std::lower_bound(b, e, (int32_t)v, [](const Out &x, int32_t t) { return x.to < t; });
            } else {
                while (b < e && b->to < v) ++b;
            }
            if (b == e || b->to != v) return Pairing::open;
            s.twin[out[i].h] = b->h;
        }
    return Pairing::ok;
}

sal_status validate(HostSurface &s, int idx, bool auto_orient) {
    const std::string who = "surface " + std::to_string(idx) + ": ";
    if (s.nv < 3 || s.nt < 4 || !s.xyz || s.tri.empty())
        return set_error(SAL_ERR_INVALID_ARG, who + "needs >= 3 vertices and >= 4 triangles");
    if (s.label <= 0) return set_error(SAL_ERR_INVALID_ARG, who + "label must be > 0");
    if (s.nt > (int64_t)1 << 30 || s.nv > (int64_t)1 << 30)
        return set_error(SAL_ERR_CAPACITY, who + "more than 2^30 vertices or triangles");
    for (int64_t i = 0; i < 3 * s.nv; ++i)
        if (!std::isfinite(s.xyz[i]))
            return set_error(SAL_ERR_INVALID_ARG, who + "non-finite vertex coordinate");
    const std::string twice = who + "a directed edge is used twice";
    for (int64_t t = 0; t < s.nt; ++t) {
        const int32_t *f = &s.tri[3 * t];
        const char *bad = nullptr;
        for (int c = 0; c < 3 && !bad; ++c)
            if (f[c] < 0 || f[c] >= s.nv) bad = "vertex index out of range";
        if (!bad && (f[0] == f[1] || f[1] == f[2] || f[0] == f[2])) bad = "triangle repeats a vertex";
        if (!bad) {
            const float *A = s.xyz + 3 * f[0], *B = s.xyz + 3 * f[1], *C = s.xyz + 3 * f[2];
            const double e1[3] = {(double)B[0] - A[0], (double)B[1] - A[1], (double)B[2] - A[2]};
            const double e2[3] = {(double)C[0] - A[0], (double)C[1] - A[1], (double)C[2] - A[2]};
            const double n[3] = {e1[1] * e2[2] - e1[2] * e2[1], e1[2] * e2[0] - e1[0] * e2[2],
                                 e1[0] * e2[1] - e1[1] * e2[0]};
            if (n[0] == 0.0 && n[1] == 0.0 && n[2] == 0.0) bad = "zero-area triangle";
        }
        if (bad) {   // the first fault in triangle order is the one reported
            if (repeated_edge(s, t)) return set_error(SAL_ERR_NOT_CLOSED, twice);
            return set_error(SAL_ERR_INVALID_ARG, who + bad);
        }
    }
    Pairing p = pair_half_edges(s);
    if (p == Pairing::repeated) return set_error(SAL_ERR_NOT_CLOSED, twice);
    if (p == Pairing::open)
        return set_error(SAL_ERR_NOT_CLOSED, who + "boundary edge (surface is open)");
    // enclosed volume, about the vertex centroid for accuracy
    double c[3] = {0, 0, 0};
    for (int64_t i = 0; i < s.nv; ++i)
        for (int d = 0; d < 3; ++d) c[d] += s.xyz[3 * i + d];
    for (int d = 0; d < 3; ++d) c[d] /= (double)s.nv;
    double vol = 0.0;
    for (int64_t t = 0; t < s.nt; ++t) {
        const int32_t *f = &s.tri[3 * t];
        double v[3][3];
        for (int r = 0; r < 3; ++r)
            for (int d = 0; d < 3; ++d) v[r][d] = (double)s.xyz[3 * (int64_t)f[r] + d] - c[d];
        vol += v[0][0] * (v[1][1] * v[2][2] - v[1][2] * v[2][1]) +
               v[0][1] * (v[1][2] * v[2][0] - v[1][0] * v[2][2]) +
               v[0][2] * (v[1][0] * v[2][1] - v[1][1] * v[2][0]);
    }
    if (!(vol != 0.0)) return set_error(SAL_ERR_ORIENTATION, who + "encloses zero volume");
    if (vol < 0.0) {
        if (!auto_orient)
            return set_error(SAL_ERR_ORIENTATION,
                             who + "triangles are clockwise seen from outside (negative volume)");
        for (int64_t t = 0; t < s.nt; ++t) std::swap(s.tri[3 * t + 1], s.tri[3 * t + 2]);
        (void)pair_half_edges(s);   // reversed edges pair as before
    }
    return SAL_OK;
}

// Builds one surface's patch tree: the order of its triangles and the caps.
class PatchBuilder {
public:
    explicit PatchBuilder(const HostSurface &s) : s_(s) {}

    typedef std::array<int32_t, 3> Corners;

    std::vector<int32_t> order;       // triangles, leaf by leaf: their records
    std::vector<Corners> caps;        // the caps' triangles, patch by patch: the records after
    std::vector<PatchEntry> entries;  // 4 per node
    std::vector<LeafBox> leaves;      // in record order, then their groups

    void build() {
        const int64_t nt = s_.nt;
        order.resize((size_t)nt);
        cen_.resize((size_t)(3 * nt));
        for (int64_t t = 0; t < nt; ++t) {
            order[(size_t)t] = (int32_t)t;
            for (int c = 0; c < 3; ++c) {
                float sum = 0.0f;
                for (int q = 0; q < 3; ++q) sum += s_.xyz[3 * (int64_t)s_.tri[(size_t)(3 * t + q)] + c] / 3.0f;
                cen_[(size_t)(3 * t + c)] = sum;
            }
        }
        pos_.assign((size_t)nt, -1);
        first_out_.assign((size_t)s_.nv, -1);
        on_path_.assign((size_t)s_.nv, -1);
        new_node();
        std::vector<uint32_t> none;
        if (nt <= kLeafTri) leaf(0, 0, nt, &none);
        else split(0, 0, nt, &none);
        const size_t n = leaves.size();
        for (size_t b = 0; b < n; b += kLeafGroup) {
            LeafBox g = leaves[b];
            g.begin = (uint32_t)b;
            g.count = (uint32_t)std::min<size_t>(kLeafGroup, n - b);
            for (size_t i = b + 1; i < b + g.count; ++i)
                for (int c = 0; c < 3; ++c) {
                    g.lo[c] = std::min(g.lo[c], leaves[i].lo[c]);
                    g.hi[c] = std::max(g.hi[c], leaves[i].hi[c]);
                }
            leaves.push_back(g);
        }
        n_leaves = (int64_t)n;
    }
    int64_t n_leaves = 0;

private:
    struct Box {
        float lo[3], hi[3];
    };

    int32_t new_node() {
        const int32_t w = (int32_t)(entries.size() / 4);
        PatchEntry unused{};
        for (int c = 0; c < 3; ++c) {
            unused.lo[c] = INFINITY;
            unused.hi[c] = -INFINITY;
        }
        unused.child = -1;
        entries.insert(entries.end(), 4, unused);
        return w;
    }

    // Halves order[b, e) at the median of the centroids' longest extent.
    int64_t halve(int64_t b, int64_t e) {
        float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
        for (int64_t i = b; i < e; ++i)
            for (int c = 0; c < 3; ++c) {
                const float x = cen_[3 * (size_t)order[(size_t)i] + c];
                lo[c] = std::min(lo[c], x);
                hi[c] = std::max(hi[c], x);
            }
        int ax = 0;
        for (int c = 1; c < 3; ++c)
            if (hi[c] - lo[c] > hi[ax] - lo[ax]) ax = c;
        const int64_t m = b + (e - b) / 2;
        std::nth_element(order.begin() + b, order.begin() + m, order.begin() + e,
                         [&](int32_t p, int32_t q) {
                             const float x = cen_[3 * (size_t)p + ax], y = cen_[3 * (size_t)q + ax];
                             return x != y ? x < y : p < q;
                         });
        return m;
    }

    // Parts of order[b, e) (more than a leaf): the entries of node w.  The
    // patch's boundary half-edges go to *rim, its box is returned.
    Box split(int32_t w, int64_t b, int64_t e, std::vector<uint32_t> *rim) {
        int64_t cut[5] = {b, 0, 0, 0, 0};
        int parts = 0;
        const int64_t m = halve(b, e);
        const int64_t half[2][2] = {{b, m}, {m, e}};
        for (const auto &h : half) {
            if (h[1] - h[0] > kLeafTri) cut[++parts] = halve(h[0], h[1]);
            cut[++parts] = h[1];
        }
        std::vector<uint32_t> edges;
        Box box = no_box();
        for (int k = 0; k < parts; ++k) {
            const size_t ent = 4 * (size_t)w + (size_t)k;
            std::vector<uint32_t> part_rim;
            Box pb;
            if (cut[k + 1] - cut[k] <= kLeafTri) {
                pb = leaf(ent, cut[k], cut[k + 1], &part_rim);
            } else {
                const int32_t child = new_node();
                pb = split(child, cut[k], cut[k + 1], &part_rim);
                entries[ent].child = child;
                cap(ent, part_rim, cut[k], cut[k + 1] - cut[k]);
                set_box(ent, pb);
            }
            for (int c = 0; c < 3; ++c) {
                box.lo[c] = std::min(box.lo[c], pb.lo[c]);
                box.hi[c] = std::max(box.hi[c], pb.hi[c]);
            }
            edges.insert(edges.end(), part_rim.begin(), part_rim.end());
        }
        for (const uint32_t h : edges) {
            const int64_t at = pos_[s_.twin[h] / 3];   // (-1: in a patch still to come)
            if (at < b || at >= e) rim->push_back(h);
        }
        return box;
    }

    static Box no_box() {
        return Box{{INFINITY, INFINITY, INFINITY}, {-INFINITY, -INFINITY, -INFINITY}};
    }

    Box leaf(size_t ent, int64_t b, int64_t e, std::vector<uint32_t> *rim) {
        Box box = no_box();
        std::sort(order.begin() + b, order.begin() + e);
        for (int64_t i = b; i < e; ++i) {
            const int32_t t = order[(size_t)i];
            pos_[(size_t)t] = (int32_t)i;
            for (int q = 0; q < 3; ++q)
                for (int c = 0; c < 3; ++c) {
                    const float x = s_.xyz[3 * (int64_t)s_.tri[3 * (size_t)t + q] + c];
                    box.lo[c] = std::min(box.lo[c], x);
                    box.hi[c] = std::max(box.hi[c], x);
                }
        }
        for (int64_t i = b; i < e; ++i)
            for (int c = 0; c < 3; ++c) {
                const uint32_t h = 3 * (uint32_t)order[(size_t)i] + (uint32_t)c;
                const int64_t at = pos_[s_.twin[h] / 3];
                if (at < b || at >= e) rim->push_back(h);
            }
        LeafBox lb;
        for (int c = 0; c < 3; ++c) {
            lb.lo[c] = box.lo[c];
            lb.hi[c] = box.hi[c];
        }
        lb.begin = (uint32_t)b;
        lb.count = (uint32_t)(e - b);
        leaves.push_back(lb);
        cap(ent, *rim, b, e - b);
        set_box(ent, box);
        return box;
    }

    void set_box(size_t ent, const Box &box) {
        double ext = 0.0;
        for (int c = 0; c < 3; ++c) ext = std::max(ext, (double)box.hi[c] - box.lo[c]);
        const double m = kCapMargin * ext;
        for (int c = 0; c < 3; ++c) {
            entries[ent].lo[c] = std::nextafterf((float)(box.lo[c] - m), -INFINITY);
            entries[ent].hi[c] = std::nextafterf((float)(box.hi[c] + m), INFINITY);
        }
    }

    // The record ranges of a patch, triangles [begin, begin + n_tri), and its cap:
    // the boundary half-edges `rim` are cut into simple loops, each closed by a
    // zigzag with the patch's own direction along the loop.  A cap no shorter
    // than the patch is not kept.
    void cap(size_t ent, const std::vector<uint32_t> &rim, int64_t begin, int64_t n_tri) {
        PatchEntry &pe = entries[ent];
        pe.leaf_begin = (uint32_t)begin;
        pe.leaf_n = (uint32_t)n_tri;
        pe.cap_begin = pe.leaf_begin;
        pe.cap_n = pe.leaf_n;
        if ((int64_t)rim.size() >= n_tri) return;
        const size_t cap0 = caps.size();
        next_out_.assign(rim.size(), -1);
        for (size_t i = 0; i < rim.size(); ++i) {
            int32_t &head = first_out_[(size_t)s_.from(rim[i])];
            next_out_[i] = head;
            head = (int32_t)i;
        }
        std::vector<int32_t> path;
        for (size_t i = 0; i < rim.size(); ++i) {
            const int32_t v0 = s_.from(rim[i]);
            if (first_out_[(size_t)v0] < 0) continue;
            path.assign(1, v0);
            on_path_[(size_t)v0] = 0;
            for (;;) {
                const int32_t v = path.back();
                const int32_t e = first_out_[(size_t)v];
                if (e < 0) break;   // only v0 can run out: every loop through it is closed
                first_out_[(size_t)v] = next_out_[(size_t)e];
                const int32_t w = s_.to(rim[(size_t)e]);
                const int32_t k = on_path_[(size_t)w];
                if (k < 0) {
                    on_path_[(size_t)w] = (int32_t)path.size();
                    path.push_back(w);
                    continue;
                }
                zigzag(path.data() + k, (int64_t)path.size() - k);
                while ((int32_t)path.size() > k + 1) {
                    on_path_[(size_t)path.back()] = -1;
                    path.pop_back();
                }
            }
            for (const int32_t v : path) on_path_[(size_t)v] = -1;
        }
        pe.cap_begin = (uint32_t)(s_.nt + (int64_t)cap0);
        pe.cap_n = (uint32_t)(caps.size() - cap0);
    }

    // Loop v_0 -> v_1 -> ... -> v_{L-1}: the strip v_0, v_1, v_{L-1}, v_2, v_{L-2},
    // ...; its even triangles are outward in strip order, its odd ones reversed.
    void zigzag(const int32_t *v, int64_t L) {
        int64_t i = 1, j = L - 1;
        int32_t x = v[0], y = v[1];
        for (int64_t t = 0; t < L - 2; ++t) {
            const int32_t z = (t & 1) == 0 ? v[j--] : v[++i];
            if ((t & 1) == 0) caps.push_back({x, y, z});
            else caps.push_back({x, z, y});
            x = y;
            y = z;
        }
    }

    const HostSurface &s_;
    std::vector<float> cen_;
    std::vector<int32_t> pos_;        // a triangle's place in `order` once its leaf is built
    std::vector<int32_t> first_out_, next_out_, on_path_;
};

// Squared distance from p to triangle (a, b, c), in double: the closest
// point found by the Voronoi-region walk over vertices, edges and face
// (Ericson, Real-Time Collision Detection, section 5.1.5).
double dist2_point_triangle(const double p[3], const double a[3], const double b[3], const double c[3]) {
    auto sub = [](const double *u, const double *v, double *o) {
        for (int k = 0; k < 3; ++k) o[k] = u[k] - v[k];
    };
    auto dot = [](const double *u, const double *v) { return u[0] * v[0] + u[1] * v[1] + u[2] * v[2]; };
    double ab[3], ac[3], ap[3], q[3];
    sub(b, a, ab);
    sub(c, a, ac);
    sub(p, a, ap);
    const double d1 = dot(ab, ap), d2 = dot(ac, ap);
    auto at = [&](double u, double v) {   // a + u ab + v ac
        for (int k = 0; k < 3; ++k) q[k] = a[k] + u * ab[k] + v * ac[k];
    };
    if (d1 <= 0 && d2 <= 0) {
        at(0, 0);
    } else {
        double bp[3];
        sub(p, b, bp);
        const double d3 = dot(ab, bp), d4 = dot(ac, bp);
        if (d3 >= 0 && d4 <= d3) {
            at(1, 0);
        } else {
            const double vc = d1 * d4 - d3 * d2;
            if (vc <= 0 && d1 >= 0 && d3 <= 0) {
                at(d1 / (d1 - d3), 0);
            } else {
                double cp[3];
                sub(p, c, cp);
                const double d5 = dot(ab, cp), d6 = dot(ac, cp);
                if (d6 >= 0 && d5 <= d6) {
                    at(0, 1);
                } else {
                    const double vb = d5 * d2 - d1 * d6;
                    if (vb <= 0 && d2 >= 0 && d6 <= 0) {
                        at(0, d2 / (d2 - d6));
                    } else {
                        const double va = d3 * d6 - d5 * d4;
                        if (va <= 0 && (d4 - d3) >= 0 && (d5 - d6) >= 0) {
                            const double w = (d4 - d3) / ((d4 - d3) + (d5 - d6));
                            at(1 - w, w);
                        } else {
                            const double den = 1.0 / (va + vb + vc);
                            at(vb * den, vc * den);
                        }
                    }
                }
            }
        }
    }
    double d[3];
    sub(p, q, d);
    return dot(d, d);
}

TriRec record(const float *V, int32_t a, int32_t b, int32_t c) {
    const float *A = V + 3 * (int64_t)a, *B = V + 3 * (int64_t)b, *C = V + 3 * (int64_t)c;
    const double e1[3] = {(double)B[0] - A[0], (double)B[1] - A[1], (double)B[2] - A[2]};
    const double e2[3] = {(double)C[0] - A[0], (double)C[1] - A[1], (double)C[2] - A[2]};
    const double n[3] = {e1[1] * e2[2] - e1[2] * e2[1], e1[2] * e2[0] - e1[0] * e2[2],
                         e1[0] * e2[1] - e1[1] * e2[0]};
    TriRec r;
    for (int k = 0; k < 3; ++k) {
        r.v[k] = A[k];
        r.v[4 + k] = B[k];
        r.v[8 + k] = C[k];
        r.v[4 * k + 3] = (float)(kNScale * n[k]);
    }
    return r;
}

}  // namespace


sal_status build_surface_records(const sal_surface_desc *desc, int32_t n, uint32_t flags,
                                 SurfaceRecords *rec) {
    if (!desc || !rec) return set_error(SAL_ERR_INVALID_ARG, "NULL argument");
    if (n < 1 || n > kMaxSurfaces)
        return set_error(SAL_ERR_INVALID_ARG, "n_surfaces must be in 1..64");
    std::vector<TriRec> &recs = rec->recs;
    std::vector<SurfaceDev> &table = rec->table;
    std::vector<PatchEntry> &entries = rec->entries;
    recs.clear();
    entries.clear();
    rec->leaves.clear();
    rec->n_leaves = 0;
    table.assign((size_t)n, SurfaceDev{});
    int64_t &total_tri = rec->total_tri;
    total_tri = 0;
    for (int32_t i = 0; i < n; ++i) {
        HostSurface hs;
        hs.xyz = desc[i].xyz;
        hs.nv = desc[i].n_vertices;
        hs.nt = desc[i].n_triangles;
        hs.label = desc[i].label;
        if (hs.nt < 4 || !desc[i].tri || !desc[i].xyz)
            return set_error(SAL_ERR_INVALID_ARG,
                             "surface " + std::to_string(i) + ": needs >= 4 triangles");
        hs.tri.assign(desc[i].tri, desc[i].tri + 3 * hs.nt);
        sal_status st = validate(hs, i, (flags & SAL_SURF_AUTO_ORIENT) != 0);
        if (st != SAL_OK) return st;
        PatchBuilder patches(hs);
        patches.build();
        SurfaceDev &sd = table[(size_t)i];
        sd.rec_begin = (int64_t)recs.size();
        sd.n_tri = hs.nt;
        sd.label = hs.label;
        sd.leaf_begin = (int64_t)rec->leaves.size();
        sd.n_leaves = (int32_t)patches.n_leaves;
        rec->leaves.insert(rec->leaves.end(), patches.leaves.begin(), patches.leaves.end());
        for (int c = 0; c < 3; ++c) {
            sd.lo[c] = INFINITY;
            sd.hi[c] = -INFINITY;
        }
        for (int64_t v = 0; v < hs.nv; ++v)
            for (int c = 0; c < 3; ++c) {
                sd.lo[c] = std::min(sd.lo[c], hs.xyz[3 * v + c]);
                sd.hi[c] = std::max(sd.hi[c], hs.xyz[3 * v + c]);
            }
        // a ball about the vertex mean (rounded to float) that the surface
        // does not cross: radius = distance to the nearest triangle, less a
        // margin far above the rounding of the device's float distance test
        {
            double m[3] = {0, 0, 0};
            for (int64_t v = 0; v < hs.nv; ++v)
                for (int c = 0; c < 3; ++c) m[c] += hs.xyz[3 * v + c];
            double cen[3];
            for (int c = 0; c < 3; ++c) {
                sd.ball[c] = (float)(m[c] / (double)hs.nv);
                cen[c] = sd.ball[c];
            }
            double r2 = INFINITY;
            for (int64_t t = 0; t < hs.nt; ++t) {
                double P[3][3];
                for (int q = 0; q < 3; ++q)
                    for (int c = 0; c < 3; ++c) P[q][c] = hs.xyz[3 * (int64_t)hs.tri[3 * t + q] + c];
                r2 = std::min(r2, dist2_point_triangle(cen, P[0], P[1], P[2]));
            }
            const double scale = std::max({std::fabs(cen[0]), std::fabs(cen[1]), std::fabs(cen[2])});
            const double r = std::sqrt(r2) - 1e-5 * (std::sqrt(r2) + scale);
            sd.ball[3] = r > 0 ? (float)(r * r * (1.0 - 1e-6)) : 0.0f;
            sd.ball_w = -1;   // set by ensure_surface_balls, on first use
            sd.pad2 = 0;
        }
        total_tri += hs.nt;
        recs.reserve(recs.size() + patches.order.size() + patches.caps.size());
        for (const int32_t t : patches.order)
            recs.push_back(record(hs.xyz, hs.tri[3 * (size_t)t], hs.tri[3 * (size_t)t + 1], hs.tri[3 * (size_t)t + 2]));
        sd.rec_end = (int64_t)recs.size();
        for (const auto &c : patches.caps) recs.push_back(record(hs.xyz, c[0], c[1], c[2]));
        rec->n_leaves += patches.n_leaves;
        sd.node_begin = (int64_t)(entries.size() / 4);
        entries.insert(entries.end(), patches.entries.begin(), patches.entries.end());
    }
    return SAL_OK;
}

}  // namespace sal

extern "C" sal_status sal_surface_set_check(const sal_surface_desc *surfaces, int32_t n_surfaces,
                                            uint32_t flags, sal_surface_set_info *info) {
    try {
        sal::SurfaceRecords rec;
        const sal_status st = sal::build_surface_records(surfaces, n_surfaces, flags, &rec);
        if (st != SAL_OK) return st;
        if (info) {
            info->n_surfaces = n_surfaces;
            info->n_triangles = rec.total_tri;
            info->n_strips = rec.n_leaves;
            info->device_bytes = (int64_t)(rec.recs.size() * sizeof(sal::TriRec) +
                                           rec.table.size() * sizeof(sal::SurfaceDev) +
                                           rec.entries.size() * sizeof(sal::PatchEntry) +
                                           rec.leaves.size() * sizeof(sal::LeafBox));
        }
        return SAL_OK;
    } catch (const std::bad_alloc &) {
        return sal::set_error(SAL_ERR_OUT_OF_MEMORY, "host allocation failed");
    } catch (...) {
        return sal::set_error(SAL_ERR_INTERNAL, "exception in sal_surface_set_check");
    }
}
