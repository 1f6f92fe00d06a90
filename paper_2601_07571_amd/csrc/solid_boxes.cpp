// solid_boxes.cpp -- boxes that lie wholly inside the scene's closed meshes, and a small
// tree over them, for the visibility test (host only, at scene creation).
//
// A box that no triangle of a closed mesh touches and whose points the mesh winds around
// (winding number not zero) separates: a segment from a point of it to any point outside the
// mesh's bounding box crosses the mesh.  So a segment that meets such a box on its way to an
// eye outside the mesh's box is occluded, whichever triangle does it, and needs no walk of
// the triangles (Sec. 3.2.2).
//
// Per mesh: a grid of about as many cells as the mesh has triangles; cells that a triangle's
// (widened) box meets are surface; the others form regions connected by their faces, inside
// each of which the winding number is constant, so one evaluation (the sum of the triangles'
// solid angles, van Oosterom and Strackee 1983) settles a region.  The cells of regions with
// a non-zero winding number are covered, largest cubes first, by boxes stretched as far as
// they go.  Nothing here is assumed about self-intersection or outward normals; only that
// the mesh has no boundary, which the caller has checked.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <limits>
#include <vector>

#include "gm_internal.h"

namespace gm {

namespace {

struct IBox {
    int lo[3], hi[3];  // cells, hi exclusive
};

struct Grid {
    int n[3];
    double org[3], cell;
    int64_t at(int x, int y, int z) const { return ((int64_t)z * n[1] + y) * n[0] + x; }
    int64_t size() const { return (int64_t)n[0] * n[1] * n[2]; }
};

// winding number of the mesh around p, in turns
double winding(const float* V, const int32_t* I, int64_t T, const double* p)
{
    double sum = 0.0;
    for (int64_t t = 0; t < T; ++t) {
        double a[3], b[3], c[3];
        for (int k = 0; k < 3; ++k) {
            a[k] = V[3 * (int64_t)I[3 * t] + k] - p[k];
            b[k] = V[3 * (int64_t)I[3 * t + 1] + k] - p[k];
            c[k] = V[3 * (int64_t)I[3 * t + 2] + k] - p[k];
        }
        const double la = std::sqrt(a[0] * a[0] + a[1] * a[1] + a[2] * a[2]);
        const double lb = std::sqrt(b[0] * b[0] + b[1] * b[1] + b[2] * b[2]);
        const double lc = std::sqrt(c[0] * c[0] + c[1] * c[1] + c[2] * c[2]);
        const double det = a[0] * (b[1] * c[2] - b[2] * c[1]) + a[1] * (b[2] * c[0] - b[0] * c[2]) +
                           a[2] * (b[0] * c[1] - b[1] * c[0]);
        const double ab = a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
        const double bc = b[0] * c[0] + b[1] * c[1] + b[2] * c[2];
        const double ca = c[0] * a[0] + c[1] * a[1] + c[2] * a[2];
        sum += std::atan2(det, la * lb * lc + ab * lc + bc * la + ca * lb);
    }
    return sum / (2.0 * M_PI);  // the solid angle is twice the arc tangent; 4 pi a turn
}

}  // namespace

double solid_boxes(const float* V, const int32_t* I, int64_t T, double scene_scale, int max_boxes, int32_t mesh,
                   std::vector<SolidBox>& out)
{
    const double none = std::numeric_limits<double>::infinity();
    if (T < 4 || max_boxes < 1) return none;
    double lo[3], hi[3], ext = 0.0;
    for (int a = 0; a < 3; ++a) {
        lo[a] = std::numeric_limits<double>::infinity();
        hi[a] = -lo[a];
    }
    for (int64_t i = 0; i < 3 * T; ++i)
        for (int a = 0; a < 3; ++a) {
            const double v = V[3 * (int64_t)I[i] + a];
            lo[a] = std::min(lo[a], v);
            hi[a] = std::max(hi[a], v);
        }
    for (int a = 0; a < 3; ++a) ext = std::max(ext, hi[a] - lo[a]);
    if (!(ext > 0.0)) return none;
    // the boxes keep this distance from every triangle: far above the rounding of the
    // device's FP32 slab test (a few 1e-7 of the coordinates)
    const double pad = 1e-4 * ext + 1e-5 * scene_scale;
    Grid g;
    const int res = (int)std::min(64.0, std::max(12.0, std::cbrt((double)T)));
    g.cell = ext / res;
    if (pad > 0.25 * g.cell) return none;
    for (int a = 0; a < 3; ++a) {
        g.n[a] = std::min(res, std::max(1, (int)std::ceil((hi[a] - lo[a]) / g.cell))) + 2;  // one empty cell around
        const double mid = 0.5 * (lo[a] + hi[a]);
        g.org[a] = mid - 0.5 * g.cell * g.n[a];
    }
    // 0: free, 1: surface, 2 and up: region labels.  A triangle's block of cells is counted at its
    // corners, and running sums along the axes give the cells' counts: long triangles that each
    // span most of the grid cost no more than small ones (a rod of 400,000: 28 s -> 0.05 s)
    std::vector<uint16_t> lab((size_t)g.size(), 0);
    const int ex = g.n[0] + 1, ey = g.n[1] + 1;
    std::vector<uint32_t> met((size_t)ex * ey * (g.n[2] + 1), 0);
    for (int64_t t = 0; t < T; ++t) {
        int c0[3], c1[3];
        for (int a = 0; a < 3; ++a) {
            const double v0 = V[3 * (int64_t)I[3 * t] + a], v1 = V[3 * (int64_t)I[3 * t + 1] + a],
                         v2 = V[3 * (int64_t)I[3 * t + 2] + a];
            c0[a] = std::max(0, (int)std::floor((std::min(v0, std::min(v1, v2)) - pad - g.org[a]) / g.cell));
            c1[a] = std::min(g.n[a] - 1, (int)std::floor((std::max(v0, std::max(v1, v2)) + pad - g.org[a]) / g.cell));
        }
        if (c0[0] > c1[0] || c0[1] > c1[1] || c0[2] > c1[2]) continue;
        for (int k = 0; k < 8; ++k) {
            const int x = (k & 1) ? c1[0] + 1 : c0[0], y = (k & 2) ? c1[1] + 1 : c0[1], z = (k & 4) ? c1[2] + 1 : c0[2];
            met[((size_t)z * ey + y) * ex + x] += ((k & 1) + ((k >> 1) & 1) + (k >> 2)) & 1 ? ~0u : 1u;
        }
    }
    for (int z = 0; z <= g.n[2]; ++z)
        for (int y = 0; y <= g.n[1]; ++y)
            for (int x = 1; x <= g.n[0]; ++x) met[((size_t)z * ey + y) * ex + x] += met[((size_t)z * ey + y) * ex + x - 1];
    for (int z = 0; z <= g.n[2]; ++z)
        for (int y = 1; y <= g.n[1]; ++y)
            for (int x = 0; x <= g.n[0]; ++x) met[((size_t)z * ey + y) * ex + x] += met[((size_t)z * ey + y - 1) * ex + x];
    for (int z = 1; z <= g.n[2]; ++z)
        for (int y = 0; y <= g.n[1]; ++y)
            for (int x = 0; x <= g.n[0]; ++x) met[((size_t)z * ey + y) * ex + x] += met[((size_t)(z - 1) * ey + y) * ex + x];
    for (int z = 0; z < g.n[2]; ++z)
        for (int y = 0; y < g.n[1]; ++y)
            for (int x = 0; x < g.n[0]; ++x)
                if (met[((size_t)z * ey + y) * ex + x] != 0) lab[(size_t)g.at(x, y, z)] = 1;
    // regions of free cells; the first (from the corner) is the outside
    struct Region {
        int64_t size, seed;
    };
    std::vector<Region> regions;
    std::vector<int64_t> queue;
    for (int64_t s = 0; s < g.size() && regions.size() < 1000; ++s) {
        if (lab[(size_t)s] != 0) continue;
        const uint16_t id = (uint16_t)(2 + regions.size());
        queue.assign(1, s);
        lab[(size_t)s] = id;
        for (size_t q = 0; q < queue.size(); ++q) {
            const int64_t c = queue[q];
            const int x = (int)(c % g.n[0]), y = (int)(c / g.n[0] % g.n[1]), z = (int)(c / g.n[0] / g.n[1]);
            const int nb[6][3] = {{x - 1, y, z}, {x + 1, y, z}, {x, y - 1, z}, {x, y + 1, z}, {x, y, z - 1}, {x, y, z + 1}};
            for (const auto& b : nb) {
                if (b[0] < 0 || b[1] < 0 || b[2] < 0 || b[0] >= g.n[0] || b[1] >= g.n[1] || b[2] >= g.n[2]) continue;
                const int64_t d = g.at(b[0], b[1], b[2]);
                if (lab[(size_t)d] == 0) {
                    lab[(size_t)d] = id;
                    queue.push_back(d);
                }
            }
        }
        regions.push_back({(int64_t)queue.size(), s});
    }
    // the winding number of the largest regions but the outside
    std::vector<uint8_t> inside(regions.size() + 2, 0);
    std::vector<size_t> order;
    for (size_t r = 0; r < regions.size(); ++r)
        if (regions[r].seed != 0 && regions[r].size >= 8) order.push_back(r);
    std::sort(order.begin(), order.end(), [&](size_t a, size_t b) { return regions[a].size > regions[b].size; });
    if (order.size() > 4) order.resize(4);
    bool any = false;
    for (size_t r : order) {
        const int64_t c = regions[r].seed;
        const int xyz[3] = {(int)(c % g.n[0]), (int)(c / g.n[0] % g.n[1]), (int)(c / g.n[0] / g.n[1])};
        double p[3];
        for (int a = 0; a < 3; ++a) p[a] = g.org[a] + g.cell * (xyz[a] + 0.5);
        const double w = winding(V, I, T, p), near = std::nearbyint(w);
        if (near != 0.0 && std::fabs(w - near) < 1e-3) {
            inside[r + 2] = 1;
            any = true;
        }
    }
    if (!any) return none;
    // counts of inside cells below a corner (for "is this block all inside"), and the largest
    // inside cube whose upper corner is the cell
    const int mx = g.n[0] + 1, my = g.n[1] + 1;
    std::vector<int32_t> pre((size_t)mx * my * (g.n[2] + 1), 0);
    std::vector<uint8_t> cube((size_t)g.size(), 0);
    auto pat = [&](int x, int y, int z) -> int32_t& { return pre[((size_t)z * my + y) * mx + x]; };
    std::vector<std::vector<int64_t>> by_size(256);
    for (int z = 0; z < g.n[2]; ++z)
        for (int y = 0; y < g.n[1]; ++y)
            for (int x = 0; x < g.n[0]; ++x) {
                const int64_t c = g.at(x, y, z);
                const bool in = lab[(size_t)c] >= 2 && inside[lab[(size_t)c]] != 0;
                pat(x + 1, y + 1, z + 1) = (in ? 1 : 0) + pat(x, y + 1, z + 1) + pat(x + 1, y, z + 1) + pat(x + 1, y + 1, z) -
                                           pat(x, y, z + 1) - pat(x, y + 1, z) - pat(x + 1, y, z) + pat(x, y, z);
                if (!in) continue;
                int m = 255;
                for (int k = 1; k < 8; ++k) {
                    const int u = x - (k & 1), v = y - ((k >> 1) & 1), w = z - (k >> 2);
                    m = std::min(m, u < 0 || v < 0 || w < 0 ? 0 : (int)cube[(size_t)g.at(u, v, w)]);
                }
                cube[(size_t)c] = (uint8_t)std::min(254, m + 1);
                by_size[cube[(size_t)c]].push_back(c);
            }
    auto full = [&](const int* a, const int* b) {
        const int32_t cnt = pat(b[0], b[1], b[2]) - pat(a[0], b[1], b[2]) - pat(b[0], a[1], b[2]) - pat(b[0], b[1], a[2]) +
                            pat(a[0], a[1], b[2]) + pat(a[0], b[1], a[2]) + pat(b[0], a[1], a[2]) - pat(a[0], a[1], a[2]);
        return (int64_t)cnt == (int64_t)(b[0] - a[0]) * (b[1] - a[1]) * (b[2] - a[2]);
    };
    std::vector<uint8_t> covered((size_t)g.size(), 0);
    int made = 0;
    for (int s = 255; s >= 1 && made < max_boxes; --s)
        for (size_t i = 0; i < by_size[(size_t)s].size() && made < max_boxes; ++i) {
            const int64_t c = by_size[(size_t)s][i];
            const int x = (int)(c % g.n[0]), y = (int)(c / g.n[0] % g.n[1]), z = (int)(c / g.n[0] / g.n[1]);
            // the cube's middle cell not covered yet
            if (covered[(size_t)g.at(x - s / 2, y - s / 2, z - s / 2)]) continue;
            IBox b = {{x - s + 1, y - s + 1, z - s + 1}, {x + 1, y + 1, z + 1}};
            for (bool grew = true; grew;) {
                grew = false;
                for (int a = 0; a < 3; ++a)
                    for (int side = 0; side < 2; ++side) {
                        IBox e = b;
                        if (side) ++e.hi[a]; else --e.lo[a];
                        if (e.lo[a] < 0 || e.hi[a] > g.n[a] || !full(e.lo, e.hi)) continue;
                        b = e;
                        grew = true;
                    }
            }
            for (int w = b.lo[2]; w < b.hi[2]; ++w)
                for (int v = b.lo[1]; v < b.hi[1]; ++v)
                    for (int u = b.lo[0]; u < b.hi[0]; ++u) covered[(size_t)g.at(u, v, w)] = 1;
            SolidBox o;
            for (int a = 0; a < 3; ++a) {
                // the cells' own planes: every triangle is at least pad away from a free cell
                o.lo[a] = (float)(g.org[a] + g.cell * b.lo[a]);
                o.hi[a] = (float)(g.org[a] + g.cell * b.hi[a]);
            }
            o.mesh = mesh;
            out.push_back(o);
            ++made;
        }
    return pad;
}

namespace {

// median split along the longest axis of the boxes' centres; leaves hold one box, their
// child index is ~mesh
int32_t build_solid(std::vector<SolidBox>& b, int64_t first, int64_t last, std::vector<BvhNode>& nodes)
{
    const int32_t id = (int32_t)nodes.size();
    nodes.emplace_back();
    float clo[3] = {INFINITY, INFINITY, INFINITY}, chi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int64_t i = first; i < last; ++i)
        for (int a = 0; a < 3; ++a) {
            const float c = 0.5f * (b[(size_t)i].lo[a] + b[(size_t)i].hi[a]);
            clo[a] = std::min(clo[a], c);
            chi[a] = std::max(chi[a], c);
        }
    int axis = 0;
    for (int a = 1; a < 3; ++a)
        if (chi[a] - clo[a] > chi[axis] - clo[axis]) axis = a;
    const int64_t mid = first + (last - first) / 2;
    std::nth_element(b.begin() + first, b.begin() + mid, b.begin() + last, [&](const SolidBox& p, const SolidBox& q) {
        return p.lo[axis] + p.hi[axis] < q.lo[axis] + q.hi[axis];
    });
    BvhNode nd;
    std::memset(&nd, 0, sizeof(nd));
    // a single box (the root of a one-box tree) is both children: an empty child's inverted
    // box would read as an unbounded one in the octant copies
    const bool one = last - first == 1;
    const int64_t rb[2] = {first, one ? first : mid}, re[2] = {one ? last : mid, last};
    for (int c = 0; c < 2; ++c) {
        float lo[3] = {3.0e38f, 3.0e38f, 3.0e38f}, hi[3] = {-3.0e38f, -3.0e38f, -3.0e38f};
        for (int64_t i = rb[c]; i < re[c]; ++i)
            for (int a = 0; a < 3; ++a) {
                lo[a] = std::min(lo[a], b[(size_t)i].lo[a]);
                hi[a] = std::max(hi[a], b[(size_t)i].hi[a]);
            }
        int32_t child = -1, count = 0;
        if (re[c] - rb[c] == 1) {
            child = ~b[(size_t)rb[c]].mesh;
            count = 1;
        } else {
            child = build_solid(b, rb[c], re[c], nodes);
        }
        std::memcpy(c == 0 ? nd.lo0 : nd.lo1, lo, sizeof(lo));
        std::memcpy(c == 0 ? nd.hi0 : nd.hi1, hi, sizeof(hi));
        if (c == 0) { nd.child0 = child; nd.count0 = count; }
        else { nd.child1 = child; nd.count1 = count; }
    }
    nd.count0 |= axis << kSplitAxisShift;
    nodes[(size_t)id] = nd;
    return id;
}

}  // namespace

void build_solid_tree(std::vector<SolidBox> boxes, std::vector<BvhNode>& nodes)
{
    nodes.clear();
    if (!boxes.empty()) (void)build_solid(boxes, 0, (int64_t)boxes.size(), nodes);
}

}  // namespace gm
