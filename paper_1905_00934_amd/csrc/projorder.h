// The projector's workgroup lists, built by the plan on the host.  Plain C++, shared with the
// host-side check of their coverage.
#pragma once

#include <algorithm>
#include <vector>

#include "projidx.h"

namespace dect {

// Bins of a base view whose rays step along the same axis: [0, split) and [split, D); first:
// the axis of bin 0 (0: x-stepped, 1: y-stepped).
struct ViewSplit {
    int split, first;
};

// What a workgroup costs beside its lines, in lines: its start and end (a lone workgroup of a
// 101^2 fan with 13 lines per wave takes 8 us, of which the lines are about a third).  16 left
// the XCDs with few lines with many more workgroups than the others; 64, 512 and 4096 measured
// within 2 % of this.
constexpr long kProjStart = 128;

// Workgroup list of the projector for one lane layout (64 / bv bins of nv views each): one
// workgroup per tile and axis that any of its rays steps along (tiles at a view's 45 degree
// bin have both; a workgroup serves the rays of one axis), each XCD's in the order of the lines
// their rays cross, longest first.  In the plain order with both axes of a tile in one
// workgroup, such a workgroup started last and ran alone: at 512^2 the others ended at 60 us,
// the launch at 107.  A tile goes to the XCD of the XCD-aware order (proj_tile) while that one
// has less than its share and a sixteenth, else to the one with least: detectors of few bin
// groups left XCDs idle (64^2 / 90 x 95 parallel ran on three of the eight: 10.1 us, now 9.5;
// 100^2 / 140 x 149 in double precision 12.5 us, now 11.6); from about 384^2 on the order is
// balanced as it is.  Entry: 2 (bg gy + vg) + axis, or -1 (none).
inline std::vector<int> proj_launch_order(const dect_geometry& g, int Vb, const ViewSplit* splits,
                                          int bv, int nv, int chunk) {
    const int D = g.n_det;
    const int gx = proj_grid_x(D, bv), gy = proj_grid_y(Vb, nv), bb = 64 / bv;
    const unsigned blocks = proj_blocks(gx, gy, chunk);
    struct Tile {
        int code, lines, xcd;
    };
    std::vector<HostView> view(Vb);
    for (int v = 0; v < Vb; ++v) view[v] = host_view(g, v);
    std::vector<Tile> tiles;
    long total = 0;
    for (unsigned id = 0; id < blocks; ++id) {
        int bg, vg;
        proj_tile(id, gy, chunk, bg, vg);
        if (bg >= gx) continue;
        const int b0 = bg * bb, b1 = std::min(b0 + bb, D) - 1;
        const int v0 = vg * nv, v1 = std::min(v0 + nv, Vb) - 1;
        int axes = 0, lines = 0;
        for (int v = v0; v <= v1; ++v) {
            const ViewSplit& q = splits[v];
            if (b0 < q.split) axes |= 1 << q.first;
            if (b1 >= q.split) axes |= 2 >> q.first;
        }
        for (int c = 0; c < 4; ++c) {  // the corner rays
            const HostRay r = host_ray(g, view[c & 2 ? v1 : v0], c & 1 ? b1 : b0);
            int k0, k1;
            proj_ray_range<double>(r.phi0, r.slope, r.xstep ? g.nx : g.ny, r.xstep ? g.ny : g.nx,
                                   k0, k1);
            lines = std::max(lines, k1 - k0 + 1);
        }
        for (int ax = 0; ax < 2; ++ax)
            if (axes >> ax & 1) {
                tiles.push_back({2 * (bg * gy + vg) + ax, lines, (int)(id % kXcds)});
                total += lines + kProjStart;
            }
    }
    std::stable_sort(tiles.begin(), tiles.end(),
                     [](const Tile& a, const Tile& b) { return a.lines > b.lines; });
    const long most = total / kXcds + total / (16 * kXcds) +
                      (tiles.empty() ? 0 : tiles[0].lines + kProjStart);
    std::vector<int> by_xcd[kXcds];
    long load[kXcds] = {};
    size_t longest = 0;
    for (const Tile& t : tiles) {
        int x = t.xcd;
        if (load[x] + t.lines + kProjStart > most)
            x = (int)(std::min_element(load, load + kXcds) - load);
        load[x] += t.lines + kProjStart;
        by_xcd[x].push_back(t.code);
        longest = std::max(longest, by_xcd[x].size());
    }
    std::vector<int> order(longest * kXcds, -1);
    for (int x = 0; x < kXcds; ++x)
        for (size_t n = 0; n < by_xcd[x].size(); ++n) order[n * kXcds + x] = by_xcd[x][n];
    return order;
}

}  // namespace dect
