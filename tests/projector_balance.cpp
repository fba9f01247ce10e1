// Host check of the projector's workgroup lists (projorder.h, the plan's own code): no XCD has
// much more than its share of the launch.  Plain C++.
//
// usage: projector_balance kind nx ny pixel V D det_cm offset src_iso src_det angle0 span sym
#include <cstdio>
#include <cstdlib>

#include "projorder.h"

using namespace dect;

int main(int argc, char** argv) {
    if (argc != 14) return 2;
    dect_geometry g{};
    g.kind = std::atoi(argv[1]);
    g.nx = std::atoi(argv[2]);
    g.ny = std::atoi(argv[3]);
    g.pixel_cm = std::atof(argv[4]);
    g.n_views = std::atoi(argv[5]);
    g.n_det = std::atoi(argv[6]);
    g.det_cm = std::atof(argv[7]);
    g.det_offset = std::atof(argv[8]);
    g.src_iso_cm = std::atof(argv[9]);
    g.src_det_cm = std::atof(argv[10]);
    g.angle0 = std::atof(argv[11]);
    g.span = std::atof(argv[12]);
    const int Vb = g.n_views / std::atoi(argv[13]), D = g.n_det;
    std::vector<ViewSplit> splits;
    for (int v = 0; v < Vb; ++v) {
        const bool first = host_ray(g, v, 0).xstep;
        int split = 1;
        while (split < D && host_ray(g, v, split).xstep == first) ++split;
        splits.push_back({split, first ? 0 : 1});
    }
    int bad = 0;
    for (int R = 1; R <= 2; ++R)
        for (int views : {1, 2, 8})
            for (int chunk : {1, 3}) {
                const int bv = R * views, nv = R * R * views, bb = 64 / bv;
                const int gy = proj_grid_y(Vb, nv);
                const std::vector<int> list =
                    proj_launch_order(g, Vb, splits.data(), bv, nv, chunk);
                long load[kXcds] = {}, total = 0, largest = 0;
                for (size_t i = 0; i < list.size(); ++i) {
                    if (list[i] < 0) continue;
                    const int bg = (list[i] >> 1) / gy, vg = (list[i] >> 1) % gy;
                    long lines = 0;
                    for (int c = 0; c < 4; ++c) {
                        const HostRay r =
                            host_ray(g, std::min(vg * nv + (c & 2 ? nv - 1 : 0), Vb - 1),
                                     std::min(bg * bb + (c & 1 ? bb - 1 : 0), D - 1));
                        int k0, k1;
                        proj_ray_range<double>(r.phi0, r.slope, r.xstep ? g.nx : g.ny,
                                               r.xstep ? g.ny : g.nx, k0, k1);
                        lines = std::max<long>(lines, k1 - k0 + 1);
                    }
                    load[i % kXcds] += lines + kProjStart;
                    total += lines + kProjStart;
                    largest = std::max(largest, lines + kProjStart);
                }
                // A moved tile finds an XCD at or below the mean.
                const long most = total / kXcds + total / (16 * kXcds) + largest;
                for (long x : load) bad += x > most;
            }
    std::printf(bad ? "%d errors\nFAILED\n" : "%d errors\nOK\n", bad);
    return bad != 0;
}
