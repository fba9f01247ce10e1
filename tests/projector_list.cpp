// Host check of the projector's workgroup lists (projorder.h, the plan's own code): every ray
// is served by exactly one workgroup, that of its tile and axis, for every lane layout of one
// and two rays per lane; lists hold no entry outside the tiles.  Plain C++.
//
// usage: projector_list kind nx ny pixel V D det_cm offset src_iso src_det angle0 span sym
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
    std::vector<int> axis((size_t)Vb * D);
    std::vector<ViewSplit> splits;
    for (int v = 0; v < Vb; ++v) {
        int split = D;
        for (int b = 0; b < D; ++b) {
            axis[(size_t)v * D + b] = host_ray(g, v, b).xstep ? 0 : 1;
            if (b && axis[(size_t)v * D + b] != axis[(size_t)v * D + b - 1]) split = b;
        }
        splits.push_back({split, axis[(size_t)v * D]});
    }
    int bad = 0;
    for (int R = 1; R <= 2; ++R)
        for (int views = 1; R * views <= 64; views *= 2)
            for (int chunk : {1, 2, 5, 16}) {
                const int bv = R * views, nv = R * R * views, bb = 64 / bv;
                const int gx = proj_grid_x(D, bv), gy = proj_grid_y(Vb, nv);
                std::vector<int> seen((size_t)Vb * D, 0);
                for (int e : proj_launch_order(g, Vb, splits.data(), bv, nv, chunk)) {
                    if (e < 0) continue;
                    const int ax = e & 1, bg = (e >> 1) / gy, vg = (e >> 1) % gy;
                    if (bg >= gx) {
                        ++bad;
                        continue;
                    }
                    for (int r = 0; r < R; ++r)
                        for (int lane = 0; lane < 64; ++lane) {
                            const int v = (vg * R + r) * bv + lane % bv, b = bg * bb + lane / bv;
                            if (v < Vb && b < D && axis[(size_t)v * D + b] == ax)
                                ++seen[(size_t)v * D + b];
                        }
                }
                for (int n : seen) bad += n != 1;
            }
    std::printf(bad ? "%d errors\nFAILED\n" : "%d errors\nOK\n", bad);
    return bad != 0;
}
