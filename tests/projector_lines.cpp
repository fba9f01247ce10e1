// Host check of the staged projector, from the kernel's own helpers (projidx.h) and the plan's
// own workgroup lists (projorder.h), for one and two rays per lane: for every workgroup, wave,
// lane and ray of a launch, the union of the rays' lines and each wave's share of it, the window
// that a wave stages of each line around its extreme rays, and every tap.  Checks that staged
// lines lie in the image, that a load reads its own record or, past either end of the line,
// nothing (every record size, whole and in halves), that a sample's two taps are floor(phi) and
// floor(phi) + 1 of the zero-extended line whether staged or read directly, that every sample
// with a tap inside the image is taken once, and that every ray is stored once.  Plain C++.
//
// usage: projector_lines kind nx ny pixel V D det_cm offset src_iso src_det angle0 span sym
//        precision(32|64)
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <limits>

#include "projorder.h"

using namespace dect;

static int g_errors = 0;
static void wrong(const char* what, long a, long b, long c) {
    if (g_errors++ < 10) std::printf("%s: %ld %ld %ld\n", what, a, b, c);
}

// A raw buffer load of 4 bytes at `off`: read inside the buffer's bytes, else zero.
static bool reads(unsigned off, unsigned bytes) { return (unsigned long)off + 4 <= bytes; }

// The window's loads of a line of wl records, against the record each lane is to hold.
static void check_loads(int start, int wl) {
    for (unsigned bytes : {4u, 8u, 16u, 32u, 64u})
        for (int parts = 1; parts <= (bytes == 64 ? 2 : 1); ++parts)
            for (int part = 0; part < parts; ++part)
                for (int lane = 0; lane < kProjWin; ++lane)
                    for (unsigned at = 0; at < bytes; at += 4) {
                        const unsigned off = proj_line_offset(start, lane, parts, bytes) + at;
                        const bool in = reads(off, proj_line_bytes(wl, parts, part, bytes));
                        const long t = (long)start + lane;
                        if (in != (t >= 0 && t < wl)) wrong("load past the line", start, lane, wl);
                        if (in && off != (unsigned long)t * parts * bytes + at)
                            wrong("record of another tap", start, lane, wl);
                    }
}

template <typename T>
struct Ray {
    T phi0, slope;
    int axis;
};

template <typename T>
static void check(const dect_geometry& g, int Vb, const std::vector<Ray<T>>& rays,
                  const std::vector<ViewSplit>& splits, int R, int views, int KS, int chunk,
                  bool loads) {
    const int D = g.n_det, bv = R * views, lbv = __builtin_ctz((unsigned)bv);
    const int gy = proj_grid_y(Vb, bv * R);
    std::vector<int> stored((size_t)Vb * D, 0);
    std::vector<long> taken((size_t)Vb * D, 0);
    for (int entry : proj_launch_order(g, Vb, splits.data(), bv, bv * R, chunk)) {
        if (entry < 0) continue;
        const int ax = entry & 1, bg = (entry >> 1) / gy, vg = (entry >> 1) % gy;
        const int n_steps = ax == 0 ? g.nx : g.ny, wl = ax == 0 ? g.ny : g.nx;
        bool on[2][64];
        T phi0[2][64], slope[2][64];
        long ray[2][64];
        int s0 = 1 << 30, s1 = -1, first = -1, last = -1;
        for (int lane = 0; lane < 64; ++lane)
            for (int r = 0; r < R; ++r) {
                const int v = proj_lane_view(vg, r, R, lbv, lane), b = proj_lane_bin(bg, lbv, lane);
                on[r][lane] = b < D && v < Vb && rays[(size_t)v * D + b].axis == ax;
                phi0[r][lane] = T(-1e30);
                slope[r][lane] = T(0);
                if (!on[r][lane]) continue;
                ray[r][lane] = (long)v * D + b;
                phi0[r][lane] = rays[ray[r][lane]].phi0;
                slope[r][lane] = rays[ray[r][lane]].slope;
                ++stored[ray[r][lane]];
                int k0, k1;
                proj_ray_range<T>(phi0[r][lane], slope[r][lane], n_steps, wl, k0, k1);
                if (k0 <= k1) s0 = std::min(s0, k0), s1 = std::max(s1, k1);
                if (first < 0) first = lane;
                last = lane;
            }
        if (first < 0) {
            wrong("workgroup without a ray", entry, R, views);
            continue;
        }
        const int rf = on[0][first] ? 0 : 1, rl = on[R - 1][last] ? R - 1 : R - 2;
        int wa, wb;
        proj_window_line<T>(phi0[rf][first], slope[rf][first], phi0[rl][last], slope[rl][last], wa,
                            wb);
        for (int wave = 0; wave < KS; ++wave) {
            int c0, c1;
            proj_wave_share(s0, s1, wave, KS, c0, c1);
            for (int k = c0; k <= c1; ++k) {
                if (k < 0 || k >= n_steps) wrong("line outside the image", k, n_steps, entry);
                const int s = proj_window(wa, wb, k);
                if (loads) check_loads(s, wl);
                for (int r = 0; r < R; ++r)
                    for (int lane = 0; lane < 64; ++lane) {
                        if (!on[r][lane]) continue;
                        const T ph = std::fma(slope[r][lane], (T)k, phi0[r][lane]);
                        const T fl = std::floor(ph), w1 = ph - fl;
                        const unsigned idx = (unsigned)((int)fl - s);
                        const bool inside = ph > T(-1) && ph < (T)wl;
                        taken[ray[r][lane]] += inside;
                        if (idx <= (unsigned)(kProjWin - 2)) {
                            if (s + (long)idx != (long)fl)
                                wrong("staged tap", ray[r][lane], k, (long)idx);
                        } else if (inside) {
                            T u0, u1;
                            const int j = proj_taps<T>(phi0[r][lane], slope[r][lane], (T)k, wl, u0,
                                                       u1);
                            if (j < 0 || j > wl - 2) wrong("direct tap", ray[r][lane], k, j);
                            // The same weights on the same taps (alpha is exact; 1 - alpha and
                            // the tent's 2 - t round once).
                            for (int t = -1; t <= 2; ++t) {
                                const long at = (long)fl + t;
                                const T a = at < 0 || at >= wl ? T(0) : t == 0 ? T(1) - w1
                                                                  : t == 1 ? w1 : T(0);
                                const T b = at == j ? u0 : at == j + 1 ? u1 : T(0);
                                if (std::fabs((double)a - (double)b) >
                                    4 * std::numeric_limits<T>::epsilon())
                                    wrong("direct weight", ray[r][lane], k, t);
                            }
                        }
                    }
            }
        }
    }
    for (long i = 0; i < (long)Vb * D; ++i) {
        if (stored[i] != 1) wrong("rays stored", i, stored[i], R);
        const int n_steps = rays[i].axis == 0 ? g.nx : g.ny, wl = rays[i].axis == 0 ? g.ny : g.nx;
        long want = 0;
        for (int k = 0; k < n_steps; ++k) {
            const T ph = std::fma(rays[i].slope, (T)k, rays[i].phi0);
            want += ph > T(-1) && ph < (T)wl;
        }
        if (taken[i] != want) wrong("samples of a ray", i, taken[i], want);
    }
}

template <typename T>
static void check_all(const dect_geometry& g, int sym) {
    const int Vb = g.n_views / sym, D = g.n_det;
    std::vector<Ray<T>> rays((size_t)Vb * D);
    std::vector<ViewSplit> splits;
    for (int v = 0; v < Vb; ++v) {
        int split = D;
        for (int b = 0; b < D; ++b) {
            const HostRay r = host_ray(g, v, b);
            rays[(size_t)v * D + b] = {(T)r.phi0, (T)r.slope, r.xstep ? 0 : 1};
            if (b && rays[(size_t)v * D + b].axis != rays[(size_t)v * D + b - 1].axis) split = b;
        }
        splits.push_back({split, rays[(size_t)v * D].axis});
    }
    const bool small = (long)Vb * D * g.nx < 4000000;
    for (int R = 1; R <= 2; ++R)
        for (int views : {1, 2, 8})
            for (int KS : {2, 8})
                for (int chunk : {1, 3}) {
                    const bool usual = views == 2 && KS == 8 && chunk == 1;
                    if (small || usual) check<T>(g, Vb, rays, splits, R, views, KS, chunk,
                                                 small && usual);
                }
}

int main(int argc, char** argv) {
    if (argc != 15) return 2;
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
    const int sym = std::atoi(argv[13]);
    // Windows at both ends of short, long and one-window lines, and as far off as they get.
    const int far = 1 << 23;
    for (int wl : {2, 3, 63, 64, 65, 512, 32768, 1 << 25, 1 << 29})
        for (int start : {-far, -65, -64, -63, -31, -1, 0, 1, wl - 65, wl - 64, wl - 63, wl - 1,
                          wl, wl + 1, far})
            if (start <= far) check_loads(start, wl);
    if (std::atoi(argv[14]) == 64) check_all<double>(g, sym);
    else check_all<float>(g, sym);
    std::printf(g_errors ? "%d errors\nFAILED\n" : "%d errors\nOK\n", g_errors);
    return g_errors != 0;
}
