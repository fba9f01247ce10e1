// Host check of the transposed projector's staged windows, with the kernel's own
// arithmetic (bpidx.h): for every base view, orbit member, 8x8 block and pixel, every bin
// whose ray has a nonzero weight on the pixel (evaluated in double from the ray geometry)
// is among the C candidates the pixel takes, and every candidate lies inside the staged
// window; a slot reported empty has no weight at all.  Plain C++.
//
// usage: transpose_bounds kind nx ny pixel V D det_cm offset src_iso src_det angle0 span
//        sym precision(32|64)
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "bpidx.h"

using namespace dect;

template <typename T>
struct View {
    T ni, nj, d0, di, dj, boff;
};

template <typename T, int SYM>
static int check(const dect_geometry& g) {
    const int Vb = g.n_views / SYM, D = g.n_det, nx = g.nx, ny = g.ny;
    const int dx = SYM == 4 ? nx / 2 : nx, dy = SYM == 4 ? ny / 2 : ny;
    long slots = 0, longs = 0, direct = 0, empty = 0, taken = 0, hits = 0;
    int errors = 0;
    std::vector<HostRay> rays(D);
    // Every view of small problems, a spread of them of large ones.
    const int vstep = (long)dx * dy * Vb > 4000000 ? 13 : 1;
    for (int v = 0; v < Vb; v += vstep) {
        for (int b = 0; b < D; ++b) rays[b] = host_ray(g, v, b);
        const double t = g.angle0 + (double)v * g.span / (double)g.n_views;
        const double c = std::cos(t), s = std::sin(t), d = g.pixel_cm;
        View<T> w;
        if (g.kind == DECT_PARALLEL) {
            w = View<T>{(T)(d * c / g.det_cm), (T)(d * s / g.det_cm), (T)1, (T)0, (T)0, (T)0};
        } else {
            const double K = g.src_det_cm / g.det_cm;
            w = View<T>{(T)(-K * d * s), (T)(K * d * c), (T)g.src_iso_cm, (T)(-d * c), (T)(-d * s),
                        (T)0};
        }
        w.boff = (T)(0.5 * (D - 1) - g.det_offset);
        for (int mm = 0; mm < SYM; ++mm)
            for (int j0 = 0; j0 < dy; j0 += 8)
                for (int i0 = 0; i0 < dx; i0 += 8) {
                    const BpSlot e = bp_slot<SYM>(w, mm, i0, j0, nx, ny, D);
                    const int C = e.info & (kBpLong - 1), L = bp_slot_window(e.info);
                    const int win = e.info & kBpLong ? 2 * kBpWin : kBpWin;
                    ++slots;
                    direct += (e.info & kBpDirect) != 0;
                    longs += (e.info & kBpLong) != 0;
                    empty += e.info == 0;
                    if (e.info & kBpDirect) continue;
                    for (int oj = 0; oj < 8; ++oj)
                        for (int oi = 0; oi < 8; ++oi) {
                            int first = 0, last = -1;
                            if (C > 0) {
                                first = bp_slot_start(e, (float)oi, (float)oj);
                                last = first + C - 1;
                                if (first < 0 || last >= win || C < 2) {
                                    if (errors++ < 10)
                                        std::printf("view %d member %d block (%d, %d) pixel (%d, "
                                                    "%d): candidates %d..%d outside the window\n",
                                                    v, mm, i0, j0, oi, oj, first, last);
                                }
                            }
                            const int i = i0 + oi, j = j0 + oj;
                            if (i >= dx || j >= dy) continue;
                            int im = i, jm = j;
                            for (int k = 0; k < mm; ++k) {
                                const int o = im;
                                im = nx - 1 - jm;
                                jm = o;
                            }
                            taken += C;
                            // All bins of small detectors, those near the window otherwise.
                            const int lo = D <= 600 ? 0 : std::max(0, L - 100);
                            const int hi = D <= 600 ? D - 1 : std::min(D - 1, L + 140);
                            for (int b = lo; b <= hi; ++b) {
                                const HostRay& r = rays[b];
                                const double phi = r.phi0 + r.slope * (r.xstep ? im : jm);
                                if (std::fabs(phi - (r.xstep ? jm : im)) >= 1.0) continue;
                                ++hits;
                                if (C == 0 || b < L + first || b > L + last)
                                    if (errors++ < 10)
                                        std::printf("view %d member %d pixel (%d, %d): bin %d is "
                                                    "not among %d..%d\n", v, mm, i, j, b,
                                                    L + first, L + last);
                            }
                        }
                }
    }
    std::printf("%ld slots, %ld long, %ld direct, %ld empty, %.3f candidates and %.3f weights per pixel, "
                "%d errors\n", slots, longs, direct, empty, (double)taken / (slots * 64.0),
                (double)hits / (slots * 64.0), errors);
    return errors;
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
    const int sym = std::atoi(argv[13]), prec = std::atoi(argv[14]);
    const int e = prec == 64 ? (sym == 4 ? check<double, 4>(g) : check<double, 1>(g))
                             : (sym == 4 ? check<float, 4>(g) : check<float, 1>(g));
    std::printf(e ? "FAILED\n" : "OK\n");
    return e != 0;
}
