// Footprint arithmetic of the transposed projector's staged gather, shared by the kernel
// and by the host-side check of its bounds: per 8x8 block, base view and orbit member the
// window of candidate bins and the plane that places each pixel's candidates in it.
// Plain C++ (no runtime calls), so it also compiles for the host alone.
#pragma once

#include <cmath>

#include "projidx.h"

namespace dect {

constexpr int kBpWin = 32;      // bins of a slot's window
// Flags beside a slot's candidate count (below 64): its window takes up to 2 kBpWin bins;
// its candidates are found one by one.
constexpr int kBpLong = 64, kBpDirect = 128;

// One slot of the block whose first pixel is (i0, j0): plane coefficients relative to the
// window start L (px at the first pixel, pi and pj per pixel step along i and j), and L,
// the flags and the candidate count C packed as 256 L + flags + C.
struct alignas(16) BpSlot {
    float px, pi, pj;
    int info;
};
DECT_HD inline int bp_slot_window(int info) { return info >> 8; }

// The slot of base view w (ViewParam) and orbit member mm.  C is 0 when no candidate lies
// on the detector or the slot is kBpDirect, else at least 2.
template <int SYM, typename V>
DECT_HD inline BpSlot bp_slot(const V& w, int mm, int i0, int j0, int nx, int ny, int D) {
    // Centre of the block, centred coordinates, turned by mm quarter turns.
    double x = (double)i0 + 3.5 - 0.5 * (nx - 1), y = (double)j0 + 3.5 - 0.5 * (ny - 1);
    if (SYM == 4) {
        const double cx = x, cy = y;
        x = mm == 0 ? cx : mm == 1 ? -cy : mm == 2 ? -cx : cy;
        y = mm == 0 ? cy : mm == 1 ? cx : mm == 2 ? -cy : -cx;
    }
    const double inv = 1.0 / ((double)w.d0 + (double)w.di * x + (double)w.dj * y);
    const double bq = ((double)w.ni * x + (double)w.nj * y) * inv;
    const double gx = ((double)w.ni - bq * (double)w.di) * inv;
    const double gy = ((double)w.nj - bq * (double)w.dj) * inv;
    const double ex = (double)w.di * inv, ey = (double)w.dj * inv;
    const double q = 3.5 * (fabs(ex) + fabs(ey));
    const double span = 3.5 * (fabs(gx) + fabs(gy));
    BpSlot out{0.0f, 0.0f, 0.0f, kBpDirect};  // until shown otherwise
    if (!(inv > 0.0) || !(q < 0.4) || !(fabs(ex) < 0.1) || !(fabs(ey) < 0.1)) return out;
    const double iq = 1.0 / (1.0 - q);
    const double gn = sqrt(gx * gx + gy * gy), en = sqrt(ex * ex + ey * ey);
    const double E = 12.25 * (gn * en + fabs(gx * ex + gy * ey)) * iq;
    const double db = span * iq;  // largest change of beta over the block
    // Gradient of beta anywhere in the block: (g - dbeta e) / (1 + e.t).  A point one pixel
    // away along an axis moves beta by |g_axis| / (1 - |e_axis|) at most.  Plus the rounding
    // of the view and ray tables in single precision.
    const double hx = (fabs(gx) + db * fabs(ex)) * iq, hy = (fabs(gy) + db * fabs(ey)) * iq;
    const double hm = fmax(hx / (1.0 - fabs(ex) * iq), hy / (1.0 - fabs(ey) * iq));
    const double hb = hm * 1.001 + 0.004 + 4e-6 * D;
    const double beta = bq + (double)w.boff;
    if (beta + db + hb < 0.0 || beta - db - hb > (double)(D - 1)) {
        out.info = 0;
        return out;
    }
    // floor(P) is at most the first candidate, P = beta (affine) - E - hb + 1.
    const double P0 = beta - E - hb + 1.0;  // at the block's centre
    const double C = fmax(ceil(2.0 * (hb + E)), 2.0);
    const double L = floor(P0 - span - 1e-3);
    const double len = C + ceil(2.0 * span) + 1.0;
    if (!(len <= 2.0 * kBpWin) || !(fabs(L) < 4194304.0)) return out;
    // A pixel step along i and j as member mm sees it.
    double si = gx, sj = gy;
    if (SYM == 4 && mm == 1) { si = gy; sj = -gx; }
    if (SYM == 4 && mm == 2) { si = -gx; sj = -gy; }
    if (SYM == 4 && mm == 3) { si = -gy; sj = gx; }
    out.px = (float)(P0 - L - 3.5 * (si + sj));
    out.pi = (float)si;
    out.pj = (float)sj;
    out.info = (int)L * 256 + (len <= (double)kBpWin ? 0 : kBpLong) + (int)C;
    return out;
}

// Window index of the first candidate of pixel (i0 + oi, j0 + oj), oi and oj in [0, 7]: the
// plane is positive over the block, so truncation is the floor.
DECT_HD inline int bp_slot_start(const BpSlot& e, float oi, float oj) {
    return (int)fmaf(e.pj, oj, fmaf(e.pi, oi, e.px));
}

}  // namespace dect
