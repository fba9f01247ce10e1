// Joseph projector R (ray-driven) and its exact transpose R^T (pixel-driven
// gather, no atomics), for gfx950.
//
// Rotational symmetry.  For a fan beam over a full turn with n_views divisible
// by 4 and a square image, view v + k V/4 is view v turned by k quarter turns,
// and the pixel grid maps onto itself.  The plan then defines the rays of those
// views as exact rotations of the V/4 base views (SYM = 4): one Joseph weight
// computation serves four views.  Otherwise SYM = 1 and every view is a base view.
//
// Projector: one or two base rays per lane; a wave holds consecutive bins of a few
// neighbouring base views, so output writes are coalesced along the detector.  It
// reads an "orbit" image O[j][i] = (X[rot^k (i, j)], k < SYM) -- the SYM rotated
// copies interleaved per pixel -- or its transpose for x-stepped rays, so that one
// record per tap serves all SYM views; a wave stages the part of each image line its
// rays cross in LDS and its lanes read their taps from there.
//
// Transpose: one lane owns the rotation orbit of a pixel.  For every base view
// and every orbit member it locates the bins whose samples can touch the pixel and
// re-evaluates each candidate's interpolation weight from the same ray geometry;
// each weight serves SYM (pixel, view) pairs.  The projector weighs a sample's two taps by the
// fraction of its position and scales by the step length at the end, while the transpose forms
// each weight step max(0, 1 - |d|) from the signed distance d of its own ray records, so the
// pair is a transpose up to rounding (FP64 adjointness to 1e-12), not bit for bit.  The views
// are split over the waves of a workgroup and the wave sums are added in a fixed order through
// LDS.
#include <mutex>

#include "bpidx.h"
#include "common.h"
#include "epilogue.h"
#include "kernels.h"
#include "profile.h"

namespace dect {

namespace {

// Pixel (i, j) turned by k quarter turns about the image centre (n x n image).
__device__ inline void rot(int k, int n, int i, int j, int& io, int& jo) {
    switch (k & 3) {
        case 0: io = i; jo = j; break;
        case 1: io = n - 1 - j; jo = i; break;
        case 2: io = n - 1 - i; jo = n - 1 - j; break;
        default: io = j; jo = n - 1 - i; break;
    }
}

// Orbit record of pixel (i, j): component k*CH + c = channel c of X at rot^k(i, j).
template <typename T, int CH, int SYM>
__device__ inline vec<T, CH * SYM> orbit_record(const vec<T, CH>* __restrict__ X, int nx, int i,
                                                int j) {
    vec<T, CH * SYM> o;
#pragma unroll
    for (int k = 0; k < SYM; ++k) {
        int io, jo;
        rot(k, nx, i, j, io, jo);
        const vec<T, CH> x = X[(size_t)jo * nx + io];
#pragma unroll
        for (int c = 0; c < CH; ++c) o.v[k * CH + c] = x.v[c];
    }
    return o;
}

// Orbit image O[j][i] and its transpose OT[i][j] in one pass: thread idx writes
// record idx of both.  SYM = 1 gives X and X^T.
template <typename T, int CH, int SYM, bool BATCH>
__global__ __launch_bounds__(256) void k_orbit(const OrbitArgs<T>* __restrict__ dev,
                                               OrbitArgs<T> one) {
    const OrbitArgs<T> A = pick_args<BATCH>(dev, one);
    const int nx = A.nx, ny = A.ny;
    const vec<T, CH>* __restrict__ X = reinterpret_cast<const vec<T, CH>*>(A.X);
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (long)nx * ny) return;
    reinterpret_cast<vec<T, CH * SYM>*>(A.O)[idx] =
        orbit_record<T, CH, SYM>(X, nx, (int)(idx % nx), (int)(idx / nx));
    reinterpret_cast<vec<T, CH * SYM>*>(A.OT)[idx] =
        orbit_record<T, CH, SYM>(X, nx, (int)(idx / ny), (int)(idx % ny));
}

// The same two orbit images for the quarter-turn symmetric square image, by tiles of
// TS x TS pixels: the four rotated TS x TS regions of X that a tile's records draw on
// are loaded into LDS with coalesced reads (each along its own contiguous axis), then
// the tile's records are written to O along i and to OT along j, both coalesced.
template <typename T, int CH, bool BATCH>
__global__ __launch_bounds__(256) void k_orbit_tiled(const OrbitArgs<T>* __restrict__ dev,
                                                     OrbitArgs<T> one) {
    using X1 = vec<T, CH>;
    using R = vec<T, CH * 4>;
    constexpr int TS = 16;
    __shared__ X1 xs[4][TS][TS + 1];  // xs[k][a][b] = X at rot^k(i0 + b, j0 + a)
    const OrbitArgs<T> A = pick_args<BATCH>(dev, one);
    const int n = A.nx;
    const int tiles = (n + TS - 1) / TS;
    if ((int)blockIdx.x >= tiles * tiles) return;  // beyond this slice (whole block)
    const int i0 = (int)(blockIdx.x % tiles) * TS, j0 = (int)(blockIdx.x / tiles) * TS;
    const X1* __restrict__ X = reinterpret_cast<const X1*>(A.X);
    for (int t = threadIdx.x; t < TS * TS; t += blockDim.x) {
        const int u = t / TS, w = t % TS;  // w is the fast index of this pass
        // rot^0 (i, j) and rot^2 (n-1-i, n-1-j): X rows follow a, columns follow b.
        // rot^1 (n-1-j, i) and rot^3 (j, n-1-i): X rows follow b, columns follow a.
        {
            const int a = u, b = w, i = i0 + b, j = j0 + a;
            if (i < n && j < n) {
                xs[0][a][b] = X[(size_t)j * n + i];
                xs[2][a][b] = X[(size_t)(n - 1 - j) * n + (n - 1 - i)];
            }
        }
        {
            const int b = u, a = w, i = i0 + b, j = j0 + a;
            if (i < n && j < n) {
                xs[1][a][b] = X[(size_t)i * n + (n - 1 - j)];
                xs[3][a][b] = X[(size_t)(n - 1 - i) * n + j];
            }
        }
    }
    __syncthreads();
    auto rec = [&](int a, int b) {
        R o;
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int c = 0; c < CH; ++c) o.v[k * CH + c] = xs[k][a][b].v[c];
        return o;
    };
    for (int t = threadIdx.x; t < TS * TS; t += blockDim.x) {
        {
            const int a = t / TS, b = t % TS, i = i0 + b, j = j0 + a;  // along i
            if (i < n && j < n) reinterpret_cast<R*>(A.O)[(size_t)j * n + i] = rec(a, b);
        }
        {
            const int b = t / TS, a = t % TS, i = i0 + b, j = j0 + a;  // along j
            if (i < n && j < n) reinterpret_cast<R*>(A.OT)[(size_t)i * n + j] = rec(a, b);
        }
    }
}

// The CG right-hand side of Eq. (12) (what k_rhs computes) and the orbit images of
// it (what k_orbit_tiled writes) in one launch, for a quarter-turn symmetric square
// image with n % 16 == 0.  A workgroup owns an 8x8 tile of the first quadrant and its
// three rotations: wave k computes r0 on rotation k of the tile in memory order, the
// four tiles' values meet in LDS, and every record of the four tiles is written to O
// along i and to OT along j.  Each partial of |r0|^2 covers the workgroup's 256
// pixels.  The quadrant's tiles are dealt to the XCDs in bands of consecutive tiles,
// so that most stencil neighbours of a tile are read through the same L2.
template <typename T, bool BATCH>
__global__ __launch_bounds__(256) void k_rhs_orbit(const BpArgs<T>* __restrict__ dev,
                                                   BpArgs<T> one,
                                                   const OrbitArgs<T>* __restrict__ odev,
                                                   OrbitArgs<T> oone) {
    using V2 = vec<T, 2>;
    using R = vec<T, 8>;
    constexpr int TS = 8;
    __shared__ V2 xs[4][TS][TS + 1];  // xs[k][a][b] = r0 at rot^k(i0 + b, j0 + a)
    const BpArgs<T> A = pick_args<BATCH>(dev, one);
    const OrbitArgs<T> Ob = pick_args<BATCH>(odev, oone);
    const int n = A.nx;
    const unsigned h = (unsigned)n / (2 * TS), tiles = h * h, id = blockIdx.x;
    if (id >= tiles) return;  // beyond this slice (whole block)
    const unsigned tile =
        tiles % kXcds == 0 ? (id % kXcds) * (tiles / kXcds) + id / kXcds : id;
    const int i0 = (int)(tile % h) * TS, j0 = (int)(tile / h) * TS;
    const int k = (int)(threadIdx.x >> 6), l = (int)(threadIdx.x & 63);
    // Lower corner (ci, cj) of rotation k of the tile [i0, i0 + TS) x [j0, j0 + TS).
    int ci, cj;
    switch (k) {
        case 0: ci = i0; cj = j0; break;
        case 1: ci = n - TS - j0; cj = i0; break;
        case 2: ci = n - TS - i0; cj = n - TS - j0; break;
        default: ci = j0; cj = n - TS - i0; break;
    }
    const int back = (4 - k) & 3;  // rot^back undoes rot^k
    {
        const int pi = ci + (l & (TS - 1)), pj = cj + (l >> 3);
        const size_t pix = (size_t)pj * n + pi;
        T res[2];
        rhs_tracked(A, pix, res);
        double part[2] = {0.0, 0.0};
        epilogue<T, EPI_RHS>(A, pi, pj, res, part);
        int ib, jb;
        rot(back, n, pi, pj, ib, jb);
        V2& d = xs[k][jb - j0][ib - i0];
        d.v[0] = res[0];
        d.v[1] = res[1];
        block_sum_store<2>(part, A.part_img + (size_t)tile * kPartialSlots);
    }
    __syncthreads();
    // The record of pixel P = rot^k(B), B = (i0 + b, j0 + a): component kk of it is r0
    // at rot^kk(P) = rot^(kk + k)(B).
    auto rec = [&](int pi, int pj) {
        int ib, jb;
        rot(back, n, pi, pj, ib, jb);
        const int a = jb - j0, b = ib - i0;
        R o;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int c = 0; c < 2; ++c) o.v[kk * 2 + c] = xs[(kk + k) & 3][a][b].v[c];
        return o;
    };
    {
        const int pi = ci + (l & (TS - 1)), pj = cj + (l >> 3);  // along i
        reinterpret_cast<R*>(Ob.O)[(size_t)pj * n + pi] = rec(pi, pj);
    }
    {
        const int pi = ci + (l >> 3), pj = cj + (l & (TS - 1));  // along j
        reinterpret_cast<R*>(Ob.OT)[(size_t)pi * n + pj] = rec(pi, pj);
    }
}

// The value of x in lane l (uniform).
__device__ inline float lane_value(float x, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}
__device__ inline double lane_value(double x, int l) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// The largest x of the wave, whose lanes are all active.  Row shifts and broadcasts: twelve
// shuffles through LDS took 0.5 us of the 8.6 us of a 101^2 projection.
__device__ inline int wave_max(int x) {
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x111, 0xf, 0xf, false));  // row_shr:1
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x112, 0xf, 0xf, false));  // row_shr:2
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x114, 0xf, 0xf, false));  // row_shr:4
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x118, 0xf, 0xf, false));  // row_shr:8
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x142, 0xa, 0xf, false));  // row_bcast:15
    x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x143, 0xc, 0xf, false));  // row_bcast:31
    return __builtin_amdgcn_readlane(x, 63);
}

// 16 bytes (or the record, if shorter) of a line at a byte offset, zeros past its end: the
// buffer's bounds check extends the line by zeros on both sides (an offset below zero wraps
// far past the end).
template <typename U>
__device__ inline U line_load(__amdgpu_buffer_rsrc_t line, unsigned off) {
    U o;
    if constexpr (sizeof(U) == 16) {
        const auto x = __builtin_amdgcn_raw_buffer_load_b128(line, (int)off, 0, 0);
        __builtin_memcpy(&o, &x, sizeof(U));
    } else if constexpr (sizeof(U) == 8) {
        const auto x = __builtin_amdgcn_raw_buffer_load_b64(line, (int)off, 0, 0);
        __builtin_memcpy(&o, &x, sizeof(U));
    } else {
        const auto x = __builtin_amdgcn_raw_buffer_load_b32(line, (int)off, 0, 0);
        __builtin_memcpy(&o, &x, sizeof(U));
    }
    return o;
}

// R for base rays: QUAD = true writes [Vb][D][SYM][CH] records, false writes the standard
// [V][D][CH] layout (view v + k*Vb for rotation k).  A workgroup owns the rays of 64 / BV
// consecutive bins and RPL BV consecutive base views, BV = RPL views (RPL rays per lane, BV
// views apart), that step along one axis, by the plan's workgroup list (XCD-aware, long
// workgroups first); its KS waves step through KS disjoint ranges of the image
// lines its rays cross (so the lanes of a wave read one image line together) and the waves'
// partial sums are added in order.
//
// Per line a wave stages the kProjWin taps around its mean trajectory in LDS, one orbit
// record per lane in pieces of up to 16 bytes held in separate arrays (16-byte records put
// records r and r + 16, not r + 8, on the same banks), the next line's loads in flight while
// the current one is summed.  Taps past the image's edge are staged as zeros, so a sample's
// weights are those of plain linear interpolation.  LDS takes 13.8 cycles for the write of a
// 16-byte piece by a wave and 4.6 for a read (measured), so a record's two writes cost more
// than a ray's four reads: RPL = 2 halves the writes, loads and loop overhead per ray.
// Measured at 512^2 / 720 x 1024, FP32, two channels: 77 us against 94-101 us
// with one ray per lane and workgroups of both axes; 350 x 301 pixels, 451 x 481 parallel rays,
// one channel: 34 us against 58.  What bounds it now is LDS (50 % of its cycles active) and
// VALU issue (69 %).
//
// Records of 128 bytes (four FP64 channels, quarter-turn symmetric) go in two halves of two
// rotations, a workgroup each (blockIdx.y): 512^2 598 us, 256^2 91 us against 805 and 137
// whole, whose eight pieces of LDS leave room for half the waves and whose sums for none to
// share a line.
template <typename T, int W>
constexpr int proj_parts() {
    return (int)sizeof(T) * W > 64 ? 2 : 1;
}

template <typename T, int CH, int SYM, bool QUAD, int KS, int RPL, bool BATCH>
__global__ __launch_bounds__(64 * KS) void k_project(const ProjArgs<T>* __restrict__ dev,
                                                     const int* __restrict__ list,
                                                     ProjArgs<T> one) {
    constexpr int PARTS = proj_parts<T, CH * SYM>(), SP = SYM / PARTS, W = CH * SP;
    static_assert(!QUAD || PARTS == 1, "quad records are written whole");
    const int part = PARTS == 1 ? 0 : (int)blockIdx.y;  // rotations part SP ... of each record
    using V = vec<T, W>;
    constexpr int CE = W * (int)sizeof(T) > 16 ? 16 / (int)sizeof(T) : W;  // values per piece
    constexpr int NCH = W / CE;
    using VC = vec<T, CE>;
    __shared__ VC s_win[KS][NCH][kProjWin];
    const ProjArgs<T> A = pick_args<BATCH>(dev, one);
    const int nx = A.nx, ny = A.ny, Vb = A.Vb, D = A.D;
    const int BV = RPL * A.views, lbv = __builtin_ctz((unsigned)BV);
    if (BATCH && (int)blockIdx.x >= A.blocks[RPL - 1]) return;  // beyond this slice
    // One slice's list is an argument of its own, in registers when the kernel starts: its entry
    // loads beside the other arguments, not after them (160^2 / 224 x 320, FP32, one channel:
    // 12.1 us against 12.8).
    const int entry = BATCH ? A.order[RPL - 1][blockIdx.x] : list[blockIdx.x];
    const int gy = proj_grid_y(Vb, BV * RPL);
    if (entry < 0) return;
    // The tile (bin group bg, view group vg) and the axis of the rays served.
    const int ax = entry & 1, bg = (entry >> 1) / gy, vg = (entry >> 1) % gy;
    const int n_steps = ax == 0 ? nx : ny;  // samples along a ray
    const int wl = ax == 0 ? ny : nx;       // interpolation axis
    const V* __restrict__ img = reinterpret_cast<const V*>(ax == 0 ? A.OT : A.O) + part;
    const RayParam<T>* __restrict__ rays = A.rays;
    T* __restrict__ sino = A.sino;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = proj_lane_bin(bg, lbv, lane);
    T phi0[RPL], slope[RPL], step[RPL];  // a ray of the other axis, or none: never inside
    bool on[RPL];
    // The lines the workgroup's rays cross: outside a ray's range both taps of every sample
    // are outside the image, so the restriction changes no term.  Every wave holds the same
    // rays, so each computes the same union [s0, s1] of their ranges and takes its KS-th of
    // it (an even split of all lines would leave most waves idle on short chords).  An empty
    // union gives [0, -1]: no wave enters the sample loop.
    int s0 = 1 << 30, s1 = -1;
    bool any = false;
    T acc[RPL][W];
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
        const int v = proj_lane_view(vg, r, RPL, lbv, lane);
        const RayParam<T> q = rays[(size_t)(v < Vb ? v : Vb - 1) * D + (b < D ? b : D - 1)];
        on[r] = b < D && v < Vb && (q.pad == T(0)) == (ax == 0);
        any = any || on[r];
        phi0[r] = on[r] ? q.phi0 : T(-1e30);
        slope[r] = on[r] ? q.slope : T(0);
        step[r] = q.step;
        if (on[r]) {
            int k0, k1;
            proj_ray_range<T>(phi0[r], slope[r], n_steps, wl, k0, k1);
            if (k0 <= k1) {
                s0 = k0 < s0 ? k0 : s0;
                s1 = k1 > s1 ? k1 : s1;
            }
        }
#pragma unroll
        for (int c = 0; c < W; ++c) acc[r][c] = T(0);
    }
    s0 = -wave_max(-s0);
    s1 = wave_max(s1);
    const unsigned long long who = __ballot(any);
    int c0, c1;
    proj_wave_share(s0, s1, wave, KS, c0, c1);
    c0 = __builtin_amdgcn_readfirstlane(c0);  // the same in every lane
    c1 = __builtin_amdgcn_readfirstlane(c1);
    if (c0 <= c1 && who != 0ull) {
        // The window's trajectory: the mean of the extreme rays, the first ray of the first
        // lane and the last of the last lane that hold one.
        const int first = __ffsll((long long)who) - 1, last = 63 - __builtin_clzll(who);
        T pf = phi0[0], sf = slope[0], pl = phi0[RPL - 1], sb = slope[RPL - 1];
        if constexpr (RPL > 1) {
            bool have_f = on[0], have_l = on[RPL - 1];
#pragma unroll
            for (int r = 1; r < RPL; ++r) {
                if (!have_f && on[r]) pf = phi0[r], sf = slope[r], have_f = true;
                const int m = RPL - 1 - r;
                if (!have_l && on[m]) pl = phi0[m], sb = slope[m], have_l = true;
            }
        }
        int wa, wb;
        proj_window_line<T>(lane_value(pf, first), lane_value(sf, first), lane_value(pl, last),
                            lane_value(sb, last), wa, wb);
        wa = __builtin_amdgcn_readfirstlane(wa);
        wb = __builtin_amdgcn_readfirstlane(wb);
        const unsigned line_bytes = proj_line_bytes(wl, PARTS, part, sizeof(V));
        auto load_line = [&](int k, int start, VC (&o)[NCH]) {
            __amdgpu_buffer_rsrc_t line = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<V*>(img + (size_t)k * wl * PARTS), 0, (int)line_bytes, 0x00027000);
            const unsigned off = proj_line_offset(start, lane, PARTS, sizeof(V));
#pragma unroll
            for (int h = 0; h < NCH; ++h) o[h] = line_load<VC>(line, off + h * sizeof(VC));
        };
        VC staged[NCH];
        int s_next = proj_window(wa, wb, c0);
        load_line(c0, s_next, staged);
        for (int k = c0; k <= c1; ++k) {
            const int s0w = s_next;
#pragma unroll
            for (int h = 0; h < NCH; ++h) s_win[wave][h][lane] = staged[h];
            // LDS operations of one wave complete in order; the barrier only keeps the
            // compiler from moving the reads above the write.
            __builtin_amdgcn_wave_barrier();
            if (k < c1) {
                s_next = proj_window(wa, wb, k + 1);
                load_line(k + 1, s_next, staged);
            }
            const T kf = (T)k;
            bool out = false;
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                const T ph = fma(slope[r], kf, phi0[r]);
                const T fl = floor(ph);
                const T w1 = ph - fl, w0 = T(1) - w1;
                const unsigned idx = (unsigned)((int)fl - s0w);
                if (idx <= (unsigned)(kProjWin - 2)) {
#pragma unroll
                    for (int h = 0; h < NCH; ++h) {
                        const VC x0 = s_win[wave][h][idx], x1 = s_win[wave][h][idx + 1];
#pragma unroll
                        for (int c = 0; c < CE; ++c) {
                            T& a = acc[r][h * CE + c];
                            a = fma(w0, x0.v[c], a);
                            a = fma(w1, x1.v[c], a);
                        }
                    }
                } else {
                    out = out || (ph > T(-1) && ph < (T)wl);
                }
            }
            if (__any(out)) {  // rays outside the window (rare): from the image itself
#pragma unroll
                for (int r = 0; r < RPL; ++r) {
                    const T ph = fma(slope[r], kf, phi0[r]);
                    const unsigned idx = (unsigned)((int)floor(ph) - s0w);
                    if (idx > (unsigned)(kProjWin - 2) && ph > T(-1) && ph < (T)wl) {
                        T w0, w1;
                        const int j = proj_taps<T>(phi0[r], slope[r], kf, wl, w0, w1);
                        const V* q = img + ((size_t)k * wl + j) * PARTS;
                        const V a0 = q[0], a1 = q[PARTS];
#pragma unroll
                        for (int c = 0; c < W; ++c)
                            acc[r][c] = fma(w1, a1.v[c], fma(w0, a0.v[c], acc[r][c]));
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
        // A sum that is not finite is formed again from the taps that have weight: a ray that
        // passes exactly over a line of pixels, or exactly one line outside the image, took the
        // next pixel with weight zero above, and an infinity there is none of its own.
#pragma unroll
        for (int r = 0; r < RPL; ++r) {
            bool finite = true;
#pragma unroll
            for (int c = 0; c < W; ++c) finite = finite && isfinite(acc[r][c]);
            if (finite) continue;
#pragma unroll
            for (int c = 0; c < W; ++c) acc[r][c] = T(0);
#pragma unroll 1
            for (int k = c0; k <= c1; ++k) {
                T w0, w1;
                const int j = proj_taps<T>(phi0[r], slope[r], (T)k, wl, w0, w1);
                const V* q = img + ((size_t)k * wl + j) * PARTS;
                if (w0 > T(0))
#pragma unroll
                    for (int c = 0; c < W; ++c) acc[r][c] = fma(w0, q[0].v[c], acc[r][c]);
                if (w1 > T(0))
#pragma unroll
                    for (int c = 0; c < W; ++c) acc[r][c] = fma(w1, q[PARTS].v[c], acc[r][c]);
            }
        }
    }
    // The waves' sums meet in their windows, one ray of every lane at a time; wave r % KS
    // adds those of ray r in wave order and stores them.
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
        if (r > 0) __syncthreads();
#pragma unroll
        for (int c = 0; c < W; ++c) s_win[wave][c / CE][lane].v[c % CE] = acc[r][c];
        __syncthreads();
        if (wave != r % KS || !on[r]) continue;
        const int v = proj_lane_view(vg, r, RPL, lbv, lane);
        T sum[W];
#pragma unroll
        for (int c = 0; c < W; ++c) sum[c] = s_win[0][c / CE][lane].v[c % CE];
        for (int w = 1; w < KS; ++w)
#pragma unroll
            for (int c = 0; c < W; ++c) sum[c] += s_win[w][c / CE][lane].v[c % CE];
        if constexpr (QUAD) {
            V out;
#pragma unroll
            for (int c = 0; c < W; ++c) out.v[c] = sum[c] * step[r];
            reinterpret_cast<V*>(sino)[(size_t)v * D + b] = out;
        } else {
#pragma unroll
            for (int s = 0; s < SP; ++s) {
                vec<T, CH> out;
#pragma unroll
                for (int c = 0; c < CH; ++c) out.v[c] = sum[s * CH + c] * step[r];
                const int vs = v + (part * SP + s) * Vb;
                reinterpret_cast<vec<T, CH>*>(sino)[(size_t)vs * D + b] = out;
            }
        }
    }
}

template <typename T>
__device__ inline T fast_rcp(T x) { return T(1) / x; }
template <>
__device__ inline float fast_rcp<float>(float x) { return __builtin_amdgcn_rcpf(x); }

// The transposed gather of one wave: an 8x8 block of pixel orbits, one orbit per lane.
//
// Pixel rot^k(p) seen from view v + k' Vb has the weight of base view v at pixel
// rot^(k - k')(p), so for every orbit member p_m = rot^m(p) the base-view weights are
// evaluated once and routed to acc[(m + k') mod SYM] with the sinogram value of view
// v + k' Vb, for all k'.
//
// Candidates of a pixel are the bins within h of its detector coordinate beta, h the largest
// change of beta over one pixel along an axis (a ray more than one pixel step away along its
// minor axis has no tap on the pixel); the weight max(0, step (1 - |d|)) of a candidate, d its signed
// minor-axis distance, is the projector's linear-interpolation weight.
//
// Per view and member ("slot") the block's candidates lie in a window of kBpWin bins.
// The window, and where each pixel's candidates start in it, come from one plane per
// slot: beta is projective in the pixel, beta - beta0 = (g.t) / (1 + e.t) with t the
// offset from the block's centre, g its gradient there and e the relative gradient of the
// denominator, so an affine beta is off by at most
//   E = |t|^2 / 2 (|g||e| + |g.e|) / (1 - q),  q = max|e.t|,
// and h by no more than the bound hb formed in bp_slot.  Each pixel then takes the C =
// ceil(2 hb + 2 E) bins from floor(plane) + 1 on: all its candidates are among them, the
// others have weight exactly zero, and C is the same for the whole wave.  The planes of
// kBpBatch slots at a time are formed by the wave's lanes (one each) and kept in LDS, so a
// pixel spends four instructions per slot on its footprint instead of about thirty.
//
// The windows of kBpSlots slots are staged at once, one record (ray record and the SYM *
// CH sinogram values of the bin) per lane, the next group's loads in flight while the
// current one is summed.  A record is held in 16-byte pieces, each piece an array of its
// own, so that lanes reading neighbouring records never meet on a bank.
//
// A slot whose window would be too long (a block so near the source that the fan spreads
// over more than kBpWin bins), and every slot of a wave whose sums came out non-finite
// (zero weights must not carry a NaN or an infinity of the sinogram to other pixels), is
// gathered candidate by candidate from global memory, those without weight left out.
//
// What bounds it: LDS and VALU issue, about equally.  Per view and 64 pixels at
// 512^2 / 720 x 1024 (two channels, FP32) 204 VALU instructions (341 with a footprint per
// pixel, which took 62.9 M per launch against 37.2 M) and 46 LDS instructions of which the
// 34 candidate reads take 4.6 cycles each and the 6 staging writes 13.8 (measured alone).
// A launch takes 102-111 us (118-122 us before, at 4 waves per workgroup, 110-114 at 8);
// 27 us at 256^2 (58 and 38); a plain one-channel transpose of 350 x 301 pixels over 451 x 481
// parallel rays 46 us (97).
constexpr int kBpSlots = 2;
constexpr int kBpBatch = 64;

// Sinograms of one and two channels are read by quarter-turn symmetric plans as quad records
// ([Vb][D][SYM][CH]: one 16- or 32-byte load per record); four channels are 16-byte pieces in
// their views' own rows already, and read there they share no scratch between calls (FP32 and
// FP64: 256^2 32 and 59 us against 38 and 77 us reordered, 512^2 188 and 338 against 194 and
// 422; 1024^2 FP32 1388 against 1295).
constexpr bool bp_quads(int ch, int sym) { return sym == 4 && ch < 4; }

// Pieces of a staged record: the ray record in 16-byte pieces, the values in 16-byte
// pieces or, below 16 bytes, in one piece of their size.
template <typename T, int W>
struct BpWindow {
    static constexpr int PE = 16 / (int)sizeof(T);  // values per 16 bytes
    static constexpr int RC = 4 / PE;               // pieces of a ray record
    static constexpr int VE = W < PE ? W : PE;      // values per value piece
    static constexpr int VC = W / VE;
    vec<T, PE> ray[RC][kBpWin * kBpSlots];
    vec<T, VE> val[VC][kBpWin * kBpSlots];
};

template <typename T, typename A, int CH, int SYM, int VS>
__device__ inline void gather_windows(const BpArgs<T>& a, int wave, int lane, int bx, int by,
                                      BpWindow<T, CH * SYM>& win, BpSlot* slots,
                                      A (&acc)[SYM][CH]) {
    constexpr int W = CH * SYM;
    using Win = BpWindow<T, W>;
    // A group is kBpSlots slots staged together: SYM / kBpSlots groups per view, or one
    // group of kBpSlots views.
    constexpr int GPV = SYM == 4 ? SYM / kBpSlots : 1;  // groups per view step
    constexpr int VPG = SYM == 4 ? 1 : kBpSlots;        // views per group
    constexpr int SPV = GPV * kBpSlots;                 // slots per view step
    constexpr int STEPS = kBpBatch / SPV;               // view steps per batch of slots
    const int D = a.D, Vb = a.Vb, n = a.nx;
    const int i0 = bx * 8, j0 = by * 8;
    const int i = i0 + (lane & 7), j = j0 + (lane >> 3);
    const float oi = (float)(lane & 7), oj = (float)(lane >> 3);
    using GC = const __attribute__((address_space(1))) char;

    // A U at byte `off` of a row (uniform base, 32-bit offset).
    auto load = [&](auto tag, const void* row, unsigned off) {
        using U = decltype(tag);
        using GU = const __attribute__((address_space(1))) U;
        GU* q = (GU*)((GC*)row + off);
        U o;
        using GT = const __attribute__((address_space(1))) T;
#pragma unroll
        for (unsigned c = 0; c < sizeof(U) / sizeof(T); ++c)
            reinterpret_cast<T*>(&o)[c] = ((GT*)q)[c];
        return o;
    };
    auto ray_at = [&](int v, unsigned b) {
        const BpRay<T>* row = a.brays + (size_t)v * (unsigned)(D + 1);
        return load(BpRay<T>{}, row, b * (unsigned)sizeof(BpRay<T>));
    };
    // The values of bin b of base view v in all SYM views it stands for (a record, or CH values
    // of each view's row).
    auto values_at = [&](int v, unsigned b, T (&s)[W]) {
        constexpr int ROWS = bp_quads(CH, SYM) ? 1 : SYM, R = W / ROWS;
#pragma unroll
        for (int k = 0; k < ROWS; ++k) {
            const vec<T, R> t = load(vec<T, R>{}, a.sino + (size_t)(v + k * Vb) * (unsigned)D * R,
                                     b * (unsigned)sizeof(vec<T, R>));
#pragma unroll
            for (int c = 0; c < R; ++c) s[k * R + c] = t.v[c];
        }
    };
    // Record `lane` of the window written; record o read.
    auto store = [&](const BpRay<T>& r, const T (&s)[W]) {
        const T* rp = &r.phi0;
#pragma unroll
        for (int h = 0; h < Win::RC; ++h)
#pragma unroll
            for (int c = 0; c < Win::PE; ++c) win.ray[h][lane].v[c] = rp[h * Win::PE + c];
#pragma unroll
        for (int h = 0; h < Win::VC; ++h)
#pragma unroll
            for (int c = 0; c < Win::VE; ++c) win.val[h][lane].v[c] = s[h * Win::VE + c];
    };
    auto fetch = [&](int o, BpRay<T>& r, T (&s)[W]) {
        T* rp = &r.phi0;
#pragma unroll
        for (int h = 0; h < Win::RC; ++h)
#pragma unroll
            for (int c = 0; c < Win::PE; ++c) rp[h * Win::PE + c] = win.ray[h][o].v[c];
#pragma unroll
        for (int h = 0; h < Win::VC; ++h)
#pragma unroll
            for (int c = 0; c < Win::VE; ++c) s[h * Win::VE + c] = win.val[h][o].v[c];
    };
    auto weight = [&](const BpRay<T>& r, T fi, T fj) {
        const T d = fma(r.ci, fi, fma(r.cj, fj, r.phi0));
        return fmax(T(0), fma(-r.step, fabs(d), r.step));
    };
    // Base view of slot sl of view step t of this wave: view (SYM = 4) or kBpSlots
    // consecutive views (SYM = 1) number wave, wave + VS, ...
    auto view_of = [&](int t, int sl) {
        return SYM == 4 ? wave + VS * t : (wave + VS * t) * VPG + sl;
    };
    const int nsteps = (Vb + VPG - 1) / VPG;
    const int mine = nsteps > wave ? (nsteps - wave + VS - 1) / VS : 0;

    int redo = 0;
    for (;;) {
        asm volatile("" : "+s"(redo));  // one loop body for both passes
#pragma unroll 1
        for (int t0 = 0; t0 < mine; t0 += STEPS) {
            const int nt = mine - t0 < STEPS ? mine - t0 : STEPS;
            unsigned long long left;
            {  // this lane's slot of the batch
                const int t = lane / SPV, sl = lane % SPV, v = view_of(t0 + t, sl);
                BpSlot e{0.0f, 0.0f, 0.0f, 0};
                if (t < nt && v < Vb) {
                    e = bp_slot<SYM>(a.views[v], SYM == 4 ? sl : 0, i0, j0, n, a.ny, D);
                    if (redo && (e.info & 255) != 0) e.info = kBpDirect;
                }
                left = __ballot((e.info & (kBpDirect | kBpLong)) != 0);
                slots[lane] = e;
                __builtin_amdgcn_wave_barrier();
            }
            if (!redo) {
                // Record `lane` of a group: bin lane % kBpWin of slot lane / kBpWin; off the
                // detector the zero record that ends each row of the ray table.
                BpRay<T> pr;
                T pv[W];
                const int ssl = lane / kBpWin, sk = lane % kBpWin;
                auto stage = [&](int t, int g) {
                    const unsigned b =
                        (unsigned)(bp_slot_window(slots[t * SPV + g * kBpSlots + ssl].info) + sk);
                    const unsigned br = min(b, (unsigned)D), bs = min(b, (unsigned)(D - 1));
                    if constexpr (SYM == 4) {
                        const int v = view_of(t0 + t, 0);
                        pr = ray_at(v, br);
                        values_at(v, bs, pv);
                    } else {
                        // Two views: the second one's row is one stride further (the last
                        // row is its own partner when the views run out; its slot has C = 0).
                        const int v = view_of(t0 + t, 0);
                        const unsigned more = v + 1 < Vb ? (unsigned)ssl : 0u;
                        pr = ray_at(v, br + more * (unsigned)(D + 1));
                        values_at(v, bs + more * (unsigned)D, pv);
                    }
                };
                stage(0, 0);
#pragma unroll 1
                for (int t = 0; t < nt; ++t) {
#pragma unroll
                    for (int g = 0; g < GPV; ++g) {
                        BpSlot e[kBpSlots];
#pragma unroll
                        for (int sl = 0; sl < kBpSlots; ++sl)
                            e[sl] = slots[t * SPV + g * kBpSlots + sl];
                        store(pr, pv);
                        // LDS operations of one wave complete in order; the barrier only
                        // keeps the compiler from moving the reads above the writes.
                        __builtin_amdgcn_wave_barrier();
                        if (g + 1 < GPV) stage(t, g + 1);
                        else if (t + 1 < nt) stage(t + 1, 0);
#pragma unroll
                        for (int sl = 0; sl < kBpSlots; ++sl) {
                            const int mm = SYM == 4 ? g * kBpSlots + sl : 0;
                            int im, jm;
                            rot(mm, n, i, j, im, jm);
                            const T fi = (T)im, fj = (T)jm;
                            const int C = __builtin_amdgcn_readfirstlane(e[sl].info) & 255;
                            const int o = sl * kBpWin + bp_slot_start(e[sl], oi, oj);
                            auto take = [&](int k) {
                                BpRay<T> r;
                                T s[W];
                                fetch(o + k, r, s);
                                const T wt = weight(r, fi, fj);
#pragma unroll
                                for (int kp = 0; kp < SYM; ++kp)
#pragma unroll
                                    for (int c = 0; c < CH; ++c) {
                                        A& x = acc[(mm + kp) % SYM][c];
                                        x = fma((A)wt, (A)s[kp * CH + c], x);
                                    }
                            };
                            if ((unsigned)(C - 1) < (unsigned)(kBpLong - 1)) {
                                take(0);
                                take(1);
#pragma unroll 1
                                for (int k = 2; k < C; ++k) take(k);
                            }
                        }
                        __builtin_amdgcn_wave_barrier();
                    }
                }
            }
#pragma unroll 1
            while (left) {  // slots with long windows, and direct ones
                const int s0 = __ffsll((long long)left) - 1;
                left &= left - 1;
                const int v = view_of(t0 + s0 / SPV, s0 % SPV), mm = SYM == 4 ? s0 % SPV : 0;
                int im, jm;
                rot(mm, n, i, j, im, jm);
                const T fi = (T)im, fj = (T)jm;
                A sum[W];
#pragma unroll
                for (int c = 0; c < W; ++c) sum[c] = A(0);
                auto add = [&](T wt, const T (&s)[W]) {
#pragma unroll
                    for (int c = 0; c < W; ++c) sum[c] = fma((A)wt, (A)s[c], sum[c]);
                };
                const BpSlot e = slots[s0];
                const int info = __builtin_amdgcn_readfirstlane(e.info);
                if (info & kBpLong) {  // one slot staged by all lanes
                    const unsigned b = (unsigned)(bp_slot_window(info) + lane);
                    T s[W];
                    BpRay<T> r = ray_at(v, min(b, (unsigned)D));
                    values_at(v, min(b, (unsigned)(D - 1)), s);
                    store(r, s);
                    __builtin_amdgcn_wave_barrier();
                    const int o = bp_slot_start(e, oi, oj), C = info & (kBpLong - 1);
                    for (int k = 0; k < C; ++k) {
                        fetch(o + k, r, s);
                        add(weight(r, fi, fj), s);
                    }
                    __builtin_amdgcn_wave_barrier();
                } else {  // candidate by candidate from global memory
                    const ViewParam<T> w = a.views[v];
                    const T ip = fi - T(0.5) * (T)(n - 1), jp = fj - T(0.5) * (T)(a.ny - 1);
                    const T inv = fast_rcp<T>(w.d0 + w.di * ip + w.dj * jp);
                    const T bq = (w.ni * ip + w.nj * jp) * inv;
                    // A point one pixel away along an axis is off by |g| / (1 - |e|) at most
                    // (|e| < 1/2: the source is two pixels outside the image's circle).
                    const T h =
                        fmax(fabs((w.nj - bq * w.dj) * inv) / (T(1) - fabs(w.dj * inv)),
                             fabs((w.ni - bq * w.di) * inv) / (T(1) - fabs(w.di * inv))) +
                        T(0.02);
                    const T bc = bq + w.boff;
                    const int lo = (int)ceil(fmin(fmax(bc - h, T(0)), (T)D));
                    const int hi = (int)floor(fmax(fmin(bc + h, (T)(D - 1)), T(-1)));
                    for (int b = lo; b <= hi; ++b) {
                        const T wt = weight(ray_at(v, (unsigned)b), fi, fj);
                        if (!(wt > T(0))) continue;  // nothing of it, finite or not
                        T s[W];
                        values_at(v, (unsigned)b, s);
                        add(wt, s);
                    }
                }
#pragma unroll
                for (int m = 0; m < SYM; ++m)
                    if (m == mm)
#pragma unroll
                        for (int kp = 0; kp < SYM; ++kp)
#pragma unroll
                            for (int c = 0; c < CH; ++c)
                                acc[(m + kp) % SYM][c] += sum[kp * CH + c];
            }
        }
        bool finite = true;
#pragma unroll
        for (int k = 0; k < SYM; ++k)
#pragma unroll
            for (int c = 0; c < CH; ++c) finite = finite && isfinite(acc[k][c]);
        if (redo || !__any(!finite)) break;
        redo = 1;
#pragma unroll
        for (int k = 0; k < SYM; ++k)
#pragma unroll
            for (int c = 0; c < CH; ++c) acc[k][c] = A(0);
    }
}

// R^T (+ epilogue).  A workgroup owns an 8x8 block of pixel orbits (the block
// lies in the first quadrant when SYM = 4) and has VS waves, each summing a
// disjoint subset of the base views.  Sinograms are records of the SYM views of a base
// ray (bp_quads) or plain.  A: the type the sums are kept in (T, or double for an FP32
// plan's sums in double precision: each product of two FP32 values is exact in double, so
// only the sums round); the finished values are rounded to T once.
//
// Waves per SIMD that the registers are held to (the second launch bound).  The staged gather
// waits on LDS, so it wants as many waves as its registers allow; what is spilled for them (FP32
// two-channel quad records: 12 to 18 values a lane, 50 MB of writes at 512^2) is the batch's
// set-up and the epilogue, outside the candidate loops.  At 4 waves, without spills, the q
// transpose takes 118 us against 101.6 at 512^2 and a plain one of 350 x 301 pixels 69 against
// 54, but at 256^2 24.4 against 26.6 and at 1024^2 681 against 704.
template <typename T, typename A, int W>
constexpr int bp_min_waves() {
    if (sizeof(T) == 8) return W <= 2 ? 6 : W <= 4 ? 5 : W <= 8 ? 3 : 2;
    if (sizeof(A) == 8) return W <= 2 ? 8 : 5;
    return W <= 8 ? 8 : 5;
}

template <typename T, int CH, int SYM, int EPI, int VS, bool BATCH, typename A = T>
__global__ __launch_bounds__(64 * VS, (bp_min_waves<T, A, CH * SYM>())) void k_backproject(
    const BpArgs<T>* __restrict__ dev, BpArgs<T> one, unsigned nslices) {
    constexpr int W = SYM * CH;
    // Each wave's staging window; once its view sums are done it stores them over it.
    using Win = BpWindow<T, W>;
    union alignas(16) Row {
        Win win;
        A sum[64][W];
        __device__ Row() {}
    };
    __shared__ Row s_row[VS];
    __shared__ BpSlot s_slot[VS][kBpBatch];
    // The orbit block (bx, by) of this workgroup: by launch position in the plan's order; in
    // a batch each XCD takes an equal contiguous share of the slices' positions (one.gx,
    // one.gy: the group's block grid, the same for all its slices).
    unsigned slice = 0, pos = blockIdx.x;
    if constexpr (BATCH) {
        if (!xcd_slice_tile(blockIdx.x, (unsigned)(one.gx * one.gy), nslices, slice, pos)) return;
    }
    const BpArgs<T> a = pick_args<BATCH>(dev, one, slice);
    const int tile = a.order[pos], bx = tile % a.gx, by = tile / a.gx;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    A acc[SYM][CH];
#pragma unroll
    for (int k = 0; k < SYM; ++k)
#pragma unroll
        for (int c = 0; c < CH; ++c) acc[k][c] = A(0);
    gather_windows<T, A, CH, SYM, VS>(a, wave, lane, bx, by, s_row[wave].win, s_slot[wave],
                                            acc);
    // Every wave's view sums go to LDS; wave w then finishes orbit members w, w + VS, ...:
    // it adds the waves' sums in wave order and stores the member's pixels or runs its
    // epilogue, whose partials it reduces over its lanes; thread 0 adds the members'
    // partials in member order.
#pragma unroll
    for (int k = 0; k < SYM; ++k)
#pragma unroll
        for (int c = 0; c < CH; ++c) s_row[wave].sum[lane][k * CH + c] = acc[k][c];
    __shared__ double wpart[SYM][2];
    __syncthreads();
    const int i = bx * 8 + (lane & 7), j = by * 8 + (lane >> 3);
    const int dom_x = SYM == 4 ? a.nx / 2 : a.nx, dom_y = SYM == 4 ? a.ny / 2 : a.ny;
    const bool inside = i < dom_x && j < dom_y;
    for (int k = wave; k < SYM; k += VS) {
        A sum[CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) sum[c] = A(0);
        for (int w = 0; w < VS; ++w)
#pragma unroll
            for (int c = 0; c < CH; ++c) sum[c] += s_row[w].sum[lane][k * CH + c];
        int io, jo;
        rot(k, a.nx, i, j, io, jo);
        if constexpr (EPI == EPI_NONE) {
            if (inside) {
                vec<T, CH> o;
#pragma unroll
                for (int c = 0; c < CH; ++c) o.v[c] = (T)sum[c];
                reinterpret_cast<vec<T, CH>*>(a.out)[(size_t)jo * a.nx + io] = o;
            }
        } else {
            T res[2] = {(T)sum[0], (T)sum[CH > 1 ? 1 : 0]};
            double part[2] = {0.0, 0.0};
            if (inside) epilogue<T, EPI>(a, io, jo, res, part);
#pragma unroll
            for (int c = 0; c < 2; ++c)
                for (int off = 32; off > 0; off >>= 1) part[c] += __shfl_down(part[c], off, 64);
            if (lane == 0) {
                wpart[k][0] = part[0];
                wpart[k][1] = part[1];
            }
        }
    }
    if constexpr (EPI != EPI_NONE) {
        __syncthreads();
        if (threadIdx.x == 0) {
            double o0 = 0.0, o1 = 0.0;
            for (int k = 0; k < SYM; ++k) {
                o0 += wpart[k][0];
                o1 += wpart[k][1];
            }
            double* o = a.partials + (size_t)(by * a.gx + bx) * kPartialSlots;
            o[0] = o0;
            o[1] = o1;
        }
    }
}

// Waves per workgroup of the plain projector; the other kernels take theirs from the plan
// (2, 4 or 8; see dect_plan_tune).  8 projector
// waves took the LM1 x CG1 iteration at 512^2 from 1.01 to 0.96 ms against 4.
constexpr int kLineSplit = 8;

template <typename T, int CH, int SYM, bool QUAD, bool BATCH, int KS>
void project_launch(const OrbitArgs<T>* odev, const OrbitArgs<T>& oone, const ProjArgs<T>* pdev,
                    const ProjArgs<T>& pone, int n, long pixels, hipStream_t s, bool orbit) {
    if (orbit) {
        ProfScope pt("orbit", s);
        if constexpr (SYM == 4) {
            constexpr int TS = 16;
            const unsigned tiles = (unsigned)((oone.nx + TS - 1) / TS);
            hipLaunchKernelGGL((k_orbit_tiled<T, CH, BATCH>), dim3(tiles * tiles, 1, n), dim3(256),
                               0, s, odev, oone);
        } else {
            hipLaunchKernelGGL((k_orbit<T, CH, SYM, BATCH>), dim3((unsigned)((pixels + 255) / 256), 1, n),
                               dim3(256), 0, s, odev, oone);
        }
    }
    ProfScope pp("project", s);
    constexpr int PARTS = proj_parts<T, CH * SYM>();
    const int R = proj_rays((int)sizeof(T) * CH * SYM / PARTS, pone.Vb, pone.D, pone.views, KS);
    // A batch's slices may have lists of different lengths (pone.grid: the longest).
    const dim3 g((unsigned)(BATCH ? std::max(pone.grid, pone.blocks[R - 1]) : pone.blocks[R - 1]),
                 PARTS, n);
    if (R == 2)
        hipLaunchKernelGGL((k_project<T, CH, SYM, QUAD, KS, 2, BATCH>), g, dim3(64 * KS), 0, s,
                           pdev, pone.order[R - 1], pone);
    else
        hipLaunchKernelGGL((k_project<T, CH, SYM, QUAD, KS, 1, BATCH>), g, dim3(64 * KS), 0, s,
                           pdev, pone.order[R - 1], pone);
}

template <typename T, int CH, int SYM, bool QUAD, int KS>
hipError_t project_t(const OrbitArgs<T>* odev, const OrbitArgs<T>& oone,
                     const ProjArgs<T>* pdev, const ProjArgs<T>& pone, int n, long pixels,
                     hipStream_t s, bool orbit = true) {
    if (odev)
        project_launch<T, CH, SYM, QUAD, true, KS>(odev, oone, pdev, pone, n, pixels, s, orbit);
    else
        project_launch<T, CH, SYM, QUAD, false, KS>(odev, oone, pdev, pone, n, pixels, s, orbit);
    return hipGetLastError();
}

// A standard [V][D][CH] sinogram as quad records [Vb][D][4][CH] (view v + k Vb is
// rotation k of base view v), times the ray weights if there are any, the layout the
// transpose of a quarter-turn symmetric plan reads: one record per thread, the four views' rows
// read and the records written along b.
template <typename T, int CH>
__global__ __launch_bounds__(256) void k_quad_records(const T* __restrict__ sino,
                                                      const T* __restrict__ weight, int Vb, int D,
                                                      T* __restrict__ quad) {
    const long r = (long)blockIdx.x * blockDim.x + threadIdx.x;  // (vb, b)
    const long rows = (long)Vb * D;
    if (r >= rows) return;
    vec<T, 4 * CH> o;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const vec<T, CH> t = reinterpret_cast<const vec<T, CH>*>(sino)[r + k * rows];
#pragma unroll
        for (int c = 0; c < CH; ++c) o.v[k * CH + c] = t.v[c];
        if (weight) {
#pragma unroll
            for (int c = 0; c < CH; ++c) o.v[k * CH + c] *= weight[r + k * rows];
        }
    }
    reinterpret_cast<vec<T, 4 * CH>*>(quad)[r] = o;
}

// Plain R^T of a standard [V][D][CH] sinogram with `waves` waves per workgroup; on a
// quarter-turn symmetric plan one or two channels are first reordered into quad records (plan
// scratch): staging two channels straight from the four views' rows measured 146 us against
// 105 us + 4 us.
template <typename T, int CH, int SYM, int VS>
hipError_t bp_plain(const BpArgs<T>& one, T* quad, hipStream_t s) {
    BpArgs<T> a = one;
    if constexpr (bp_quads(CH, SYM)) {
        const long recs = (long)one.Vb * one.D;
        hipLaunchKernelGGL((k_quad_records<T, CH>), dim3((unsigned)((recs + 255) / 256)), dim3(256),
                           0, s, one.sino, one.weight, one.Vb, one.D, quad);
        a.sino = quad;
    }
    hipLaunchKernelGGL((k_backproject<T, CH, SYM, EPI_NONE, VS, false>), dim3(one.gx * one.gy),
                       dim3(64 * VS), 0, s, nullptr, a, 1u);
    return hipGetLastError();
}

template <typename T, int CH, int SYM>
hipError_t bp_plain_w(int waves, const BpArgs<T>& one, T* quad, hipStream_t s) {
    switch (bp_waves_for(sizeof(T), CH * SYM, waves, one.gx * one.gy)) {
        case 2: return bp_plain<T, CH, SYM, 2>(one, quad, s);
        case 4: return bp_plain<T, CH, SYM, 4>(one, quad, s);
        case 8: return bp_plain<T, CH, SYM, 8>(one, quad, s);
        case 16:
            if constexpr (sizeof(T) == 4 || CH * SYM <= 4)
                return bp_plain<T, CH, SYM, 16>(one, quad, s);
    }
    return hipErrorInvalidValue;
}

// The ADMM's own sinograms are two-channel quad records.
template <typename T, int SYM, bool BATCH, int VS, typename A>
hipError_t bp_admm_t(int epi, const BpArgs<T>* dev, const BpArgs<T>& one, int n, int gx, int gy,
                     hipStream_t s) {
    // One slice: a workgroup per block.  A batch: each XCD an equal contiguous share of the
    // slices' blocks; the kernel takes the block grid from `one`, the same for every slice
    // of the group.
    if (gx != one.gx || gy != one.gy) return hipErrorInvalidValue;
    const dim3 g(BATCH ? xcd_slice_blocks((unsigned)(gx * gy), (unsigned)n) : (unsigned)(gx * gy));
    const dim3 blk(64 * VS);
    const unsigned nsl = (unsigned)n;
    switch (epi) {
        case EPI_Q:
            hipLaunchKernelGGL((k_backproject<T, 2, SYM, EPI_Q, VS, BATCH, A>), g, blk, 0, s,
                               dev, one, nsl);
            break;
        case EPI_DUAL:
            hipLaunchKernelGGL((k_backproject<T, 2, SYM, EPI_DUAL, VS, BATCH, A>), g, blk, 0,
                               s, dev, one, nsl);
            break;
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename T, int SYM, bool BATCH, typename A>
hipError_t bp_admm_w(int waves, int epi, const BpArgs<T>* dev, const BpArgs<T>& one, int n, int gx,
                     int gy, hipStream_t s) {
    switch (bp_waves_for(sizeof(T), 2 * SYM, waves, gx * gy)) {
        case 2: return bp_admm_t<T, SYM, BATCH, 2, A>(epi, dev, one, n, gx, gy, s);
        case 4: return bp_admm_t<T, SYM, BATCH, 4, A>(epi, dev, one, n, gx, gy, s);
        case 8: return bp_admm_t<T, SYM, BATCH, 8, A>(epi, dev, one, n, gx, gy, s);
        case 16:
            if constexpr (sizeof(T) == 4 || SYM == 1)
                return bp_admm_t<T, SYM, BATCH, 16, A>(epi, dev, one, n, gx, gy, s);
    }
    return hipErrorInvalidValue;
}

template <typename T, int SYM, typename A>
hipError_t bp_admm(int waves, int epi, const BpArgs<T>* dev, const BpArgs<T>& one, int n, int gx,
                   int gy, hipStream_t s) {
    return dev ? bp_admm_w<T, SYM, true, A>(waves, epi, dev, one, n, gx, gy, s)
               : bp_admm_w<T, SYM, false, A>(waves, epi, dev, one, n, gx, gy, s);
}

template <typename T, int SYM>
hipError_t project_pair_w(int waves, const OrbitArgs<T>* odev, const OrbitArgs<T>& oone,
                          const ProjArgs<T>* pdev, const ProjArgs<T>& pone, int n, long pixels,
                          hipStream_t s, bool orbit) {
    switch (waves) {
        case 2: return project_t<T, 2, SYM, true, 2>(odev, oone, pdev, pone, n, pixels, s, orbit);
        case 4: return project_t<T, 2, SYM, true, 4>(odev, oone, pdev, pone, n, pixels, s, orbit);
        case 8: return project_t<T, 2, SYM, true, 8>(odev, oone, pdev, pone, n, pixels, s, orbit);
    }
    return hipErrorInvalidValue;
}

const char* bp_name(int epi) {
    static const char* names[4] = {"backproject", "backproject_rhs", "backproject_q",
                                   "backproject_dual"};
    return names[epi & 3];
}

}  // namespace

template <typename T>
void fill_bp_plan(const dect_plan* p, BpArgs<T>& a) {
    a.brays = static_cast<const BpRay<T>*>(p->bp_rays);
    a.views = static_cast<const ViewParam<T>*>(p->views);
    a.nx = p->nx;
    a.ny = p->ny;
    a.Vb = p->Vb;
    a.D = p->D;
    const int dx = p->sym == 4 ? p->nx / 2 : p->nx, dy = p->sym == 4 ? p->ny / 2 : p->ny;
    a.gx = (dx + 7) / 8;
    a.gy = (dy + 7) / 8;
    a.order = p->bp_order;
}

// R into the standard sinogram layout, with the two orbit images of the image in O and
// OT (each N * ch * sym values of T).
template <typename T>
hipError_t launch_project_with(const dect_plan* p, const void* img, void* sino, int ch, void* O_,
                               void* OT_, hipStream_t s) {
    T* O = static_cast<T*>(O_);
    T* OT = static_cast<T*>(OT_);
    OrbitArgs<T> o{static_cast<const T*>(img), O, OT, p->nx, p->ny};
    ProjArgs<T> q{static_cast<const RayParam<T>*>(p->rays), O, OT, static_cast<T*>(sino), p->nx,
                  p->ny, p->Vb, p->D};
    proj_take_shape(q, *p->pj_shape.load());
    if (p->sym == 4) {
        switch (ch) {
            case 1: return project_t<T, 1, 4, false, kLineSplit>(nullptr, o, nullptr, q, 1, p->N, s);
            case 2: return project_t<T, 2, 4, false, kLineSplit>(nullptr, o, nullptr, q, 1, p->N, s);
            case 4: return project_t<T, 4, 4, false, kLineSplit>(nullptr, o, nullptr, q, 1, p->N, s);
        }
    } else {
        switch (ch) {
            case 1: return project_t<T, 1, 1, false, kLineSplit>(nullptr, o, nullptr, q, 1, p->N, s);
            case 2: return project_t<T, 2, 1, false, kLineSplit>(nullptr, o, nullptr, q, 1, p->N, s);
            case 4: return project_t<T, 4, 1, false, kLineSplit>(nullptr, o, nullptr, q, 1, p->N, s);
        }
    }
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_project(const dect_plan* p, const void* img, void* sino, int ch, hipStream_t s) {
    return launch_project_with<T>(p, img, sino, ch, p->scratch_O, p->scratch_OT, s);
}

template <typename T>
hipError_t launch_project_pair(int sym, int waves, const OrbitArgs<T>* odev,
                               const OrbitArgs<T>& oone, const ProjArgs<T>* pdev,
                               const ProjArgs<T>& pone, int n, long pixels, hipStream_t s,
                               bool orbit) {
    return sym == 4
               ? project_pair_w<T, 4>(waves, odev, oone, pdev, pone, n, pixels, s, orbit)
               : project_pair_w<T, 1>(waves, odev, oone, pdev, pone, n, pixels, s, orbit);
}

template <typename T>
hipError_t launch_rhs_orbit(const BpArgs<T>* dev, const BpArgs<T>& one, const OrbitArgs<T>* odev,
                            const OrbitArgs<T>& oone, int nsl, hipStream_t s) {
    if (!rhs_orbit_fits(4, one.nx, one.ny) || oone.nx != one.nx || oone.ny != one.ny ||
        (dev == nullptr) != (odev == nullptr) || nsl < 1 || (dev == nullptr && nsl != 1))
        return hipErrorInvalidValue;
    const unsigned h = (unsigned)one.nx / 16;
    const dim3 g(h * h, 1, (unsigned)nsl);
    if (dev)
        hipLaunchKernelGGL((k_rhs_orbit<T, true>), g, dim3(256), 0, s, dev, one, odev, oone);
    else
        hipLaunchKernelGGL((k_rhs_orbit<T, false>), g, dim3(256), 0, s, nullptr, one, nullptr,
                           oone);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_backproject(const dect_plan* p, int ch, const BpArgs<T>& a0, hipStream_t s) {
    BpArgs<T> a = a0;
    fill_bp_plan<T>(p, a);
    ProfScope ps(bp_name(EPI_NONE), s);
    if (p->sym == 4) {
        T* quad = static_cast<T*>(p->scratch_sq);
        switch (ch) {
            case 1: return bp_plain_w<T, 1, 4>(p->bp_waves, a, quad, s);
            case 2: return bp_plain_w<T, 2, 4>(p->bp_waves, a, quad, s);
            case 4: return bp_plain_w<T, 4, 4>(p->bp_waves, a, quad, s);
        }
    } else {
        switch (ch) {
            case 1: return bp_plain_w<T, 1, 1>(p->bp_waves, a, nullptr, s);
            case 2: return bp_plain_w<T, 2, 1>(p->bp_waves, a, nullptr, s);
            case 4: return bp_plain_w<T, 4, 1>(p->bp_waves, a, nullptr, s);
        }
    }
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_backproject_admm(int sym, int waves, int epi, const BpArgs<T>* dev,
                                   const BpArgs<T>& one, int n, int gx, int gy, hipStream_t s,
                                   bool sums64) {
    ProfScope ps(bp_name(epi), s);
    if (sums64)  // an FP64 plan sums in double anyway
        return sym == 4 ? bp_admm<T, 4, double>(waves, epi, dev, one, n, gx, gy, s)
                        : bp_admm<T, 1, double>(waves, epi, dev, one, n, gx, gy, s);
    return sym == 4 ? bp_admm<T, 4, T>(waves, epi, dev, one, n, gx, gy, s)
                    : bp_admm<T, 1, T>(waves, epi, dev, one, n, gx, gy, s);
}

#define DECT_INST(T)                                                                          \
    template void fill_bp_plan<T>(const dect_plan*, BpArgs<T>&);                              \
    template hipError_t launch_project<T>(const dect_plan*, const void*, void*, int, hipStream_t); \
    template hipError_t launch_project_pair<T>(int, int, const OrbitArgs<T>*, const OrbitArgs<T>&, \
                                               const ProjArgs<T>*, const ProjArgs<T>&, int, long, \
                                               hipStream_t, bool);                                \
    template hipError_t launch_rhs_orbit<T>(const BpArgs<T>*, const BpArgs<T>&,                  \
                                            const OrbitArgs<T>*, const OrbitArgs<T>&, int,       \
                                            hipStream_t);                                        \
    template hipError_t launch_backproject<T>(const dect_plan*, int, const BpArgs<T>&, hipStream_t); \
    template hipError_t launch_backproject_admm<T>(int, int, int, const BpArgs<T>*,              \
                                                   const BpArgs<T>&, int, int, int, hipStream_t, \
                                                   bool);
DECT_INST(float)
DECT_INST(double)
#undef DECT_INST

}  // namespace dect

// ------------------------------------------------------------------------------
// R without any allocation: the orbit images live in a static device array.
//
// `scratch` is a file-scope device array of kNoAllocScratchBytes.  Each device the
// library runs on holds its own copy until the process ends.  In host code its
// name is only a stand-in for the device symbol, so the device address of each
// device's copy is looked up once (hipGetSymbolAddress, with that device current)
// and kept; kernels receive that address, never the name.
namespace dect {
namespace {

constexpr size_t kNoAllocScratchBytes = size_t(32) << 20;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// The device address of `device`'s copy of scratch (looked up on first use).
dect_status scratch_address(int device, void** out) {
    if (device < 0 || device >= kMaxDevices)
        return fail(DECT_E_DEVICE, "device %d is beyond the %d the library tracks", device,
                    kMaxDevices);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        int cur = -1;
        DECT_HIP(hipGetDevice(&cur));
        if (cur != device) DECT_HIP(hipSetDevice(device));
        void* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (cur != device) (void)hipSetDevice(cur);
        if (e != hipSuccess || !ptr)
            return fail(DECT_E_DEVICE, "no address for the static scratch on device %d: %s",
                        device, hipGetErrorString(e));
        g_scratch_ptr[device] = ptr;
    }
    *out = g_scratch_ptr[device];
    return DECT_OK;
}

}  // namespace
}  // namespace dect

extern "C" dect_status dect_project_noalloc(const dect_plan* p, const void* img, void* sino,
                                            int ch, void* stream) {
    using namespace dect;
    if (!p || !img || !sino) return fail(DECT_E_ARG, "null argument");
    if (ch != 1 && ch != 2 && ch != 4) return fail(DECT_E_ARG, "ch must be 1, 2 or 4 (got %d)", ch);
    // The orbit image and its transpose, the second at the next 256-byte boundary.
    const size_t image = (size_t)p->N * (size_t)ch * (size_t)p->sym * p->elem;
    const size_t second = (image + 255) / 256 * 256;
    if (second + image > kNoAllocScratchBytes)
        return fail(DECT_E_CAPACITY,
                    "the two orbit images need %zu bytes; the static scratch holds %zu "
                    "(%dx%d, %d channels, symmetry %d, %zu-byte values)",
                    second + image, kNoAllocScratchBytes, p->nx, p->ny, ch, p->sym, p->elem);
    void* base = nullptr;
    const dect_status st = scratch_address(p->device, &base);
    if (st != DECT_OK) return st;
    // Both orbit images are written in full before the projector reads them, so the
    // previous call's contents need no clearing.
    void* O = base;
    void* OT = static_cast<char*>(base) + second;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const hipError_t e = p->dtype == DECT_F32
                             ? launch_project_with<float>(p, img, sino, ch, O, OT, s)
                             : launch_project_with<double>(p, img, sino, ch, O, OT, s);
    if (e != hipSuccess) return fail(DECT_E_DEVICE, "launch failed: %s", hipGetErrorString(e));
    return DECT_OK;
}
