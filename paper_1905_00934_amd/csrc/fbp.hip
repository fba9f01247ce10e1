// The projection-wise baseline and initial image (Sec. 2, CDM; Sec. 4, set-up):
// constrained per-ray decomposition, filtered backprojection of the line integrals,
// and the ADMM start from an image.
//
// FBP (textbook parallel and equispaced-fan formulas): each view's row, weighted by
// D / sqrt(D^2 + u^2) for a fan (u on the detector scaled to the isocentre), is
// convolved with the discrete Ram-Lak kernel by an FFT of the zero-padded row (two
// channels as one complex row; the kernel is real and even); then every pixel
// gathers, over the views, the filtered row linearly interpolated at its detector
// coordinate, weighted by U^-2 = (D / L)^2 for a fan (L the distance from the
// source to the pixel along the central ray), and the sum is scaled by span / V.
#include "common.h"
#include "fftcore.h"
#include "kernels.h"
#include "profile.h"

namespace dect {
namespace {

// A filtered row as the gather reads it: per bin interval k = floor(bin), its left value and
// the step to its right one, for k = -2 ... D with zeros off the detector (record k + 2), so
// that any bin clamped to [-2, D] reads what it should without a test.
template <typename T, int CH>
struct IntervalOf {  // (q[k], q[k + 1] - q[k]), CH values each
    typedef T type __attribute__((ext_vector_type(2 * CH)));
};
template <typename T, int CH>
using Interval = typename IntervalOf<T, CH>::type;

// The row's FFT, filter and inverse in registers and LDS (fftcore.h).  13-15 us for 720 rows of
// 2048 points, FP32 (33 us with radix-2 passes on reordered rows); the chain of seven passes and
// their barriers bounds it, with 2.8 blocks per compute unit.
// One view per block, two channels as one complex row.
template <typename T, int CH>
__global__ __launch_bounds__(256) void k_fbp_filter(const T* __restrict__ sino, int D, int lg,
                                                    const T* __restrict__ H,
                                                    const T* __restrict__ tw,
                                                    const T* __restrict__ wpre, T* __restrict__ Q) {
    extern __shared__ char smem[];
    cx<T>* buf = reinterpret_cast<cx<T>*>(smem);
    const int v = blockIdx.x;
    const T* row = sino + (size_t)v * D * CH;
    const LdsSeq<T> l{buf, fft_buf(lg)};
    fft_convolve<false, T>(
        buf, 1, lg, tw,
        [&](int, int i) {
            cx<T> x{T(0), T(0)};
            if (i < D) {
                const T w = wpre[i];
                x.re = row[(size_t)i * CH] * w;
                if constexpr (CH == 2) x.im = row[2 * (size_t)i + 1] * w;
            }
            return x;
        },
        [&](int, int p) { return H[p]; }, l);
    __syncthreads();
    Interval<T, CH>* q = reinterpret_cast<Interval<T, CH>*>(Q) + (size_t)v * (D + 3);
    for (int r = threadIdx.x; r < D + 3; r += blockDim.x) {
        const int k = r - 2;
        cx<T> a{T(0), T(0)}, b{T(0), T(0)};
        if (k >= 0 && k < D) a = l(0, k);
        if (k >= -1 && k < D - 1) b = l(0, k + 1);
        if constexpr (CH == 2)
            q[r] = Interval<T, CH>{a.re, a.im, b.re - a.re, b.im - a.im};
        else
            q[r] = Interval<T, CH>{a.re, b.re - a.re};
    }
}

template <typename T>
__device__ inline T recip(T d) {
    if constexpr (sizeof(T) == 4)
        return __builtin_amdgcn_rcpf(d);  // 1 ulp; the bin position is good to ~1e-4 bins
    else
        return T(1) / d;
}

constexpr int kFbpWin = 64;         // staged intervals of a window, one per lane
constexpr float kFbpNear = 0.015625f;  // least U, and largest |bin|, of a staged window: the
constexpr float kFbpFar = 16384.0f;    // bins of its pixels are then good to half a bin

// The gather of FBP, on a tile of 8 x 8 PX pixels per workgroup (per orbit domain on a
// quarter-turn symmetric plan) whose VS waves take equal shares of the views and add up at
// the end.  For a view a wave stages in LDS the intervals its tile can reach, between the
// extremes of the tile's corners (a projective bin is monotone along lines while U > 0), one
// per lane; a view that needs more, or whose corners come too near the source, is read from
// memory.  SYM = 4: base view v sees pixel rot_a(p) at the same bin and weight as view v + k
// Vb sees rot_(a+k)(p), so each bin and weight serves four views (k) and goes into four
// pixels' sums; views an even and an odd number of turns on each take the bin and weight that
// they would round to by themselves (two forms of one sum: bins differ by 1e-4 between them,
// which is what single precision can tell).  The next window's loads are in flight while one is
// used.
//
// Per pixel and view: 11 vector instructions on a symmetric plan (37 where every pixel read
// its two taps from memory behind four comparisons, one thread per pixel walking all views)
// and an LDS read of 16 bytes (FP32, two channels).  FBP with its filter, FP32, two channels:
// 512^2 / 720 x 1024 fan 104 us (229 before), 366^2 / 540 x 545 parallel 62 us (149), 1024^2 /
// 1440 x 2048 569 us (1435); instruction issue and LDS reads, about equally, bound it.
template <typename T, int CH, int SYM, bool FAN, int VS, int PX>
__global__ __launch_bounds__(64 * VS) void k_fbp_back(const T* __restrict__ Q, int nx, int ny,
                                                      int Vb, int D, T b0,
                                                      const T* __restrict__ view, T dtheta,
                                                      T* __restrict__ img) {
    using R = Interval<T, CH>;
    constexpr int NV = 64 / SYM;  // views per table of windows
    constexpr int ODD = SYM == 4 ? 2 : 1;
    constexpr int kOut = 64 * PX * SYM * CH;
    constexpr int kShared = VS * SYM * kFbpWin * 2 * CH > VS * kOut ? VS * SYM * kFbpWin * 2 * CH
                                                                    : VS * kOut;
    __shared__ __align__(32) T s_mem[kShared];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    R* win = reinterpret_cast<R*>(s_mem) + wave * SYM * kFbpWin;
    const R* rec = reinterpret_cast<const R*>(Q);
    const int dx = SYM == 4 ? nx / 2 : nx, dy = SYM == 4 ? ny / 2 : ny;
    const int i0 = blockIdx.x * 8, j0 = blockIdx.y * 8 * PX;
    const T hx = T(0.5) * (T)(nx - 1), hy = T(0.5) * (T)(ny - 1);
    // Centred pixel coordinates; lanes past the domain repeat its last pixels.
    const T ic = (T)min(i0 + (lane & 7), dx - 1) - hx;
    T jc[PX];
#pragma unroll
    for (int p = 0; p < PX; ++p) jc[p] = (T)min(j0 + 8 * p + (lane >> 3), dy - 1) - hy;
    const T ilo = (T)i0 - hx, ihi = (T)min(i0 + 7, dx - 1) - hx;
    const T jlo = (T)j0 - hy, jhi = (T)min(j0 + 8 * PX - 1, dy - 1) - hy;
    const int v0 = (int)((long)Vb * wave / VS), v1 = (int)((long)Vb * (wave + 1) / VS);
    T acc[PX][SYM][CH] = {};
    // odd: the order in which a view an odd number of quarter turns on rounds the same sums.
    auto bin = [&](const T* e, T i, T j, T& r, bool odd) __attribute__((always_inline)) {
        r = T(1);
        if constexpr (FAN)
            r = recip<T>(odd ? fma(e[0], i, fma(e[1], j, T(1))) : fma(e[1], j, fma(e[0], i, T(1))));
        return fma(odd ? fma(e[2], i, e[3] * j) : fma(e[3], j, e[2] * i), r, b0);
    };
    auto turned = [](int a, T i, T j, T& ti, T& tj) {  // rot_a of a centred pixel
        ti = a == 0 ? i : a == 1 ? -j : a == 2 ? -i : j;
        tj = a == 0 ? j : a == 1 ? i : a == 2 ? -j : -i;
    };
#pragma unroll 1
    for (int vc = v0; vc < v1; vc += NV) {
        const int nv = min(NV, v1 - vc);
        // Lane: the window of view vc + lane / SYM, rotation lane % SYM.
        int first = 0, count = 0;
        {
            const T* e = view + 4 * (vc + min(lane / SYM, nv - 1));
            const int a = lane % SYM;
            T lo = T(0), hi = T(0), umin = T(1);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                T ti, tj, r;
                turned(a, c & 1 ? ihi : ilo, c & 2 ? jhi : jlo, ti, tj);
                const T b = bin(e, ti, tj, r, false);
                const T u = fma(e[1], tj, fma(e[0], ti, T(1)));
                lo = c == 0 || b < lo ? b : lo;
                hi = c == 0 || b > hi ? b : hi;
                umin = c == 0 || u < umin ? u : umin;
            }
            const bool ok = umin >= (T)kFbpNear && lo >= -(T)kFbpFar && hi <= (T)kFbpFar;
            if (ok) {
                first = (int)floor(lo) - 1;
                count = (int)floor(hi) + 2 - first;
                if (count > kFbpWin) count = 0;  // 0: read from memory
            }
        }
        R nxt[SYM];
        auto fetch = [&](int n) __attribute__((always_inline)) {  // window n of the table
            const int f = __builtin_amdgcn_readlane(first, n);
            const int m = __builtin_amdgcn_readlane(count, n);
            const int k = min(max(f + min(lane, m), -2), D) + 2;  // lanes past it: one address
            const R* q = rec + (size_t)(vc + n / SYM) * (D + 3);
#pragma unroll
            for (int t = 0; t < SYM; ++t) nxt[t] = (q + (size_t)t * Vb * (D + 3))[k];
        };
        fetch(0);
#pragma unroll 1
        for (int u = 0; u < nv; ++u) {
            T e[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) e[c] = view[4 * (vc + u) + c];
            auto rotation = [&](auto turn) __attribute__((always_inline)) {
                constexpr int a = decltype(turn)::value;
                const int n = u * SYM + a;
                const int f = __builtin_amdgcn_readlane(first, n);
                const int m = __builtin_amdgcn_readlane(count, n);
                __builtin_amdgcn_wave_barrier();
                if (lane < m) {
#pragma unroll
                    for (int t = 0; t < SYM; ++t) win[t * kFbpWin + lane] = nxt[t];
                }
                __builtin_amdgcn_wave_barrier();
                fetch(min(n + 1, nv * SYM - 1));
#pragma unroll
                for (int p = 0; p < PX; ++p) {
                    T ti, tj, al[ODD], w[ODD];
                    int at[ODD];
                    turned(a, ic, jc[p], ti, tj);
#pragma unroll
                    for (int odd = 0; odd < ODD; ++odd) {
                        T r;
                        const T b = bin(e, ti, tj, r, odd != 0), fb = floor(b);
                        al[odd] = b - fb;
                        w[odd] = r * r;
                        at[odd] = (int)fb - f;
                    }
                    if (m == 0) {  // from memory, through the lane's own slots
                        const R* g = rec + (size_t)(vc + u) * (D + 3);
#pragma unroll
                        for (int t = 0; t < SYM; ++t) {
                            const int k = min(max(at[t % ODD] + f, -2), D) + 2;
                            win[t * kFbpWin + lane] = (g + (size_t)t * Vb * (D + 3))[k];
                        }
#pragma unroll
                        for (int odd = 0; odd < ODD; ++odd) at[odd] = lane;
                    }
#pragma unroll
                    for (int t = 0; t < SYM; ++t) {
                        const R q = win[t * kFbpWin + at[t % ODD]];
#pragma unroll
                        for (int c = 0; c < CH; ++c) {
                            T& s = acc[p][(a + t) % SYM][c];
                            const T x = fma(al[t % ODD], q[CH + c], q[c]);
                            s = FAN ? fma(w[t % ODD], x, s) : s + x;
                        }
                    }
                    // Keeps the sums here: moved past the next windows they would hold every
                    // interval read in registers.
#pragma unroll
                    for (int t = 0; t < SYM; ++t)
#pragma unroll
                        for (int c = 0; c < CH; ++c) asm volatile("" : "+v"(acc[p][t][c]));
                }
            };
            rotation(std::integral_constant<int, 0>{});
            if constexpr (SYM == 4) {
                rotation(std::integral_constant<int, 1>{});
                rotation(std::integral_constant<int, 2>{});
                rotation(std::integral_constant<int, 3>{});
            }
        }
    }
    // The waves' sums, added in order.
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PX; ++p)
#pragma unroll
        for (int t = 0; t < SYM; ++t)
#pragma unroll
            for (int c = 0; c < CH; ++c)
                s_mem[wave * kOut + ((p * SYM + t) * CH + c) * 64 + lane] = acc[p][t][c];
    __syncthreads();
    for (int o = threadIdx.x; o < kOut; o += 64 * VS) {
        T s = s_mem[o];
        for (int w = 1; w < VS; ++w) s += s_mem[w * kOut + o];
        const int l = o & 63, c = (o >> 6) % CH, t = (o >> 6) / CH % SYM, p = (o >> 6) / (CH * SYM);
        const int i = i0 + (l & 7), j = j0 + 8 * p + (l >> 3);
        if (i >= dx || j >= dy) continue;
        const int x = t == 0 ? i : t == 1 ? nx - 1 - j : t == 2 ? nx - 1 - i : j;
        const int y = t == 0 ? j : t == 1 ? i : t == 2 ? ny - 1 - j : ny - 1 - i;
        img[((size_t)y * nx + x) * CH + c] = s * dtheta;
    }
}

// Sums of a_c and a_p over all rays in a fixed order: kRaySumBlocks block partials
// (grid-strided), then one block adds them into the slot after the partials.
template <typename T>
__global__ __launch_bounds__(256) void k_ray_sums(const T* __restrict__ a, long M,
                                                  double* __restrict__ part) {
    double v[2] = {0.0, 0.0};
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < M;
         i += (long)gridDim.x * blockDim.x) {
        v[0] += (double)a[2 * i];
        v[1] += (double)a[2 * i + 1];
    }
    block_sum_store<2>(v, part + (size_t)blockIdx.x * kPartialSlots);
}

__global__ __launch_bounds__(256) void k_ray_sums_total(double* __restrict__ part, int nb) {
    double v[2] = {0.0, 0.0};
    if ((int)threadIdx.x < nb) {
        v[0] = part[(size_t)threadIdx.x * kPartialSlots];
        v[1] = part[(size_t)threadIdx.x * kPartialSlots + 1];
    }
    block_sum_store<2>(v, part + (size_t)nb * kPartialSlots);
}

// x0 = (x_c, s x_c) with s = sum a_p / sum a_c.
template <typename T>
__global__ __launch_bounds__(256) void k_start_image(const T* __restrict__ fbp, long N,
                                                     const double* __restrict__ sums,
                                                     T* __restrict__ x0) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const T sc = (T)(sums[0] != 0.0 ? sums[1] / sums[0] : 0.0);
    const T xc = fbp[2 * i];
    x0[2 * i] = xc;
    x0[2 * i + 1] = sc * xc;
}

// x = z = x0 and y = D x0 (forward differences, zero at the last column and row).
template <typename T>
__global__ __launch_bounds__(256) void k_init_image(const T* __restrict__ x0, int nx, int ny,
                                                    T* __restrict__ x, T* __restrict__ z,
                                                    T* __restrict__ y) {
    const long pix = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (pix >= (long)nx * ny) return;
    int i, j;
    pixel_ij(pix, nx, i, j);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const T v = x0[2 * pix + c];
        x[2 * pix + c] = v;
        z[2 * pix + c] = v;
        y[4 * pix + c] = i < nx - 1 ? x0[2 * (pix + 1) + c] - v : T(0);
        y[4 * pix + 2 + c] = j < ny - 1 ? x0[2 * (pix + nx) + c] - v : T(0);
    }
}

// The next right-hand side t = a + u^a - R x with u^a = 0 (internal ray order l).
template <typename T>
__global__ __launch_bounds__(256) void k_init_t(const T* __restrict__ a, const T* __restrict__ Rx,
                                                long M, int sym, int Vb, int D, T* __restrict__ t) {
    const long l = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= M) return;
    const long i = std_ray(l, sym, Vb, D);
    t[2 * l] = a[2 * i] - Rx[2 * i];
    t[2 * l + 1] = a[2 * i + 1] - Rx[2 * i + 1];
}

template <typename T, int CH, int SYM, bool FAN, int VS, int PX>
void fbp_back_as(const dect_plan* p, dim3 g, T dtheta, T* img, hipStream_t s) {
    hipLaunchKernelGGL((k_fbp_back<T, CH, SYM, FAN, VS, PX>), g, dim3(64 * VS), 0, s,
                       static_cast<const T*>(p->scratch_Q), p->nx, p->ny, p->Vb, p->D,
                       (T)p->fbp_b0, static_cast<const T*>(p->fbp_view), dtheta, img);
}

template <typename T, int CH, int SYM, bool FAN>
void fbp_back(const dect_plan* p, T dtheta, T* img, hipStream_t s) {
    const unsigned dx = SYM == 4 ? p->nx / 2 : p->nx, dy = SYM == 4 ? p->ny / 2 : p->ny;
    // Tall tiles stage a window for 256 pixels instead of 128 but leave half the workgroups:
    // from two per compute unit on (one form of the sums, FP32: 366^2 parallel 62 us against 67,
    // 1024^2 fan 504 against 551, but 512^2 fan, 256 tall tiles, 115 against 95).  Below two
    // small ones per unit 16 waves share the views (256^2: 31 us against 34; 512^2 with 512
    // tiles: 101 against 95).
    const unsigned gx = (dx + 7) / 8, g2 = (dy + 15) / 16, g4 = (dy + 31) / 32;
    if (gx * g4 >= 512)
        fbp_back_as<T, CH, SYM, FAN, 8, 4>(p, dim3(gx, g4), dtheta, img, s);
    else if (gx * g2 >= 512)
        fbp_back_as<T, CH, SYM, FAN, 8, 2>(p, dim3(gx, g2), dtheta, img, s);
    else
        fbp_back_as<T, CH, SYM, FAN, 16, 2>(p, dim3(gx, g2), dtheta, img, s);
}

template <typename T, int CH>
hipError_t fbp_ch(const dect_plan* p, const T* sino, T* img, hipStream_t s) {
    const size_t lds = (size_t)fft_buf(p->fbp_lg) * sizeof(cx<T>);
    hipLaunchKernelGGL((k_fbp_filter<T, CH>), dim3((unsigned)p->V), dim3(256), lds, s,
                       sino, p->D, p->fbp_lg,
                       static_cast<const T*>(p->fbp_H), static_cast<const T*>(p->fbp_tw),
                       static_cast<const T*>(p->fbp_wpre), static_cast<T*>(p->scratch_Q));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const T dtheta = (T)(p->geom.span / p->V);
    if (p->sym == 4)  // quarter-turn symmetric plans are fans
        p->geom.kind == DECT_FAN ? fbp_back<T, CH, 4, true>(p, dtheta, img, s)
                                 : fbp_back<T, CH, 4, false>(p, dtheta, img, s);
    else
        p->geom.kind == DECT_FAN ? fbp_back<T, CH, 1, true>(p, dtheta, img, s)
                                 : fbp_back<T, CH, 1, false>(p, dtheta, img, s);
    return hipGetLastError();
}

template <typename T>
hipError_t fbp_t(const dect_plan* p, const void* sino, void* img, int ch, hipStream_t s) {
    ProfScope ps("fbp", s);
    const T* in = static_cast<const T*>(sino);
    return ch == 2 ? fbp_ch<T, 2>(p, in, static_cast<T*>(img), s)
                   : fbp_ch<T, 1>(p, in, static_cast<T*>(img), s);
}

template <typename T>
hipError_t cdm_t(const dect_plan* p, const void* mh, const void* ml, const void* wh,
                 const void* wl, int iters, void* a, void* cost, hipStream_t s) {
    UdmArgs<T> u{};
    u.M = p->M;
    u.sym = 1;
    u.Vb = p->V;
    u.D = p->D;
    u.mh = static_cast<const T*>(mh);
    u.ml = static_cast<const T*>(ml);
    u.wh = static_cast<const T*>(wh);
    u.wl = static_cast<const T*>(wl);
    u.a = static_cast<T*>(a);
    u.cost = static_cast<T*>(cost);
    u.iters = iters;
    u.mu0 = 1e-3;
    // Inverse of the linearisation at a = 0: rows (mean f_KN, mean f_p) per spectrum.
    const double hc = p->mean_f[0][0], hp = p->mean_f[0][1];
    const double lc = p->mean_f[1][0], lp = p->mean_f[1][1];
    const double det = hc * lp - hp * lc;
    u.lin[0] = lp / det;
    u.lin[1] = -hp / det;
    u.lin[2] = -lc / det;
    u.lin[3] = hc / det;
    return launch_udm<T>(p, 3, u, s);
}

template <typename T>
hipError_t start_t(const dect_plan* p, const void* a, void* fbp, void* x0, hipStream_t s) {
    static_assert(kRaySumBlocks <= 256, "one block adds the partials");
    hipLaunchKernelGGL((k_ray_sums<T>), dim3(kRaySumBlocks), dim3(256), 0, s,
                       static_cast<const T*>(a), p->M, p->scratch_part);
    hipLaunchKernelGGL(k_ray_sums_total, dim3(1), dim3(256), 0, s, p->scratch_part,
                       kRaySumBlocks);
    hipLaunchKernelGGL((k_start_image<T>), dim3((unsigned)((p->N + 255) / 256)), dim3(256), 0, s,
                       static_cast<const T*>(fbp), p->N,
                       p->scratch_part + (size_t)kRaySumBlocks * kPartialSlots,
                       static_cast<T*>(x0));
    return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_init_image(const dect_plan* p, const void* x0, void* state, hipStream_t s,
                             bool sums64) {
    const dect_layout& L = p->layout;
    char* st = static_cast<char*>(state);
    T* Rx = reinterpret_cast<T*>(st + L.Rx);
    hipLaunchKernelGGL((k_init_image<T>), dim3((unsigned)((p->N + 255) / 256)), dim3(256), 0, s,
                       static_cast<const T*>(x0), p->nx, p->ny, reinterpret_cast<T*>(st + L.x),
                       reinterpret_cast<T*>(st + L.z), reinterpret_cast<T*>(st + L.y));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // R x0 into the state's R x (standard [V][D][2] order), then t = a - R x0.
    e = launch_project<T>(p, x0, Rx, 2, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_init_t<T>), dim3((unsigned)((p->M + 255) / 256)), dim3(256), 0, s,
                       reinterpret_cast<const T*>(st + L.a), Rx, p->M, p->sym, p->Vb, p->D,
                       reinterpret_cast<T*>(st + p->off_t));
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_track_init<T>(p, state, s, sums64);
}

template hipError_t launch_init_image<float>(const dect_plan*, const void*, void*, hipStream_t,
                                             bool);
template hipError_t launch_init_image<double>(const dect_plan*, const void*, void*, hipStream_t,
                                              bool);

}  // namespace dect

using namespace dect;

extern "C" {

dect_status dect_cdm(const dect_plan* p, const void* m_h, const void* m_l, const void* w_h,
                     const void* w_l, int lm_iters, void* a, void* cost, void* stream) {
    if (!p || !m_h || !m_l || !w_h || !w_l || !a) return fail(DECT_E_ARG, "null argument");
    if (lm_iters < 0) return fail(DECT_E_ARG, "lm_iters must be >= 0");
    hipStream_t s = static_cast<hipStream_t>(stream);
    const hipError_t e = p->dtype == DECT_F32
                             ? cdm_t<float>(p, m_h, m_l, w_h, w_l, lm_iters, a, cost, s)
                             : cdm_t<double>(p, m_h, m_l, w_h, w_l, lm_iters, a, cost, s);
    if (e != hipSuccess) return fail(DECT_E_DEVICE, "launch failed: %s", hipGetErrorString(e));
    return DECT_OK;
}

dect_status dect_fbp(const dect_plan* p, const void* sino, void* img, int ch, void* stream) {
    if (!p || !sino || !img) return fail(DECT_E_ARG, "null argument");
    if (ch != 1 && ch != 2) return fail(DECT_E_ARG, "ch must be 1 or 2 (got %d)", ch);
    if (!p->has_fbp)
        return fail(DECT_E_SHAPE, "no FBP filter for %d bins (padded row > %d)", p->D, kMaxFbp);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const hipError_t e = p->dtype == DECT_F32 ? fbp_t<float>(p, sino, img, ch, s)
                                              : fbp_t<double>(p, sino, img, ch, s);
    if (e != hipSuccess) return fail(DECT_E_DEVICE, "launch failed: %s", hipGetErrorString(e));
    return DECT_OK;
}

dect_status dect_cdm_fbp_start(const dect_plan* p, const void* m_h, const void* m_l,
                               const void* w_h, const void* w_l, int cdm_iters, void* a,
                               void* x0, void* fbp_out, void* stream) {
    if (!p || !m_h || !m_l || !w_h || !w_l || !a || !x0) return fail(DECT_E_ARG, "null argument");
    if (cdm_iters < 0) return fail(DECT_E_ARG, "cdm_iters must be >= 0");
    if (!p->has_fbp)
        return fail(DECT_E_SHAPE, "no FBP filter for %d bins (padded row > %d)", p->D, kMaxFbp);
    hipStream_t s = static_cast<hipStream_t>(stream);
    void* f = fbp_out ? fbp_out : x0;
    hipError_t e;
    if (p->dtype == DECT_F32) {
        e = cdm_t<float>(p, m_h, m_l, w_h, w_l, cdm_iters, a, nullptr, s);
        if (e == hipSuccess) e = fbp_t<float>(p, a, f, 2, s);
        if (e == hipSuccess) e = start_t<float>(p, a, f, x0, s);
    } else {
        e = cdm_t<double>(p, m_h, m_l, w_h, w_l, cdm_iters, a, nullptr, s);
        if (e == hipSuccess) e = fbp_t<double>(p, a, f, 2, s);
        if (e == hipSuccess) e = start_t<double>(p, a, f, x0, s);
    }
    if (e != hipSuccess) return fail(DECT_E_DEVICE, "launch failed: %s", hipGetErrorString(e));
    return DECT_OK;
}

}  // extern "C"
