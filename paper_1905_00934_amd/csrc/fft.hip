// The preconditioner of the x-update (Sec. 3.3): z = M r with M the ramp filter
// applied by a 2-D FFT on the zero-padded image.
//
// The two bases of an image pair are the real and imaginary parts of one complex
// image (the [ny][nx][2] layout is already complex), and the filter is real and
// even in frequency, so one complex transform filters both: its real part stays
// the filtered c image and its imaginary part the filtered p image.
//
// Three passes over a [ny][px] complex work grid (rows beyond ny of the padded
// grid are zero and never stored):
//   rows:    forward DFT of every image row, zero-padded to px, frequencies bit-reversed;
//   columns: forward DFT of every column (zero-padded to py), multiply by the
//            filter, inverse DFT, keep the first ny entries;
//   rows:    inverse DFT, keep the first nx entries, scale by 1/(px py); the
//            block partial sums of r . z per basis go to `partials`.
#include "common.h"
#include "fftcore.h"
#include "kernels.h"
#include "profile.h"

namespace dect {
namespace {

template <typename T, bool BATCH>
__global__ __launch_bounds__(256) void k_pre_rows_fwd(const PrecArgs<T>* __restrict__ dev,
                                                      PrecArgs<T> one) {
    extern __shared__ char smem[];
    cx<T>* buf = reinterpret_cast<cx<T>*>(smem);
    const PrecArgs<T> A = pick_args<BATCH>(dev, one);
    const int j = blockIdx.x;
    if (j >= A.ny) return;  // beyond this slice (whole block)
    const cx<T>* row = reinterpret_cast<const cx<T>*>(A.r) + (size_t)j * A.nx;
    cx<T>* w = reinterpret_cast<cx<T>*>(A.W) + (size_t)j * A.px;
    fft_forward<T>(
        buf, 1, A.lpx, A.twx,
        [&](int, int i) { return i < A.nx ? row[i] : cx<T>{T(0), T(0)}; },
        [&](int, int p, cx<T> x) { w[p] = x; });
}

// Column groups per XCD: workgroups reach the kXcds XCDs in turn, and XCD x takes
// the x-th contiguous range of column groups, so the columns that share a cache
// line of the work grid are read through the same L2.
inline unsigned pre_col_blocks(int groups) {
    return (unsigned)(kXcds * ((groups + kXcds - 1) / kXcds));
}

// C columns per block (C consecutive columns of the work grid).
template <typename T, bool BATCH, int C>
__global__ __launch_bounds__(256) void k_pre_cols(const PrecArgs<T>* __restrict__ dev,
                                                  PrecArgs<T> one) {
    extern __shared__ char smem[];
    cx<T>* buf = reinterpret_cast<cx<T>*>(smem);
    const PrecArgs<T> A = pick_args<BATCH>(dev, one);
    const int groups = (A.px + C - 1) / C, per = (groups + kXcds - 1) / kXcds;
    const int g = (int)(blockIdx.x % kXcds) * per + (int)(blockIdx.x / kXcds);
    const int c0 = g * C;
    if (g >= groups) return;  // beyond this slice (whole block)
    const int lg = A.lpy;
    cx<T>* W = reinterpret_cast<cx<T>*>(A.W);
    fft_convolve<true, T>(
        buf, C, lg, A.twy,
        [&](int cc, int j) {
            return j < A.ny && c0 + cc < A.px ? W[(size_t)j * A.px + c0 + cc]
                                              : cx<T>{T(0), T(0)};
        },
        [&](int cc, int p) {
            return c0 + cc < A.px ? A.filter[((size_t)(c0 + cc) << lg) + p] : T(0);
        },
        [&](int cc, int j, cx<T> x) {
            if (j < A.ny && c0 + cc < A.px) W[(size_t)j * A.px + c0 + cc] = x;
        });
}

template <typename T, bool BATCH>
__global__ __launch_bounds__(256) void k_pre_rows_inv(const PrecArgs<T>* __restrict__ dev,
                                                      PrecArgs<T> one) {
    extern __shared__ char smem[];
    cx<T>* buf = reinterpret_cast<cx<T>*>(smem);
    const PrecArgs<T> A = pick_args<BATCH>(dev, one);
    const int j = blockIdx.x;
    if (j >= A.ny) return;  // beyond this slice (whole block)
    const cx<T>* w = reinterpret_cast<const cx<T>*>(A.W) + (size_t)j * A.px;
    const T scale = T(1) / ((T)A.px * (T)A.py);
    const cx<T>* r = reinterpret_cast<const cx<T>*>(A.r) + (size_t)j * A.nx;
    cx<T>* z = reinterpret_cast<cx<T>*>(A.z) + (size_t)j * A.nx;
    double part[2] = {0.0, 0.0};
    fft_inverse<T>(
        buf, 1, A.lpx, A.twx, [&](int, int p) { return w[p]; },
        [&](int, int i, cx<T> x) {
            if (i >= A.nx) return;
            const cx<T> v{x.re * scale, x.im * scale};
            const cx<T> rv = r[i];
            z[i] = v;
            part[0] += (double)rv.re * (double)v.re;
            part[1] += (double)rv.im * (double)v.im;
        });
    block_sum_store<2>(part, A.partials + (size_t)j * kPartialSlots);
}

template <typename T, bool BATCH>
void precond_launch(const PrecArgs<T>* dev, const PrecArgs<T>& one, int n, hipStream_t s) {
    // Two columns per block: the work grid is read in 16-byte runs (FP32) from twice as few
    // blocks; 512^2: 23.9 us for the three kernels against 25.2 with one column and 33.4 with
    // eight, 1024^2: 52.0, 56.9 and 63.4 (41 and 125 us with the former radix-2 passes).
    constexpr int C = 2;
    const size_t row_lds = (size_t)fft_buf(one.lpx) * sizeof(cx<T>);
    const size_t col_lds = (size_t)C * fft_buf(one.lpy) * sizeof(cx<T>);
    const dim3 rows((unsigned)one.ny, 1, n), cols(pre_col_blocks((one.px + C - 1) / C), 1, n);
    hipLaunchKernelGGL((k_pre_rows_fwd<T, BATCH>), rows, dim3(256), row_lds, s, dev, one);
    hipLaunchKernelGGL((k_pre_cols<T, BATCH, C>), cols, dim3(256), col_lds, s, dev, one);
    hipLaunchKernelGGL((k_pre_rows_inv<T, BATCH>), rows, dim3(256), row_lds, s, dev, one);
}

}  // namespace

template <typename T>
void fill_precond_plan(const dect_plan* p, PrecArgs<T>& a) {
    a.nx = p->nx;
    a.ny = p->ny;
    a.px = p->px;
    a.py = p->py;
    a.lpx = p->lpx;
    a.lpy = p->lpy;
    a.filter = static_cast<const T*>(p->pre_filter);
    a.twx = static_cast<const T*>(p->pre_twx);
    a.twy = static_cast<const T*>(p->pre_twy);
}

template <typename T>
hipError_t launch_precond(const PrecArgs<T>* dev, const PrecArgs<T>& one, int n, hipStream_t s) {
    ProfScope ps("precond", s);
    if (dev)
        precond_launch<T, true>(dev, one, n, s);
    else
        precond_launch<T, false>(dev, one, n, s);
    return hipGetLastError();
}

template void fill_precond_plan<float>(const dect_plan*, PrecArgs<float>&);
template void fill_precond_plan<double>(const dect_plan*, PrecArgs<double>&);
template hipError_t launch_precond<float>(const PrecArgs<float>*, const PrecArgs<float>&, int,
                                          hipStream_t);
template hipError_t launch_precond<double>(const PrecArgs<double>*, const PrecArgs<double>&, int,
                                           hipStream_t);

}  // namespace dect

using namespace dect;

extern "C" {

dect_status dect_precondition(const dect_plan* p, const void* img, void* out, void* stream) {
    if (!p || !img || !out) return fail(DECT_E_ARG, "null argument");
    if (!p->has_precond)
        return fail(DECT_E_SHAPE, "no preconditioner for a %dx%d image (padded side > %d)", p->nx,
                    p->ny, kMaxFft);
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e;
    if (p->dtype == DECT_F32) {
        PrecArgs<float> a{};
        fill_precond_plan<float>(p, a);
        a.W = static_cast<float*>(p->scratch_W);
        a.r = static_cast<const float*>(img);
        a.z = static_cast<float*>(out);
        a.partials = p->scratch_part;
        e = launch_precond<float>(nullptr, a, 1, s);
    } else {
        PrecArgs<double> a{};
        fill_precond_plan<double>(p, a);
        a.W = static_cast<double*>(p->scratch_W);
        a.r = static_cast<const double*>(img);
        a.z = static_cast<double*>(out);
        a.partials = p->scratch_part;
        e = launch_precond<double>(nullptr, a, 1, s);
    }
    if (e != hipSuccess) return fail(DECT_E_DEVICE, "launch failed: %s", hipGetErrorString(e));
    return DECT_OK;
}

}  // extern "C"
