// FFTs in LDS shared by the preconditioner and the FBP filter.
//
// A forward transform is decimation in frequency, natural order in and bit-reversed order
// out; an inverse one (no 1/P factor) is decimation in time, bit-reversed in and natural out.
// A convolution multiplies between the two, in bit-reversed order, so nothing is ever
// reordered: filters and work grids hold their frequencies bit-reversed (P a power of two,
// twiddles tw[k] = exp(-2 pi i k / P), k < P/2, as (cos, sin) pairs).
//
// Three radix-2 stages at a time run in registers on groups of eight elements a distance m
// apart, so a transform of 2^lg takes ceil(lg / 3) passes over LDS and as many barriers; the
// first pass reads its elements from the caller's source and the last one hands them to the
// caller's sink, and the last forward and first inverse pass of a convolution are one.
// Elements are padded by one in eight: groups of neighbours (the passes of distance 1 and 8)
// then meet the banks in turn.  The former radix-2 pair passes on bit-reversed input spent
// 80 % of their LDS cycles on bank conflicts.
#pragma once

#include "common.h"

namespace dect {

template <typename T>
struct cx {
    T re, im;
};

// LDS index of element i, and the elements of a buffer of one sequence of 2^lg.
__host__ __device__ inline int fft_at(int i) { return i + (i >> 3); }
__host__ __device__ inline int fft_buf(int lg) { return (1 << lg) + ((1 << lg) >> 3) + 8; }

template <bool INV, typename T>
__device__ inline cx<T> cmul(cx<T> w, cx<T> c) {
    const T wi = INV ? -w.im : w.im;
    return cx<T>{w.re * c.re - wi * c.im, w.re * c.im + wi * c.re};
}

// LR radix-2 stages on the 2^LR elements j + r m of a block of 2^LR m (m = 2^lm): half
// distances 2^(LR-1) m down to m (forward), or up (inverse).  At half distance 2^s m the
// pair at position j + q m (q < 2^s) has the twiddle exp(-i pi (j + q m) / (2^s m)): a table
// entry for q m < quarter of the block, that entry times -i beyond.
template <int LR, bool INV, typename T>
__device__ inline void fft_stages(cx<T> (&x)[1 << LR], int j, int lm, int lg,
                                  const T* __restrict__ tw) {
    const cx<T>* w = reinterpret_cast<const cx<T>*>(tw);
#pragma unroll
    for (int n = 0; n < LR; ++n) {
        const int s = INV ? n : LR - 1 - n, h = 1 << s;
        const int sh = lg - 1 - lm - s;  // table steps per position
        cx<T> t[2];
        t[0] = w[j << sh];
        if (s == 2) t[1] = w[(j + (1 << lm)) << sh];
#pragma unroll
        for (int r = 0; r < 1 << LR; ++r) {
            if (r & h) continue;
            const int q = r & (h - 1);
            // Position q: entry q mod max(h / 2, 1), times -i for q >= h / 2 (h >= 2).
            const bool turn = h >= 2 && q >= h / 2;
            cx<T> e = t[s == 2 ? q & 1 : 0];
            if (turn) e = cx<T>{e.im, -e.re};
            cx<T> a = x[r], b = x[r + h];
            if constexpr (INV) {
                b = cmul<true>(e, b);
                x[r] = cx<T>{a.re + b.re, a.im + b.im};
                x[r + h] = cx<T>{a.re - b.re, a.im - b.im};
            } else {
                x[r] = cx<T>{a.re + b.re, a.im + b.im};
                x[r + h] = cmul<false>(e, cx<T>{a.re - b.re, a.im - b.im});
            }
        }
    }
}

// One pass of LR stages at distance m = 2^lm over `count` sequences: get(c, i) and put(c, i,
// x) read and write element i of sequence c, sequences fastest over the threads when MIX
// (coalesced access to rows that hold the sequences side by side).
template <int LR, bool INV, bool MIX, typename T, typename Get, typename Put>
__device__ inline void fft_pass(int count, int lm, int lg, const T* __restrict__ tw, Get get,
                                Put put) {
    const int groups = 1 << (lg - LR);
    for (int t = threadIdx.x; t < count * groups; t += blockDim.x) {
        const int c = MIX ? t % count : t >> (lg - LR), g = MIX ? t / count : t & (groups - 1);
        const int j = g & ((1 << lm) - 1), i0 = ((g >> lm) << (lm + LR)) + j;
        cx<T> x[1 << LR];
#pragma unroll
        for (int r = 0; r < 1 << LR; ++r) x[r] = get(c, i0 + (r << lm));
        fft_stages<LR, INV>(x, j, lm, lg, tw);
#pragma unroll
        for (int r = 0; r < 1 << LR; ++r) put(c, i0 + (r << lm), x[r]);
    }
}

template <typename T>
struct LdsSeq {
    cx<T>* buf;
    int stride;
    __device__ cx<T> operator()(int c, int i) const { return buf[c * stride + fft_at(i)]; }
    __device__ void operator()(int c, int i, cx<T> x) const { buf[c * stride + fft_at(i)] = x; }
};

// Stages of the pass at distance 1 (the others take three).
__device__ inline int fft_tail(int lg) { return lg % 3 == 0 ? 3 : lg % 3; }

// Forward transforms: get(c, i) natural, put(c, p, x) at bit-reversed positions p.  Every
// thread of the block must call it; buf is free for it on entry.
template <typename T, typename Get, typename Put>
__device__ inline void fft_forward(cx<T>* buf, int count, int lg, const T* __restrict__ tw,
                                   Get get, Put put) {
    const LdsSeq<T> l{buf, fft_buf(lg)};
    const int tail = fft_tail(lg);
    if (lg <= 3) {
        if (tail == 1) fft_pass<1, false, false>(count, 0, lg, tw, get, put);
        else if (tail == 2) fft_pass<2, false, false>(count, 0, lg, tw, get, put);
        else fft_pass<3, false, false>(count, 0, lg, tw, get, put);
        return;
    }
    fft_pass<3, false, false>(count, lg - 3, lg, tw, get, l);
    for (int lm = lg - 6; lm >= tail; lm -= 3) {
        __syncthreads();
        fft_pass<3, false, false>(count, lm, lg, tw, l, l);
    }
    __syncthreads();
    if (tail == 1) fft_pass<1, false, false>(count, 0, lg, tw, l, put);
    else if (tail == 2) fft_pass<2, false, false>(count, 0, lg, tw, l, put);
    else fft_pass<3, false, false>(count, 0, lg, tw, l, put);
}

// Inverse transforms: get(c, p) at bit-reversed positions, put(c, i, x) natural.
template <typename T, typename Get, typename Put>
__device__ inline void fft_inverse(cx<T>* buf, int count, int lg, const T* __restrict__ tw,
                                   Get get, Put put) {
    const LdsSeq<T> l{buf, fft_buf(lg)};
    const int tail = fft_tail(lg);
    if (lg <= 3) {
        if (tail == 1) fft_pass<1, true, false>(count, 0, lg, tw, get, put);
        else if (tail == 2) fft_pass<2, true, false>(count, 0, lg, tw, get, put);
        else fft_pass<3, true, false>(count, 0, lg, tw, get, put);
        return;
    }
    if (tail == 1) fft_pass<1, true, false>(count, 0, lg, tw, get, l);
    else if (tail == 2) fft_pass<2, true, false>(count, 0, lg, tw, get, l);
    else fft_pass<3, true, false>(count, 0, lg, tw, get, l);
    for (int lm = tail; lm < lg - 3; lm += 3) {
        __syncthreads();
        fft_pass<3, true, false>(count, lm, lg, tw, l, l);
    }
    __syncthreads();
    fft_pass<3, true, false>(count, lg - 3, lg, tw, l, put);
}

// The pass between a forward and an inverse transform: LR stages at distance 1, the product
// with mul(c, p) (real), and the same stages back.
template <int LR, typename T, typename Get, typename Mul, typename Put>
__device__ inline void fft_turn(int count, int lg, const T* __restrict__ tw, Get get, Mul mul,
                                Put put) {
    const int groups = 1 << (lg - LR);
    for (int t = threadIdx.x; t < count * groups; t += blockDim.x) {
        const int c = t >> (lg - LR), i0 = (t & (groups - 1)) << LR;
        cx<T> x[1 << LR];
#pragma unroll
        for (int r = 0; r < 1 << LR; ++r) x[r] = get(c, i0 + r);
        fft_stages<LR, false>(x, 0, 0, lg, tw);
#pragma unroll
        for (int r = 0; r < 1 << LR; ++r) {
            const T f = mul(c, i0 + r);
            x[r].re *= f;
            x[r].im *= f;
        }
        fft_stages<LR, true>(x, 0, 0, lg, tw);
#pragma unroll
        for (int r = 0; r < 1 << LR; ++r) put(c, i0 + r, x[r]);
    }
}

// Convolutions: forward, product with mul(c, p) at bit-reversed positions, inverse; get and
// put natural, MIX as in fft_pass for both.
template <bool MIX, typename T, typename Get, typename Mul, typename Put>
__device__ inline void fft_convolve(cx<T>* buf, int count, int lg, const T* __restrict__ tw,
                                    Get get, Mul mul, Put put) {
    const LdsSeq<T> l{buf, fft_buf(lg)};
    const int tail = fft_tail(lg);
    if (lg <= 3) {
        if (tail == 1) fft_turn<1>(count, lg, tw, get, mul, put);
        else if (tail == 2) fft_turn<2>(count, lg, tw, get, mul, put);
        else fft_turn<3>(count, lg, tw, get, mul, put);
        return;
    }
    fft_pass<3, false, MIX>(count, lg - 3, lg, tw, get, l);
    for (int lm = lg - 6; lm >= tail; lm -= 3) {
        __syncthreads();
        fft_pass<3, false, false>(count, lm, lg, tw, l, l);
    }
    __syncthreads();
    if (tail == 1) fft_turn<1>(count, lg, tw, l, mul, l);
    else if (tail == 2) fft_turn<2>(count, lg, tw, l, mul, l);
    else fft_turn<3>(count, lg, tw, l, mul, l);
    for (int lm = tail; lm < lg - 3; lm += 3) {
        __syncthreads();
        fft_pass<3, true, false>(count, lm, lg, tw, l, l);
    }
    __syncthreads();
    fft_pass<3, true, MIX>(count, lg - 3, lg, tw, l, put);
}

}  // namespace dect
