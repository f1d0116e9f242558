// fft.h -- register FFTs of the fluid solves (included by fluid.hip only).
//
// One line of n = 2^LOGN values is held by TPL = n / E threads, E values each:
// register e of thread t is element t + TPL e, before and after a transform.
// A transform is two or three Stockham passes of radix up to 16 in registers,
// with one exchange through LDS between passes (radix 2 through LDS took eight
// exchanges for n = 256 and held the fluid steps to LDS and barrier latency:
// 109 us a pass over 134 MB against about 35 now).  The element order makes
// every global access of a transform the natural one, so the passes before
// and after it (stencils, symbols) work on the registers directly.
#pragma once

#include "ibx_internal.h"

namespace ibx {

template <typename T>
struct alignas(2 * sizeof(T)) Cx {
    T x, y;
};

template <int LOGN>
struct Line {
    static constexpr int n = 1 << LOGN;
    static constexpr int E = LOGN == 4 ? 4 : (LOGN == 7 || LOGN == 8 || LOGN == 10) ? 16 : 8;
    static constexpr int TPL = n / E;
    // radices of the passes (1: no such pass)
    static constexpr int R0 = E;
    static constexpr int R1 = LOGN == 3 ? 1 : LOGN == 4 || LOGN == 5 ? 4 : LOGN == 7 ? 8 : E;
    static constexpr int R2 = LOGN == 9 ? 8 : LOGN == 10 ? 4 : 1;
    static_assert(R0 * R1 * R2 == n, "the radices multiply to n");
    // LDS elements of one line: one pad element after every 16, which spreads
    // the strided writes of an exchange over the banks
    static constexpr int LDS = n + n / 16;
};

__device__ inline int lds_at(int i) { return i + (i >> 4); }

template <typename T, bool INV>
__device__ inline Cx<T> cmul(Cx<T> a, Cx<T> w)
{
    Cx<T> r;
    if (INV) {
        r.x = a.x * w.x + a.y * w.y;
        r.y = a.y * w.x - a.x * w.y;
    } else {
        r.x = a.x * w.x - a.y * w.y;
        r.y = a.y * w.x + a.x * w.y;
    }
    return r;
}

template <typename T>
__device__ inline void dft2(Cx<T>& a, Cx<T>& b)
{
    const Cx<T> s = a;
    a.x = s.x + b.x;
    a.y = s.y + b.y;
    b.x = s.x - b.x;
    b.y = s.y - b.y;
}

// In place: outputs k = 0 .. 3 in a, b, c, d.
template <typename T, bool INV>
__device__ inline void dft4(Cx<T>& a, Cx<T>& b, Cx<T>& c, Cx<T>& d)
{
    dft2(a, c);
    dft2(b, d);
    // d times -i (forward) or +i
    const T x = d.x;
    d.x = INV ? -d.y : d.y;
    d.y = INV ? x : -x;
    const Cx<T> s = a, t = c;
    a.x = s.x + b.x;
    a.y = s.y + b.y;
    c.x = s.x - b.x;
    c.y = s.y - b.y;
    b.x = t.x + d.x;
    b.y = t.y + d.y;
    d.x = t.x - d.x;
    d.y = t.y - d.y;
}

// DFT of R values in place, natural order in and out.
template <typename T, bool INV, int R>
__device__ inline void dft(Cx<T> (&v)[R])
{
    if constexpr (R == 2) {
        dft2(v[0], v[1]);
    } else if constexpr (R == 4) {
        dft4<T, INV>(v[0], v[1], v[2], v[3]);
    } else if constexpr (R == 8) {
        dft4<T, INV>(v[0], v[2], v[4], v[6]);
        dft4<T, INV>(v[1], v[3], v[5], v[7]);
        constexpr T r = T(0.70710678118654752440);
        // times exp(-2 pi i k / 8), k = 1 .. 3 (conjugate when INV)
        Cx<T> a = v[3], b = v[5], c = v[7];
        v[3].x = INV ? r * (a.x - a.y) : r * (a.x + a.y);
        v[3].y = INV ? r * (a.y + a.x) : r * (a.y - a.x);
        v[5].x = INV ? -b.y : b.y;
        v[5].y = INV ? b.x : -b.x;
        v[7].x = INV ? -r * (c.x + c.y) : r * (c.y - c.x);
        v[7].y = INV ? r * (c.x - c.y) : -r * (c.x + c.y);
        // v[2 k + s] holds output k of the even (s = 0) and odd half
#pragma unroll
        for (int k = 0; k < 4; ++k)
            dft2(v[2 * k], v[2 * k + 1]);
        Cx<T> o[8];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            o[k] = v[2 * k];
            o[k + 4] = v[2 * k + 1];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k)
            v[k] = o[k];
    } else {
        static_assert(R == 16, "radix 2, 4, 8 or 16");
        // y[s][k] = DFT4 over q of v[4 q + s], left in v[4 k + s]
#pragma unroll
        for (int s = 0; s < 4; ++s)
            dft4<T, INV>(v[s], v[4 + s], v[8 + s], v[12 + s]);
        constexpr T c = T(0.92387953251128675613), d = T(0.38268343236508977173),
                    r = T(0.70710678118654752440);
        const Cx<T> w1 = {c, -d}, w2 = {r, -r}, w3 = {d, -c}, w6 = {-r, -r}, w9 = {-c, d};
        v[4 + 1] = cmul<T, INV>(v[4 + 1], w1);
        v[4 + 2] = cmul<T, INV>(v[4 + 2], w2);
        v[4 + 3] = cmul<T, INV>(v[4 + 3], w3);
        v[8 + 1] = cmul<T, INV>(v[8 + 1], w2);
        {
            const Cx<T> a = v[8 + 2];        // times -i (forward) or +i
            v[8 + 2].x = INV ? -a.y : a.y;
            v[8 + 2].y = INV ? a.x : -a.x;
        }
        v[8 + 3] = cmul<T, INV>(v[8 + 3], w6);
        v[12 + 1] = cmul<T, INV>(v[12 + 1], w3);
        v[12 + 2] = cmul<T, INV>(v[12 + 2], w6);
        v[12 + 3] = cmul<T, INV>(v[12 + 3], w9);
        // output k + 4 m = DFT4 over s of y[s][k], m its index
        Cx<T> o[16];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            dft4<T, INV>(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
#pragma unroll
            for (int m = 0; m < 4; ++m)
                o[k + 4 * m] = v[4 * k + m];
        }
#pragma unroll
        for (int k = 0; k < 16; ++k)
            v[k] = o[k];
    }
}

// One Stockham pass of radix R on a line whose first NS-point transforms are
// done: the butterflies j = t + TPL q of thread t take registers q + r E / R.
template <typename T, bool INV, int LOGN, int R, int NS>
__device__ inline void fft_pass(Cx<T> (&v)[Line<LOGN>::E], int t, const Cx<T>* __restrict__ W)
{
    constexpr int E = Line<LOGN>::E, TPL = Line<LOGN>::TPL, Q = E / R, n = Line<LOGN>::n;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        Cx<T> a[R];
#pragma unroll
        for (int r = 0; r < R; ++r)
            a[r] = v[q + r * Q];
        if (NS > 1) {
            const int k = ((t + TPL * q) & (NS - 1)) * (n / (NS * R));
#pragma unroll
            for (int r = 1; r < R; ++r)
                a[r] = cmul<T, INV>(a[r], W[r * k]);
        }
        dft<T, INV, R>(a);
#pragma unroll
        for (int r = 0; r < R; ++r)
            v[q + r * Q] = a[r];
    }
}

// The exchange after such a pass: element i of the line sits at at(i) of buf
// (called by every thread of the workgroup; `live` marks those with a line).
template <typename T, int LOGN, int R, int NS, typename At>
__device__ inline void fft_exchange(Cx<T> (&v)[Line<LOGN>::E], int t, bool live, Cx<T>* buf,
                                    At at)
{
    constexpr int E = Line<LOGN>::E, TPL = Line<LOGN>::TPL, Q = E / R;
    __syncthreads();
    if (live) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int j = t + TPL * q;
            const int o = (j & ~(NS - 1)) * R + (j & (NS - 1));
#pragma unroll
            for (int r = 0; r < R; ++r)
                buf[at(o + r * NS)] = v[q + r * Q];
        }
    }
    __syncthreads();
    if (live) {
#pragma unroll
        for (int e = 0; e < E; ++e)
            v[e] = buf[at(t + TPL * e)];
    }
}

// Transform of the line in v.  W[q] = exp(-2 pi i q / n), q < n, in LDS.
// Called by every thread of the workgroup.  The exchange buffer may be written
// by others before the call and after it only behind a barrier.
template <typename T, bool INV, int LOGN, typename At>
__device__ inline void fft_line(Cx<T> (&v)[Line<LOGN>::E], int t, bool live, Cx<T>* buf, At at,
                                const Cx<T>* __restrict__ W)
{
    using L = Line<LOGN>;
    fft_pass<T, INV, LOGN, L::R0, 1>(v, t, W);
    if constexpr (L::R1 > 1) {
        fft_exchange<T, LOGN, L::R0, 1>(v, t, live, buf, at);
        fft_pass<T, INV, LOGN, L::R1, L::R0>(v, t, W);
    }
    if constexpr (L::R2 > 1) {
        fft_exchange<T, LOGN, L::R1, L::R0>(v, t, live, buf, at);
        fft_pass<T, INV, LOGN, L::R2, L::R0 * L::R1>(v, t, W);
    }
}

// W[q] = exp(-2 pi i q / n) for the whole workgroup (a barrier must follow).
template <typename T, int LOGN>
__device__ inline void fill_twiddles(Cx<T>* W)
{
    constexpr int n = 1 << LOGN;
    for (int q = threadIdx.x; q < n; q += blockDim.x) {
        double s, c;
        sincospi(-2.0 * (double)q / (double)n, &s, &c);
        W[q].x = (T)c;
        W[q].y = (T)s;
    }
}

}  // namespace ibx
