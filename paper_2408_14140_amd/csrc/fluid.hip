// fluid.hip -- single-level periodic fluid steps around the IB loop (Sec. 3.1):
// Step 1, the semi-implicit predictor of Eq. (31), and Step 3, the nodal
// projection of Eqs. (ns_lp1)-(ns_lp3).
//
// Grid: n^3 cells of edge h, periodic on every axis, n a power of two.
// Velocity is cell-centred [3][n][n][n] (x fastest); pressure lives on the
// nodes [n][n][n], node (i, j, k) at the low corner of cell (i, j, k).
//   G p (cell gradient of nodal p): the difference across the cell along the
//       axis, averaged over the cell's four edges parallel to it;
//   D V (nodal divergence of cell V): the difference between the two layers
//       of cells that share the node, each averaged over its four cells
//       (D = -G^T);
//   L: the 7-point Laplacian; the convective term in central flux form with
//       face values the mean of the two cells (the paper cites a Godunov
//       scheme without giving it).
// Both implicit solves are diagonal in Fourier space: real-to-complex along x,
// complex along y and z (fft.h), a per-mode scaling, and the way back.  A solve
// is five passes over the half spectrum [z][y][pitch] (n/2 + 1 of its columns
// used): the right-hand side is formed in the x pass, and the z pass goes
// forward, scales and comes back without leaving the registers.
#include <type_traits>

#include "fft.h"
#include "paths.h"

namespace ibx {

// Complex values per x row of the half spectrum: n/2 + 1, padded so that a
// group of columns starts on a 128-byte line (64 and above) and the three
// velocity components fit the workspace (below).
constexpr int spec_pitch(int n) { return n / 2 + (n >= 64 ? 16 : n >= 16 ? 8 : 4); }

// ------------------------------------------------------------------ stencils

// The stencils take 16 bytes of x cells per thread (4 in FP32, 2 in FP64) and
// one or two neighbours at the ends, so a cell costs about a quarter of the
// loads it would alone.  n is a multiple of 8, so a segment never wraps; rows
// may start at any element of the caller's arrays (global vector loads need
// element alignment only).
template <typename T>
struct Wide {
    static constexpr int W = 16 / sizeof(T);
    typedef T type __attribute__((ext_vector_type(16 / sizeof(T)), aligned(sizeof(T))));
};

// v[0 .. LO) the LO cells before cell i of a row, then cells i .. i + W - 1,
// then the HI cells after them (LO and HI 0 or 1, wrapped).
template <typename T, int LO, int HI>
__device__ inline void load_row(const T* row, int n, int i, T (&v)[LO + Wide<T>::W + HI])
{
    constexpr int W = Wide<T>::W;
    const typename Wide<T>::type m = *reinterpret_cast<const typename Wide<T>::type*>(row + i);
    if (LO)
        v[0] = row[(i - 1) & (n - 1)];
#pragma unroll
    for (int x = 0; x < W; ++x)
        v[LO + x] = m[x];
    if (HI)
        v[LO + W + HI - 1] = row[(i + W) & (n - 1)];
}

template <typename T>
__device__ inline void store_row(T* at, const T (&v)[Wide<T>::W])
{
    typename Wide<T>::type m;
#pragma unroll
    for (int x = 0; x < Wide<T>::W; ++x)
        m[x] = v[x];
    *reinterpret_cast<typename Wide<T>::type*>(at) = m;
}

// First element of row (j, k), wrapped.
__device__ inline int64_t row_at(int n, int j, int k)
{
    return (int64_t)n * ((j & (n - 1)) + (int64_t)n * (k & (n - 1)));
}

// G p at the W cells from (i, j, k), read from values of type T, formed in A,
// times scale (1/h, or 1/(h rho)).
template <typename T, typename A>
__device__ inline void grad_cells(const T* p, int n, int i, int j, int k, A scale,
                                  A (&g)[3][Wide<T>::W])
{
    constexpr int W = Wide<T>::W;
    A yl[W + 1], yh[W + 1], zd[W + 1];       // sums over z at j, at j + 1; difference along z
    T a[W + 1], b[W + 1], c[W + 1], d[W + 1];
    load_row<T, 0, 1>(p + row_at(n, j, k), n, i, a);
    load_row<T, 0, 1>(p + row_at(n, j + 1, k), n, i, b);
    load_row<T, 0, 1>(p + row_at(n, j, k + 1), n, i, c);
    load_row<T, 0, 1>(p + row_at(n, j + 1, k + 1), n, i, d);
#pragma unroll
    for (int x = 0; x <= W; ++x) {
        yl[x] = (A)a[x] + (A)c[x];
        yh[x] = (A)b[x] + (A)d[x];
        zd[x] = ((A)c[x] + (A)d[x]) - ((A)a[x] + (A)b[x]);
    }
    const A q = A(0.25) * scale;
#pragma unroll
    for (int x = 0; x < W; ++x) {
        g[0][x] = ((yl[x + 1] + yh[x + 1]) - (yl[x] + yh[x])) * q;
        g[1][x] = ((yh[x] + yh[x + 1]) - (yl[x] + yl[x + 1])) * q;
        g[2][x] = (zd[x] + zd[x + 1]) * q;
    }
}

// rhs of Eq. (31)
template <typename T>
struct PredictRhs {
    int n;
    T h, rho, a, dt, g0, g1, g2;
    const T* u;
    const T* p;
    __device__ void cells(int i, int j, int k, T (&rv)[3][Wide<T>::W]) const
    {
        constexpr int W = Wide<T>::W;
        const int64_t N = (int64_t)n * n * n;
        const T inv_h = T(1) / h, inv_h2 = inv_h * inv_h;
        const T g[3] = {g0, g1, g2};
        T uc[3][W + 2];
#pragma unroll
        for (int c = 0; c < 3; ++c)
            load_row<T, 1, 1>(u + c * N + row_at(n, j, k), n, i, uc[c]);
        T conv[3][W], lap[3][W];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            T um[3][W], up[3][W];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                if (d == 0) {
#pragma unroll
                    for (int x = 0; x < W; ++x) {
                        um[c][x] = uc[c][x];
                        up[c][x] = uc[c][x + 2];
                    }
                } else {
                    const int dj = d == 1, dk = d == 2;
                    load_row<T, 0, 0>(u + c * N + row_at(n, j - dj, k - dk), n, i, um[c]);
                    load_row<T, 0, 0>(u + c * N + row_at(n, j + dj, k + dk), n, i, up[c]);
                }
            }
#pragma unroll
            for (int x = 0; x < W; ++x) {
                const T fd_p = T(0.5) * (uc[d][x + 1] + up[d][x]);
                const T fd_m = T(0.5) * (um[d][x] + uc[d][x + 1]);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const T v = uc[c][x + 1];
                    const T fp = fd_p * (T(0.5) * (v + up[c][x]));
                    const T fm = fd_m * (T(0.5) * (um[c][x] + v));
                    const T cv = (fp - fm) * inv_h;
                    const T lp = (up[c][x] - T(2) * v + um[c][x]) * inv_h2;
                    conv[c][x] = d == 0 ? cv : conv[c][x] + cv;
                    lap[c][x] = d == 0 ? lp : lap[c][x] + lp;
                }
            }
        }
        T gp[3][W];
        grad_cells<T, T>(p, n, i, j, k, inv_h, gp);
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int x = 0; x < W; ++x)
                rv[c][x] = uc[c][x + 1] - dt * conv[c][x] - (dt / rho) * gp[c][x] +
                           a * lap[c][x] + dt * g[c];
    }
};

// V = u*/dt + G p_old / rho (Eq. (ns_lp1))
template <typename T>
__global__ void __launch_bounds__(256)
k_proj_V(int n, T h, T rho, T dt, const T* __restrict__ us, const T* __restrict__ p_old,
         T* __restrict__ V)
{
    constexpr int W = Wide<T>::W;
    const int64_t N = (int64_t)n * n * n;
    const int64_t q = ((int64_t)blockIdx.x * 256 + threadIdx.x) * W;
    if (q >= N)
        return;
    const int i = (int)(q & (n - 1)), j = (int)((q / n) & (n - 1)), k = (int)(q / ((int64_t)n * n));
    T g[3][W];
    grad_cells<T, T>(p_old, n, i, j, k, T(1) / h, g);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        T v[W];
        load_row<T, 0, 0>(us + c * N + q - i, n, i, v);
#pragma unroll
        for (int x = 0; x < W; ++x)
            v[x] = v[x] / dt + g[c][x] / rho;
        store_row(V + c * N + q, v);
    }
}

// The FP32 projection with one step of iterative refinement.  The FFT solve
// rounds its spectrum to FP32, and the low modes of that rounding are
// amplified by up to the condition number of D G (about n^2/pi^2).  A second
// solve of the first one's residual removes that error; the residual and the
// divergences are summed in A = FP64 from the FP32 cell values (whose own
// rounding perturbs p only as much as rounding the inputs does).
//   V = u*/dt + G p_old/rho;  p1 = rho (D G)^+ D V
//   W = V - G p1/rho;  d = rho (D G)^+ D W  (D W is the residual of p1)
//   p = p1 + d;  u^{n+1} = dt (W - G d/rho)

// D V at the nodes, summed in A from V of type T, rounded to T
template <typename T, typename A>
struct DivV {
    int n;
    A h;
    const T* V;
    __device__ void cells(int i, int j, int k, T (&out)[1][Wide<T>::W]) const
    {
        constexpr int W = Wide<T>::W;
        const int64_t N = (int64_t)n * n * n;
        const A q = A(0.25) / h;
        A sx[W + 1], syz[W + 1];             // x sums of the four rows; y and z differences
        T r[4][W + 1];
        auto rows = [&](int c) {
#pragma unroll
            for (int m = 0; m < 4; ++m)      // (j - 1, k - 1), (j, k - 1), (j - 1, k), (j, k)
                load_row<T, 1, 0>(V + c * N + row_at(n, j - 1 + (m & 1), k - 1 + (m >> 1)), n, i,
                                  r[m]);
        };
        rows(0);
#pragma unroll
        for (int x = 0; x <= W; ++x)
            sx[x] = ((A)r[0][x] + (A)r[1][x]) + ((A)r[2][x] + (A)r[3][x]);
        rows(1);
#pragma unroll
        for (int x = 0; x <= W; ++x)
            syz[x] = ((A)r[1][x] + (A)r[3][x]) - ((A)r[0][x] + (A)r[2][x]);
        rows(2);
#pragma unroll
        for (int x = 0; x <= W; ++x)
            syz[x] += ((A)r[2][x] + (A)r[3][x]) - ((A)r[0][x] + (A)r[1][x]);
#pragma unroll
        for (int x = 0; x < W; ++x)
            out[0][x] = (T)(((sx[x + 1] - sx[x]) + (syz[x] + syz[x + 1])) * q);
    }
};

// W = V - G p/rho, in place, formed in A
template <typename T, typename A>
__global__ void __launch_bounds__(256)
k_proj_W(int n, A h, A rho, const T* __restrict__ p, T* __restrict__ V)
{
    constexpr int W = Wide<T>::W;
    const int64_t N = (int64_t)n * n * n;
    const int64_t q = ((int64_t)blockIdx.x * 256 + threadIdx.x) * W;
    if (q >= N)
        return;
    const int i = (int)(q & (n - 1)), j = (int)((q / n) & (n - 1)), k = (int)(q / ((int64_t)n * n));
    A g[3][W];
    grad_cells<T, A>(p, n, i, j, k, A(1) / (h * rho), g);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        T v[W];
        load_row<T, 0, 0>(V + c * N + q - i, n, i, v);
#pragma unroll
        for (int x = 0; x < W; ++x)
            v[x] = (T)((A)v[x] - g[c][x]);
        store_row(V + c * N + q, v);
    }
}

// u^{n+1} = dt (W - G d/rho) and p = p1 + d (pn holds p1)
template <typename T, typename A>
__global__ void __launch_bounds__(256)
k_proj_final_refined(int n, A h, A rho, A dt, const T* __restrict__ Wf, const T* __restrict__ dl,
                     T* __restrict__ un, T* __restrict__ pn)
{
    constexpr int W = Wide<T>::W;
    const int64_t N = (int64_t)n * n * n;
    const int64_t q = ((int64_t)blockIdx.x * 256 + threadIdx.x) * W;
    if (q >= N)
        return;
    const int i = (int)(q & (n - 1)), j = (int)((q / n) & (n - 1)), k = (int)(q / ((int64_t)n * n));
    A g[3][W];
    grad_cells<T, A>(dl, n, i, j, k, A(1) / (h * rho), g);
    T v[W], d[W];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        load_row<T, 0, 0>(Wf + c * N + q - i, n, i, v);
#pragma unroll
        for (int x = 0; x < W; ++x)
            v[x] = (T)(dt * ((A)v[x] - g[c][x]));
        store_row(un + c * N + q, v);
    }
    load_row<T, 0, 0>(pn + q - i, n, i, v);
    load_row<T, 0, 0>(dl + q - i, n, i, d);
#pragma unroll
    for (int x = 0; x < W; ++x)
        v[x] = (T)((A)v[x] + (A)d[x]);
    store_row(pn + q, v);
}

// u^{n+1} = dt (V - G p / rho), Eq. (ns_lp3)
template <typename T>
__global__ void __launch_bounds__(256)
k_proj_final(int n, T h, T rho, T dt, const T* __restrict__ V, const T* __restrict__ pr,
             T* __restrict__ un)
{
    constexpr int W = Wide<T>::W;
    const int64_t N = (int64_t)n * n * n;
    const int64_t q = ((int64_t)blockIdx.x * 256 + threadIdx.x) * W;
    if (q >= N)
        return;
    const int i = (int)(q & (n - 1)), j = (int)((q / n) & (n - 1)), k = (int)(q / ((int64_t)n * n));
    T g[3][W];
    grad_cells<T, T>(pr, n, i, j, k, T(1) / h, g);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        T v[W];
        load_row<T, 0, 0>(V + c * N + q - i, n, i, v);
#pragma unroll
        for (int x = 0; x < W; ++x)
            v[x] = dt * (v[x] - g[c][x] / rho);
        store_row(un + c * N + q, v);
    }
}

// ------------------------------------------------------------------ passes

// x pass forward: R rows of y of one z plane per workgroup, NC fields.  The
// fields' values (src.cells) are formed into LDS; rows 2 m and
// 2 m + 1 of a field then share one complex transform, and its spectrum Z
// splits into theirs, A = (Z(k) + Z*(-k)) / 2 and B = (Z(k) - Z*(-k)) / 2i.
// Rows per workgroup: about 2048 cells of each field, so that the three
// fields stay near 26 KB of LDS in FP32; fewer on grids of up to 64, whose
// n^2 rows would leave compute units idle.
template <int LOGN, int NC>
struct XFwd {
    static constexpr int R = LOGN <= 4 ? 2 : LOGN == 5 ? 4 : LOGN == 6 ? 8 : 2048 >> LOGN;
    static constexpr int NL = NC * (R / 2);
    static constexpr int NT =
        NL * Line<LOGN>::TPL > 64 ? (NL * Line<LOGN>::TPL + 63) / 64 * 64 : 64;
};

template <typename T, int LOGN, int NC, typename Src>
__global__ void __launch_bounds__((XFwd<LOGN, NC>::NT))
k_fft_x_fwd(Src src, Cx<T>* __restrict__ spec)
{
    using L = Line<LOGN>;
    using K = XFwd<LOGN, NC>;
    constexpr int n = L::n, h = n / 2, PX = spec_pitch(n), R = K::R;
    __shared__ __align__(16) Cx<T> buf[K::NL * L::LDS];
    __shared__ Cx<T> W[n];
    T* const real = reinterpret_cast<T*>(buf);        // [NC][R][n]
    fill_twiddles<T, LOGN>(W);
    const int j0 = (blockIdx.x * R) & (n - 1), k = (blockIdx.x * R) >> LOGN;
    constexpr int VW = Wide<T>::W;
    for (int q = VW * threadIdx.x; q < R * n; q += VW * K::NT) {
        T v[NC][VW];
        src.cells(q & (n - 1), j0 + (q >> LOGN), k, v);
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int x = 0; x < VW; ++x)
                real[c * R * n + q + x] = v[c][x];
    }
    __syncthreads();
    const int line = threadIdx.x / L::TPL, t = threadIdx.x % L::TPL;
    const bool live = line < K::NL;
    const int c = live ? line / (R / 2) : 0, m = live ? line % (R / 2) : 0;
    Cx<T> v[L::E];
#pragma unroll
    for (int e = 0; e < L::E; ++e) {
        const T* r = real + (c * R + 2 * m) * n + t + L::TPL * e;
        v[e].x = r[0];
        v[e].y = r[n];
    }
    Cx<T>* const lb = buf + (live ? line : 0) * L::LDS;
    fft_line<T, false, LOGN>(v, t, live, lb, lds_at, W);
    __syncthreads();
    if (live) {
#pragma unroll
        for (int e = 0; e < L::E; ++e)
            lb[lds_at(t + L::TPL * e)] = v[e];
    }
    __syncthreads();
    if (!live)
        return;
    Cx<T>* const ra = spec + (((int64_t)c * n + k) * n + j0 + 2 * m) * PX;
    Cx<T>* const rb = ra + PX;
    auto split = [&](int q) {
        const Cx<T> z = lb[lds_at(q)], w = lb[lds_at((n - q) & (n - 1))];
        ra[q] = Cx<T>{T(0.5) * (z.x + w.x), T(0.5) * (z.y - w.y)};
        rb[q] = Cx<T>{T(0.5) * (z.y + w.y), T(0.5) * (w.x - z.x)};
    };
#pragma unroll
    for (int e = 0; e < L::E / 2; ++e)
        split(t + L::TPL * e);
    if (t == 0)
        split(h);
}

// x pass back to reals: rows 2 m and 2 m + 1 as the real and imaginary part of
// one complex transform, NL pairs per workgroup; out[c][z][y][x].
template <int LOGN>
struct XInv {
    static constexpr int NL = LOGN <= 3 ? 4 : LOGN <= 6 ? 4 : 128 / Line<LOGN>::TPL;
    static constexpr int NT = NL * Line<LOGN>::TPL > 64 ? NL * Line<LOGN>::TPL : 64;
};

template <typename T, int LOGN>
__global__ void __launch_bounds__(XInv<LOGN>::NT)
k_fft_x_inv(const Cx<T>* __restrict__ spec, T* __restrict__ out)
{
    using L = Line<LOGN>;
    using K = XInv<LOGN>;
    constexpr int n = L::n, h = n / 2, PX = spec_pitch(n);
    __shared__ __align__(16) Cx<T> buf[K::NL * L::LDS];
    __shared__ Cx<T> W[n];
    fill_twiddles<T, LOGN>(W);
    const int line = threadIdx.x / L::TPL, t = threadIdx.x % L::TPL;
    const bool live = line < K::NL;
    const int64_t row = 2 * ((int64_t)blockIdx.x * K::NL + (live ? line : 0));
    const Cx<T>* const ra = spec + row * PX;
    const Cx<T>* const rb = ra + PX;
    Cx<T> v[L::E];
    // Z(k) = A(k) + i B(k), with A(n - k) = A*(k); A and B are real at 0 and h
#pragma unroll
    for (int e = 0; e < L::E / 2; ++e) {
        const int k = t + L::TPL * e;
        const Cx<T> a = ra[k], b = rb[k];
        v[e].x = k == 0 ? a.x : a.x - b.y;
        v[e].y = k == 0 ? b.x : a.y + b.x;
    }
#pragma unroll
    for (int e = L::E / 2; e < L::E; ++e) {
        const int k = n - (t + L::TPL * e);           // 1 .. h
        const Cx<T> a = ra[k], b = rb[k];
        v[e].x = k == h ? a.x : a.x + b.y;
        v[e].y = k == h ? b.x : b.x - a.y;
    }
    __syncthreads();
    fft_line<T, true, LOGN>(v, t, live, buf + (live ? line : 0) * L::LDS, lds_at, W);
    if (!live)
        return;
    constexpr T scale = T(1.0 / n);
    T* const oa = out + row * n + t;
#pragma unroll
    for (int e = 0; e < L::E; ++e) {
        oa[L::TPL * e] = v[e].x * scale;
        oa[n + L::TPL * e] = v[e].y * scale;
    }
}

// y and z passes: C neighbouring columns per workgroup, so that an access moves C
// consecutive values: 128 bytes, or what the LDS allows on lines above 256 (64 bytes
// at 512 and 32 at 1024 in FP32).  Grids up to 64 take 8 columns, which is 64 bytes in
// FP32: 16 would make 192 workgroups of a field's 33 columns on 64^3, fewer than
// compute units.
template <typename T, int LOGN>
struct Cols {
    static constexpr int C = (LOGN <= 6 ? 8 : LOGN <= 8 ? 16 : LOGN == 9 ? 8 : 4) /
                             (sizeof(T) == 8 && LOGN > 6 ? 2 : 1);
    static constexpr int NT = C * Line<LOGN>::TPL;
    static constexpr int groups = ((1 << LOGN) / 2 + C) / C;   // of the n/2 + 1 columns
};

template <typename T, int LOGN, bool INV>
__global__ void __launch_bounds__((Cols<T, LOGN>::NT))
k_fft_y(Cx<T>* __restrict__ spec)
{
    using L = Line<LOGN>;
    using K = Cols<T, LOGN>;
    constexpr int n = L::n, PX = spec_pitch(n), C = K::C;
    __shared__ __align__(16) Cx<T> buf[L::LDS * C];
    __shared__ Cx<T> W[n];
    fill_twiddles<T, LOGN>(W);
    const int c = threadIdx.x % C, t = threadIdx.x / C;
    const int col = (int)(blockIdx.x % K::groups) * C + c;
    const bool live = col <= n / 2;
    Cx<T>* const p = spec + (int64_t)(blockIdx.x / K::groups) * n * PX + col;
    Cx<T> v[L::E];
    if (live) {
#pragma unroll
        for (int e = 0; e < L::E; ++e)
            v[e] = p[(t + L::TPL * e) * PX];
    }
    __syncthreads();
    fft_line<T, INV, LOGN>(v, t, live, buf, [&](int i) { return lds_at(i) * C + c; }, W);
    if (!live)
        return;
    constexpr T scale = INV ? T(1.0 / n) : T(1);
#pragma unroll
    for (int e = 0; e < L::E; ++e) {
        v[e].x *= scale;
        v[e].y *= scale;
        p[(t + L::TPL * e) * PX] = v[e];
    }
}

// Symbols along one axis, formed once per workgroup for the three axes alike,
// and a mode's factor from them.
// 1 / (1 - a lam(k)), lam the eigenvalue of the 7-point Laplacian
struct Helmholtz {
    double h, a;
    static constexpr int tables = 1;
    template <int N>
    __device__ void fill(double (*tab)[N], int k) const
    {
        tab[0][k] = (2.0 * cospi(2.0 * (double)k / (double)N) - 2.0) / (h * h);
    }
    template <int N>
    __device__ double factor(double (*tab)[N], int kx, int ky, int kz) const
    {
        const double lam = tab[0][kx] + tab[0][ky] + tab[0][kz];
        return 1.0 / (1.0 - a * lam);
    }
};

// rho / sigma(k), or 0 where sigma (the symbol of D G) vanishes
struct Poisson {
    double h, rho;
    static constexpr int tables = 2;
    template <int N>
    __device__ void fill(double (*tab)[N], int k) const
    {
        const double sv = sinpi((double)k / (double)N), cv = cospi((double)k / (double)N);
        tab[0][k] = sv * sv;
        tab[1][k] = cv * cv;
    }
    template <int N>
    __device__ double factor(double (*tab)[N], int kx, int ky, int kz) const
    {
        const double sig =
            -4.0 / (h * h) *
            (tab[0][kx] * tab[1][ky] * tab[1][kz] + tab[0][ky] * tab[1][kx] * tab[1][kz] +
             tab[0][kz] * tab[1][kx] * tab[1][ky]);
        // the largest |sigma| over all modes is 4/h^2 (one component at Nyquist)
        return fabs(sig) > 1e-10 * 4.0 / (h * h) ? rho / sig : 0.0;
    }
};

// z pass: forward, times the symbol, back, for NC fields with one symbol.
template <typename T, int LOGN, int NC, typename Sym>
__global__ void __launch_bounds__((Cols<T, LOGN>::NT))
k_fft_z_solve(Sym sym, Cx<T>* __restrict__ spec)
{
    using L = Line<LOGN>;
    using K = Cols<T, LOGN>;
    constexpr int n = L::n, PX = spec_pitch(n), C = K::C;
    __shared__ __align__(16) Cx<T> buf[L::LDS * C];
    __shared__ Cx<T> W[n];
    __shared__ double tab[Sym::tables][n];
    fill_twiddles<T, LOGN>(W);
    for (int q = threadIdx.x; q < n; q += K::NT)
        sym.template fill<n>(tab, q);
    const int c = threadIdx.x % C, t = threadIdx.x / C;
    const int col = (int)(blockIdx.x % K::groups) * C + c, ky = (int)(blockIdx.x / K::groups);
    const bool live = col <= n / 2;
    auto at = [&](int i) { return lds_at(i) * C + c; };
    __syncthreads();
    T f[L::E];
    if (live) {
#pragma unroll
        for (int e = 0; e < L::E; ++e)
            f[e] = (T)sym.template factor<n>(tab, col, ky, t + L::TPL * e) * T(1.0 / n);
    }
#pragma unroll 1
    for (int m = 0; m < NC; ++m) {
        Cx<T>* const p = spec + ((int64_t)m * n * n + ky) * PX + col;
        Cx<T> v[L::E];
        if (live) {
#pragma unroll
            for (int e = 0; e < L::E; ++e)
                v[e] = p[(int64_t)(t + L::TPL * e) * n * PX];
        }
        fft_line<T, false, LOGN>(v, t, live, buf, at, W);
        if (live) {
#pragma unroll
            for (int e = 0; e < L::E; ++e) {
                v[e].x *= f[e];
                v[e].y *= f[e];
            }
        }
        fft_line<T, true, LOGN>(v, t, live, buf, at, W);
        if (live) {
#pragma unroll
            for (int e = 0; e < L::E; ++e)
                p[(int64_t)(t + L::TPL * e) * n * PX] = v[e];
        }
    }
}

// out = the inverse of sym applied to NC fields given cell by cell.
template <typename T, int LOGN, int NC, typename Src, typename Sym>
static void solve(const Src& src, const Sym& sym, Cx<T>* spec, T* out, hipStream_t st)
{
    constexpr unsigned n = 1u << LOGN;
    using X = XFwd<LOGN, NC>;
    using XI = XInv<LOGN>;
    using K = Cols<T, LOGN>;
    k_fft_x_fwd<T, LOGN, NC, Src><<<n * n / X::R, X::NT, 0, st>>>(src, spec);
    k_fft_y<T, LOGN, false><<<K::groups * n * NC, K::NT, 0, st>>>(spec);
    k_fft_z_solve<T, LOGN, NC, Sym><<<K::groups * n, K::NT, 0, st>>>(sym, spec);
    k_fft_y<T, LOGN, true><<<K::groups * n * NC, K::NT, 0, st>>>(spec);
    k_fft_x_inv<T, LOGN><<<NC * n * n / (2 * XI::NL), XI::NT, 0, st>>>(spec, out);
}

// ------------------------------------------------------------------ layouts

template <typename T>
__global__ void k_to_boxes(Grid g, const T* __restrict__ glob, T* __restrict__ boxed)
{
    const int64_t cells = (int64_t)g.box * g.box * g.box;
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= (int64_t)g.nbox * cells)
        return;
    const int bid = (int)(q / cells);
    const int64_t r = q - (int64_t)bid * cells;
    const int lx = (int)(r % g.box), ly = (int)((r / g.box) % g.box), lz = (int)(r / ((int64_t)g.box * g.box));
    const int cx = g.box_lo[3 * bid] + lx, cy = g.box_lo[3 * bid + 1] + ly,
              cz = g.box_lo[3 * bid + 2] + lz;
    const int64_t N = (int64_t)g.n[0] * g.n[1] * g.n[2];
    const int64_t gq = cx + (int64_t)g.n[0] * (cy + (int64_t)g.n[1] * cz);
    const int64_t bo = (int64_t)bid * g.bstride +
                       ((int64_t)(lz + g.ngrow) * g.ext + (ly + g.ngrow)) * g.ext + lx + g.ngrow;
#pragma unroll
    for (int c = 0; c < 3; ++c)
        boxed[bo + c * g.cstride] = glob[c * N + gq];
}

template <typename T>
__global__ void k_from_boxes(Grid g, const T* __restrict__ boxed, T* __restrict__ glob)
{
    const int64_t cells = (int64_t)g.box * g.box * g.box;
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= (int64_t)g.nbox * cells)
        return;
    const int bid = (int)(q / cells);
    const int64_t r = q - (int64_t)bid * cells;
    const int lx = (int)(r % g.box), ly = (int)((r / g.box) % g.box), lz = (int)(r / ((int64_t)g.box * g.box));
    const int cx = g.box_lo[3 * bid] + lx, cy = g.box_lo[3 * bid + 1] + ly,
              cz = g.box_lo[3 * bid + 2] + lz;
    const int64_t N = (int64_t)g.n[0] * g.n[1] * g.n[2];
    const int64_t gq = cx + (int64_t)g.n[0] * (cy + (int64_t)g.n[1] * cz);
    const int64_t bo = (int64_t)bid * g.bstride +
                       ((int64_t)(lz + g.ngrow) * g.ext + (ly + g.ngrow)) * g.ext + lx + g.ngrow;
#pragma unroll
    for (int c = 0; c < 3; ++c)
        glob[c * N + gq] = boxed[bo + c * g.cstride];
}

// ------------------------------------------------------------------ host

static int log2_exact(int32_t n)
{
    int l = 0;
    while ((1 << l) < n)
        ++l;
    return (1 << l) == n ? l : -1;
}

// Reals of the workspace: a predictor holds the half spectra of three fields, a
// projection V, one half spectrum and (FP32) the correction.
static size_t fluid_reals(int32_t n) { return 7 * (size_t)n * n * n; }

template <typename T, int LOGN>
static void predict_n(double h, double rho, double mu, double dt, const double* grav, const T* u,
                      const T* p, T* ustar, T* ws, hipStream_t st)
{
    constexpr int n = 1 << LOGN;
    static_assert(3 * 2 * (size_t)n * n * spec_pitch(n) <= 7 * (size_t)n * n * n,
                  "three half spectra fit the workspace");
    const double a = 0.5 * (mu / rho) * dt;
    const PredictRhs<T> src{n,          (T)h,       (T)rho,     (T)a, (T)dt,
                            (T)grav[0], (T)grav[1], (T)grav[2], u,    p};
    solve<T, LOGN, 3>(src, Helmholtz{h, a}, reinterpret_cast<Cx<T>*>(ws), ustar, st);
}

template <typename T, int LOGN>
static void project_n(double h, double rho, double dt, const T* ustar, const T* p_old, T* u_new,
                      T* p_new, T* ws, hipStream_t st)
{
    constexpr int n = 1 << LOGN;
    constexpr size_t N = (size_t)n * n * n, S = 2 * (size_t)n * n * spec_pitch(n);
    static_assert(3 * N + S + N <= 7 * N, "V, a half spectrum and the correction fit");
    const unsigned gc = (unsigned)((N / Wide<T>::W + 255) / 256);
    T* V = ws;
    Cx<T>* spec = reinterpret_cast<Cx<T>*>(ws + 3 * N);
    T* dl = ws + 3 * N + S;
    const Poisson sym{h, rho};
    // p_old, which p_new may overwrite, is read by the first kernel only
    k_proj_V<T><<<gc, 256, 0, st>>>(n, (T)h, (T)rho, (T)dt, ustar, p_old, V);
    if constexpr (sizeof(T) == 4) {
        // FP32: two solves, the divergences and the residual summed in FP64
        const DivV<T, double> div{n, h, V};
        solve<T, LOGN, 1>(div, sym, spec, p_new, st);
        k_proj_W<T, double><<<gc, 256, 0, st>>>(n, h, rho, p_new, V);
        solve<T, LOGN, 1>(div, sym, spec, dl, st);
        k_proj_final_refined<T, double><<<gc, 256, 0, st>>>(n, h, rho, dt, V, dl, u_new, p_new);
    } else {
        solve<T, LOGN, 1>(DivV<T, T>{n, (T)h, V}, sym, spec, p_new, st);
        k_proj_final<T><<<gc, 256, 0, st>>>(n, (T)h, (T)rho, (T)dt, V, p_new, u_new);
    }
}

// fn<LOGN>() for the grid's LOGN (8 <= n <= 1024 was checked).
template <typename Fn>
static void for_logn(int32_t n, Fn fn)
{
    switch (log2_exact(n)) {
    case 3: fn(std::integral_constant<int, 3>()); break;
    case 4: fn(std::integral_constant<int, 4>()); break;
    case 5: fn(std::integral_constant<int, 5>()); break;
    case 6: fn(std::integral_constant<int, 6>()); break;
    case 7: fn(std::integral_constant<int, 7>()); break;
    case 8: fn(std::integral_constant<int, 8>()); break;
    case 9: fn(std::integral_constant<int, 9>()); break;
    case 10: fn(std::integral_constant<int, 10>()); break;
    }
}

template <typename T>
static int predict_t(int32_t n, double h, double rho, double mu, double dt, const double* grav,
                     const T* u, const T* p, T* ustar, void* ws, size_t ws_bytes, hipStream_t st)
{
    if (!ws || ws_bytes < fluid_reals(n) * sizeof(T))
        return IB_EWORKSPACE;
    for_logn(n, [&](auto L) {
        predict_n<T, L.value>(h, rho, mu, dt, grav, u, p, ustar, (T*)ws, st);
    });
    return launch_status();
}

template <typename T>
static int project_t(int32_t n, double h, double rho, double dt, const T* ustar, const T* p_old,
                     T* u_new, T* p_new, void* ws, size_t ws_bytes, hipStream_t st)
{
    if (!ws || ws_bytes < fluid_reals(n) * sizeof(T))
        return IB_EWORKSPACE;
    for_logn(n, [&](auto L) {
        project_n<T, L.value>(h, rho, dt, ustar, p_old, u_new, p_new, (T*)ws, st);
    });
    return launch_status();
}

}  // namespace ibx

using namespace ibx;

static int check_fluid(int32_t n, double h, ib_prec prec)
{
    if (n < 8 || n > 1024 || log2_exact(n) < 0)
        return IB_EUNSUPPORTED;
    if (!(h > 0.0) || (prec != IB_F32 && prec != IB_F64))
        return IB_EINVAL;
    return IB_OK;
}

extern "C" size_t ib_fluid_workspace(int32_t n, ib_prec prec)
{
    if (check_fluid(n, 1.0, prec))
        return 0;
    return fluid_reals(n) * (prec == IB_F64 ? sizeof(double) : sizeof(float));
}

extern "C" int ib_fluid_predict(int32_t n, double h, ib_prec prec, double rho, double mu,
                                double dt, const double* grav, const void* u, const void* p,
                                void* ustar, void* ws, size_t ws_bytes, void* stream)
{
    int rc = check_fluid(n, h, prec);
    if (rc)
        return rc;
    if (!(rho > 0.0) || !(mu >= 0.0) || !(dt > 0.0) || !grav || !u || !p || !ustar)
        return IB_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    if (prec == IB_F64)
        return predict_t<double>(n, h, rho, mu, dt, grav, (const double*)u, (const double*)p,
                                 (double*)ustar, ws, ws_bytes, st);
    return predict_t<float>(n, h, rho, mu, dt, grav, (const float*)u, (const float*)p,
                            (float*)ustar, ws, ws_bytes, st);
}

extern "C" int ib_fluid_project(int32_t n, double h, ib_prec prec, double rho, double dt,
                                const void* ustar, const void* p_old, void* u_new, void* p_new,
                                void* ws, size_t ws_bytes, void* stream)
{
    int rc = check_fluid(n, h, prec);
    if (rc)
        return rc;
    if (!(rho > 0.0) || !(dt > 0.0) || !ustar || !p_old || !u_new || !p_new)
        return IB_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    if (prec == IB_F64)
        return project_t<double>(n, h, rho, dt, (const double*)ustar, (const double*)p_old,
                                 (double*)u_new, (double*)p_new, ws, ws_bytes, st);
    return project_t<float>(n, h, rho, dt, (const float*)ustar, (const float*)p_old,
                            (float*)u_new, (float*)p_new, ws, ws_bytes, st);
}

extern "C" int ib_field_to_boxes(const ib_level* lv, ib_prec prec, const void* glob, void* boxed,
                                 void* stream)
{
    int rc = check_level(lv);
    if (rc)
        return rc;
    if (!glob || !boxed || (prec != IB_F32 && prec != IB_F64))
        return IB_EINVAL;
    const Grid g = make_grid(lv);
    const int64_t m = (int64_t)g.nbox * g.box * g.box * g.box;
    if (m == 0)
        return IB_OK;
    const unsigned gb = (unsigned)((m + 255) / 256);
    if (prec == IB_F64)
        k_to_boxes<double><<<gb, 256, 0, (hipStream_t)stream>>>(g, (const double*)glob,
                                                                 (double*)boxed);
    else
        k_to_boxes<float><<<gb, 256, 0, (hipStream_t)stream>>>(g, (const float*)glob,
                                                                (float*)boxed);
    return launch_status();
}

extern "C" int ib_field_from_boxes(const ib_level* lv, ib_prec prec, const void* boxed,
                                   void* glob, void* stream)
{
    int rc = check_level(lv);
    if (rc)
        return rc;
    if (!glob || !boxed || (prec != IB_F32 && prec != IB_F64))
        return IB_EINVAL;
    const Grid g = make_grid(lv);
    const int64_t m = (int64_t)g.nbox * g.box * g.box * g.box;
    if (m == 0)
        return IB_OK;
    const unsigned gb = (unsigned)((m + 255) / 256);
    if (prec == IB_F64)
        k_from_boxes<double><<<gb, 256, 0, (hipStream_t)stream>>>(g, (const double*)boxed,
                                                                   (double*)glob);
    else
        k_from_boxes<float><<<gb, 256, 0, (hipStream_t)stream>>>(g, (const float*)boxed,
                                                                  (float*)glob);
    return launch_status();
}
