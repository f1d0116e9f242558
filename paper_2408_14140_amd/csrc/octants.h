// octants.h -- spreading one 8^3 tile by matrix products, octant by octant: the
// weights, and what k_spread_mfma (tiles.h) and ib_spread (plain.hip) share.
#pragma once

#include "ibx_internal.h"

namespace ibx {

// The P weights of one axis from r = s - b - 1/2.  With d = r - 1 the
// distances to the P stencil points are 1 + d, |d|, 1 - d (and 2 - d), each
// on a fixed branch of the kernel, and all branches share one square root.
// P = 4: r in [1, 2), phi = (3 - 2|x| + q)/8 or (5 - 2|x| - q')/8 with
// q^2 = 1 + 4d - 4d^2; P = 3: r in [1/2, 3/2), q^2 = 1 - 3d^2.
__device__ inline float root(float x)
{
    return __builtin_amdgcn_sqrtf(x);   // the hardware square root (1 ulp), x in [1/4, 2]
}

__device__ inline double root(double x)
{
    return sqrt(x);
}

template <typename T, int P>
__device__ inline void axis_weights_r(T r, T* w)
{
    const T d = r - T(1);
    if (P == 4) {
        const T q = root(T(1) + T(4) * d * (T(1) - d)) * T(0.125);
        const T a = T(0.375) - T(0.25) * d, b = T(0.125) + T(0.25) * d;
        w[0] = a - q;
        w[1] = a + q;
        w[2] = b + q;
        w[3] = b - q;
    } else {
        const T q = root(T(1) - T(3) * d * d);
        const T q6 = q * T(1.0 / 6.0);
        w[0] = T(1.0 / 3.0) - T(0.5) * d - q6;
        w[1] = T(1.0 / 3.0) + T(1.0 / 3.0) * q;
        w[P - 1] = T(1.0 / 3.0) + T(0.5) * d - q6;
    }
}

// Matrix products D += A B of 16 x 4 by 4 x 16 values.  Operands: lane l holds
// A[l % 16][l / 16] and B[l / 16][l % 16].  Result: register r of lane l holds
// column l % 16 and row 4 (l / 16) + r (FP32) or l / 16 + 4 r (FP64).
template <typename T>
struct Mat;
template <>
struct Mat<float> {
    typedef float acc __attribute__((ext_vector_type(4)));
    static __device__ acc mac(float a, float b, acc c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
};
template <>
struct Mat<double> {
    typedef double acc __attribute__((ext_vector_type(4)));
    static __device__ acc mac(double a, double b, acc c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
};

// Memory accesses of the wavefront's lanes before this point stay before those after
// it (no instruction: one wavefront's LDS accesses are carried out in order).
__device__ inline void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Number of set bits of m below this lane's.
__device__ inline int bits_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Spreading a tile is the matrix product
//   G[(x, c)][(y, z)] = sum over sources k of (w^x_k F_k)[(x, c)] (w^y_k w^z_k)[(y, z)]
// formed per octant of 4^3 cells on the matrix cores by one wavefront: 12 of 16
// rows (x, c), 16 columns (y, z), four sources an instruction.  A source of a
// tile reaches 1.27 (P = 4) or 1.2 (P = 3) of the tile's two halves along an
// axis on average, about a quarter of its octants, and each octant takes only
// the sources that reach it: sources are staged 64 at a time as records in LDS
// (per axis the weight of each of the tile's 8 cells, zero outside the stencil,
// and F with its factor), and each octant's sources are listed in order.  Lists
// are padded with an all-zero record.  A record is 27 values, an odd number, so
// the lanes that stage (one source each) and those that read (four sources,
// four cells) fall on different banks.  The operands need x and y at one
// lane-dependent place, c and z at another, so a group of four sources is two
// paired LDS reads, two products and one matrix instruction: about 6 vector
// instructions for 4 x 64 cells x 3.  Every cell's sum is formed in one register
// in list order: bit-reproducible.
// A source whose F is not finite would turn zero weights into NaN for its whole
// octant; such sources are added apart, to the cells that they reach only.
// SMALL: an axis may have 8 cells only, where a periodic stencil wraps onto its
// own tile.
template <typename T, int P, bool SMALL>
struct Octants {
    using Acc = typename Mat<T>::acc;
    static constexpr int S = 3 * TILE + 3, WX = 0, WY = TILE, WZ = 2 * TILE, WF = 3 * TILE;
    static constexpr int FPL = (65 * S * (int)sizeof(T) + 1023) / 1024;   // 16-byte fills a lane
    // 64 sources, one zero record, and a word per lane for what falls outside
    static constexpr int OUT = FPL * 1024 / (int)sizeof(T);
    struct Lds {
        T rec[OUT + 64];
        uint16_t list[8 * 64];              // [octant][source of a group][group]: offsets
    };
    T* rec;
    uint16_t* list;
    int lane;
    int ixy, icz;          // place of this lane's x and y, and of its c and z, in an octant
    int kq;                // source of a group that it reads; c of its results
    int cnt[8];            // sources of each octant
    uint64_t odds;         // staged sources whose F is not finite

    __device__ explicit Octants(Lds& m, int ln = threadIdx.x) : rec(m.rec), list(m.list), lane(ln)
    {
        ixy = sizeof(T) == 4 ? lane & 3 : (lane >> 2) & 3;
        icz = sizeof(T) == 4 ? (lane >> 2) & 3 : lane & 3;
        kq = lane >> 4;
    }

    // Before a batch: zero records, and lists of the zero record.  The lanes clear
    // places that other lanes fill next, so the stores must keep their order: the
    // wavefront's LDS does by itself, the fence makes the compiler do so as well.
    __device__ void clear()
    {
        typedef T Fill __attribute__((ext_vector_type(16 / sizeof(T)), may_alias));
        typedef uint32_t Fill4 __attribute__((ext_vector_type(4), may_alias));
#pragma unroll
        for (int q = 0; q < FPL; ++q)
            reinterpret_cast<Fill*>(rec)[lane + 64 * q] = Fill(T(0));
        constexpr uint32_t z = 64 * S * sizeof(T);
        reinterpret_cast<Fill4*>(list)[lane] = Fill4(z | z << 16);
        wave_order();
    }

    // Which halves of the tile a lane's source reaches.
    struct Reach {
        bool lower[3] = {false, false, false}, upper[3] = {false, false, false}, odd = false;
    };

    // Weights w of a source whose stencil starts at tile cell b along axis ax
    // (wrap: modulo 8).
    __device__ void put(Reach& r, int ax, int b, const T (&w)[P], bool wrap)
    {
        if (SMALL) {
            r.lower[ax] = r.upper[ax] = false;
#pragma unroll
            for (int o = 0; o < P; ++o) {
                const int c = wrap ? (b + o) & (TILE - 1) : b + o;
                const bool in = (unsigned)c < (unsigned)TILE;
                rec[in ? lane * S + TILE * ax + c : OUT + lane] = w[o];
                r.lower[ax] = r.lower[ax] || (in && c < TILE / 2);
                r.upper[ax] = r.upper[ax] || (in && c >= TILE / 2);
            }
        } else {
#pragma unroll
            for (int o = 0; o < P; ++o)
                rec[(unsigned)(b + o) < (unsigned)TILE ? lane * S + TILE * ax + b + o
                                                       : OUT + lane] = w[o];
            r.lower[ax] = b < TILE / 2;
            r.upper[ax] = b + P > TILE / 2;
        }
    }

    // Its F, after its weights.
    __device__ void put_force(Reach& r, T F0, T F1, T F2)
    {
        r.odd = !(fabs(F0) + fabs(F1) + fabs(F2) < (T)__builtin_inf());
        rec[lane * S + WF] = F0;
        rec[lane * S + WF + 1] = F1;
        rec[lane * S + WF + 2] = F2;
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            r.lower[ax] = r.lower[ax] && !r.odd;
            r.upper[ax] = r.upper[ax] && !r.odd;
        }
    }

    // The octants' lists (all lanes; r default where a lane has no source).
    __device__ void make_lists(const Reach& r)
    {
        odds = __ballot(r.odd);
#pragma unroll
        for (int o = 0; o < 8; ++o) {
            const bool in = (o & 1 ? r.upper[0] : r.lower[0]) &&
                            (o & 2 ? r.upper[1] : r.lower[1]) &&
                            (o & 4 ? r.upper[2] : r.lower[2]);
            const uint64_t m = __ballot(in);
            const int rank = bits_below(m);
            cnt[o] = __popcll(m);
            if (in)
                list[64 * o + 16 * (rank & 3) + (rank >> 2)] =
                    (uint16_t)(lane * S * (int)sizeof(T));
        }
    }

    // acc[o] += the batch's contributions to octant o = xh + 2 yh + 4 zh: lane
    // holds column (y, z) = (ixy, icz), c = kq (3: nothing), registers along x.
    // (Reading two octants ahead under scheduling barriers, with the lists
    // padded to eight sources, was slower: 94 us against 85.)
    __device__ void add(Acc (&acc)[8])
    {
        typedef uint32_t Pair32 __attribute__((may_alias));
        const char* const base = reinterpret_cast<const char*>(rec);
#pragma unroll
        for (int o = 0; o < 8; ++o) {
            const int ox = WX + 4 * (o & 1), oy = WY + 4 * ((o >> 1) & 1), oz = WZ + 4 * (o >> 2);
            for (int gr = 0; 4 * gr < cnt[o]; gr += 2) {
                const uint32_t e =
                    *reinterpret_cast<const Pair32*>(list + 64 * o + 16 * kq + gr);
                T a[2], b[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const T* const p =
                        reinterpret_cast<const T*>(base + (h ? e >> 16 : e & 0xffffu));
                    const T* const p1 = p + ixy;
                    const T* const p2 = p + icz;
                    a[h] = p1[ox] * p2[WF];
                    b[h] = p1[oy] * p2[oz];
                }
                acc[o] = Mat<T>::mac(a[0], b[0], acc[o]);
                acc[o] = Mat<T>::mac(a[1], b[1], acc[o]);
            }
        }
        for (uint64_t m = odds; m; m &= m - 1) {
            const T* const q = rec + __builtin_ctzll(m) * S;
#pragma unroll
            for (int o = 0; o < 8; ++o) {
                const T wyz = q[WY + 4 * ((o >> 1) & 1) + ixy] * q[WZ + 4 * (o >> 2) + icz];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const T w = q[WX + 4 * (o & 1) + i] * wyz;
                    if (kq < 3 && w != T(0))
                        acc[o][i] += q[WF + kq] * w;
                }
            }
        }
    }

    // The same for octant o, with n listed sources.
    __device__ void add_one(int o, int n, Acc& acc)
    {
        typedef uint32_t Pair32 __attribute__((may_alias));
        const char* const base = reinterpret_cast<const char*>(rec);
        const int x = WX + 4 * (o & 1), y = WY + 4 * ((o >> 1) & 1) + ixy;
        const int z = WZ + 4 * (o >> 2) + icz;
        for (int gr = 0; 4 * gr < n; gr += 2) {
            const uint32_t e = *reinterpret_cast<const Pair32*>(list + 64 * o + 16 * kq + gr);
            T a[2], b[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const T* const p = reinterpret_cast<const T*>(base + (h ? e >> 16 : e & 0xffffu));
                a[h] = p[x + ixy] * p[WF + icz];
                b[h] = p[y] * p[z];
            }
            acc = Mat<T>::mac(a[0], b[0], acc);
            acc = Mat<T>::mac(a[1], b[1], acc);
        }
        for (uint64_t m = odds; m; m &= m - 1) {
            const T* const q = rec + __builtin_ctzll(m) * S;
            const T wyz = q[y] * q[z];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const T w = q[x + i] * wyz;
                if (kq < 3 && w != T(0))
                    acc[i] += q[WF + kq] * w;
            }
        }
    }
};

}  // namespace ibx
