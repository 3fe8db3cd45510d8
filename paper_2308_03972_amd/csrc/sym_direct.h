// Direct (iteration-free) functions of small symmetric matrices for the analysis:
// Householder tridiagonalisation, a sum of shifted tridiagonal inverses
// (sqrt_poles.h) and the back transformation: four nodes per wavefront up to N = 32
// (described here), two up to 48, one up to 64.
//
// Layout: a node owns a row of 16 lanes; lane r holds rows r and r + 16 (N > 16) of
// its N x N matrix in registers.  Everything one lane needs of another's comes
// through v_fmac_f64_dpp row_newbcast, which broadcasts lane j of the row as the
// multiplicand: a matrix-vector product or a rank-2 update is one instruction per
// entry with no LDS traffic, where a Jacobi round costs six FP64 operations per entry
// and both halves of an LDS exchange, N rounds per sweep, five to six sweeps.
#pragma once
#include <type_traits>

#include "common.h"
#include "device_util.h"
#include "sqrt_poles.h"

namespace lbmletkf {
namespace dev {

// ---------------------------------------------------------------------------
// broadcasts inside the row of 16 lanes
// ---------------------------------------------------------------------------
template <int L>
__device__ __forceinline__ double row_bcast(double x) {
    return __builtin_amdgcn_mov_dpp(x, 0x150 + L, 0xF, 0xF, true);
}

// Value of lane l (0..15, wave-uniform) of each row, through the LDS crossbar.
__device__ __forceinline__ double row_bcast_dyn(double x, int l, int lane) {
    const int addr = ((lane & 48) + l) * 4;
    const int lo = __builtin_amdgcn_ds_bpermute(addr, __double2loint(x));
    const int hi = __builtin_amdgcn_ds_bpermute(addr, __double2hiint(x));
    return __hiloint2double(hi, lo);
}

// The v_fmac_f64_dpp blocks: written as assembly because the compiler does not fold
// a 64-bit row_newbcast into the multiply-add.  A DPP operand written by one of the
// two preceding VALU instructions is a hazard the compiler does not see inside an
// assembly block, so every block opens with two wait states.
#define LBM_FMAC_DPP(d, s, y, l) \
    "v_fmac_f64_dpp %" #d ", %" #s ", %" #y " row_newbcast:%" #l " row_mask:0xf bank_mask:0xf\n\t"

// a[k] += bcast(x, L + k) * y, k < CNT
template <int L, int CNT>
__device__ __forceinline__ void fmac_axpy(double* a, double x, double y) {
    if constexpr (CNT >= 8) {
        asm("s_nop 1\n\t" LBM_FMAC_DPP(0, 8, 9, 10) LBM_FMAC_DPP(1, 8, 9, 11)
                LBM_FMAC_DPP(2, 8, 9, 12) LBM_FMAC_DPP(3, 8, 9, 13) LBM_FMAC_DPP(4, 8, 9, 14)
                    LBM_FMAC_DPP(5, 8, 9, 15) LBM_FMAC_DPP(6, 8, 9, 16) LBM_FMAC_DPP(7, 8, 9, 17)
            : "+&v"(a[0]), "+&v"(a[1]), "+&v"(a[2]), "+&v"(a[3]), "+&v"(a[4]), "+&v"(a[5]),
              "+&v"(a[6]), "+&v"(a[7])
            : "v"(x), "v"(y), "n"(L), "n"(L + 1), "n"(L + 2), "n"(L + 3), "n"(L + 4), "n"(L + 5),
              "n"(L + 6), "n"(L + 7));
        if constexpr (CNT > 8) fmac_axpy<L + 8, CNT - 8>(a + 8, x, y);
    } else if constexpr (CNT >= 4) {
        asm("s_nop 1\n\t" LBM_FMAC_DPP(0, 4, 5, 6) LBM_FMAC_DPP(1, 4, 5, 7)
                LBM_FMAC_DPP(2, 4, 5, 8) LBM_FMAC_DPP(3, 4, 5, 9)
            : "+&v"(a[0]), "+&v"(a[1]), "+&v"(a[2]), "+&v"(a[3])
            : "v"(x), "v"(y), "n"(L), "n"(L + 1), "n"(L + 2), "n"(L + 3));
        if constexpr (CNT > 4) fmac_axpy<L + 4, CNT - 4>(a + 4, x, y);
    } else if constexpr (CNT >= 2) {
        asm("s_nop 1\n\t" LBM_FMAC_DPP(0, 2, 3, 4) LBM_FMAC_DPP(1, 2, 3, 5)
            : "+&v"(a[0]), "+&v"(a[1])
            : "v"(x), "v"(y), "n"(L), "n"(L + 1));
        if constexpr (CNT > 2) fmac_axpy<L + 2, CNT - 2>(a + 2, x, y);
    } else if constexpr (CNT == 1) {
        asm("s_nop 1\n\t" LBM_FMAC_DPP(0, 1, 2, 3) : "+&v"(a[0]) : "v"(x), "v"(y), "n"(L));
    }
}

// s0 + s1 += sum_k bcast(x, L + k) * a[k], k < CNT (two partial sums)
template <int L, int CNT>
__device__ __forceinline__ void fmac_dot(const double* a, double x, double& s0, double& s1) {
    if constexpr (CNT >= 8) {
        asm("s_nop 1\n\t" LBM_FMAC_DPP(0, 2, 3, 11) LBM_FMAC_DPP(1, 2, 4, 12)
                LBM_FMAC_DPP(0, 2, 5, 13) LBM_FMAC_DPP(1, 2, 6, 14) LBM_FMAC_DPP(0, 2, 7, 15)
                    LBM_FMAC_DPP(1, 2, 8, 16) LBM_FMAC_DPP(0, 2, 9, 17) LBM_FMAC_DPP(1, 2, 10, 18)
            : "+&v"(s0), "+&v"(s1)
            : "v"(x), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]),
              "v"(a[7]), "n"(L), "n"(L + 1), "n"(L + 2), "n"(L + 3), "n"(L + 4), "n"(L + 5),
              "n"(L + 6), "n"(L + 7));
        if constexpr (CNT > 8) fmac_dot<L + 8, CNT - 8>(a + 8, x, s0, s1);
    } else if constexpr (CNT >= 4) {
        asm("s_nop 1\n\t" LBM_FMAC_DPP(0, 2, 3, 7) LBM_FMAC_DPP(1, 2, 4, 8)
                LBM_FMAC_DPP(0, 2, 5, 9) LBM_FMAC_DPP(1, 2, 6, 10)
            : "+&v"(s0), "+&v"(s1)
            : "v"(x), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "n"(L), "n"(L + 1), "n"(L + 2),
              "n"(L + 3));
        if constexpr (CNT > 4) fmac_dot<L + 4, CNT - 4>(a + 4, x, s0, s1);
    } else if constexpr (CNT >= 2) {
        asm("s_nop 1\n\t" LBM_FMAC_DPP(0, 2, 3, 5) LBM_FMAC_DPP(1, 2, 4, 6)
            : "+&v"(s0), "+&v"(s1)
            : "v"(x), "v"(a[0]), "v"(a[1]), "n"(L), "n"(L + 1));
        if constexpr (CNT > 2) fmac_dot<L + 2, CNT - 2>(a + 2, x, s0, s1);
    } else if constexpr (CNT == 1) {
        asm("s_nop 1\n\t" LBM_FMAC_DPP(0, 1, 2, 3) : "+&v"(s0) : "v"(x), "v"(a[0]), "n"(L));
    }
}

// The same over columns 0 .. W - 1 of a vector kept as NS registers per lane.
template <int W, int NS>
__device__ __forceinline__ void row_axpy(double* a, const double (&x)[NS], double y) {
    fmac_axpy<0, (W < 16 ? W : 16)>(a, x[0], y);
    if constexpr (W > 16) fmac_axpy<0, W - 16>(a + 16, x[1], y);
}
template <int W, int NS>
__device__ __forceinline__ double row_dot(const double* a, const double (&x)[NS]) {
    double s0 = 0.0, s1 = 0.0;
    fmac_dot<0, (W < 16 ? W : 16)>(a, x[0], s0, s1);
    if constexpr (W > 16) fmac_dot<0, W - 16>(a + 16, x[1], s0, s1);
    return s0 + s1;
}

// Two chains of the tridiagonal inverse's recurrence at once: for k < CNT
//   ua[k] += bcast(g[k], P) * (k ? ua[k - 1] : pa),  ub[k] likewise with lane P + 1.
template <int P, int CNT>
__device__ __forceinline__ void fmac_chain(double* ua, double* ub, const double* g, double pa,
                                           double pb) {
    if constexpr (CNT >= 4) {
        asm("s_nop 1\n\t" LBM_FMAC_DPP(0, 8, 12, 14) LBM_FMAC_DPP(4, 8, 13, 15)
                LBM_FMAC_DPP(1, 9, 0, 14) LBM_FMAC_DPP(5, 9, 4, 15) LBM_FMAC_DPP(2, 10, 1, 14)
                    LBM_FMAC_DPP(6, 10, 5, 15) LBM_FMAC_DPP(3, 11, 2, 14)
                        LBM_FMAC_DPP(7, 11, 6, 15)
            : "+&v"(ua[0]), "+&v"(ua[1]), "+&v"(ua[2]), "+&v"(ua[3]), "+&v"(ub[0]), "+&v"(ub[1]),
              "+&v"(ub[2]), "+&v"(ub[3])
            : "v"(g[0]), "v"(g[1]), "v"(g[2]), "v"(g[3]), "v"(pa), "v"(pb), "n"(P), "n"(P + 1));
        if constexpr (CNT > 4) fmac_chain<P, CNT - 4>(ua + 4, ub + 4, g + 4, ua[3], ub[3]);
    } else if constexpr (CNT >= 2) {
        asm("s_nop 1\n\t" LBM_FMAC_DPP(0, 4, 6, 8) LBM_FMAC_DPP(2, 4, 7, 9)
                LBM_FMAC_DPP(1, 5, 0, 8) LBM_FMAC_DPP(3, 5, 2, 9)
            : "+&v"(ua[0]), "+&v"(ua[1]), "+&v"(ub[0]), "+&v"(ub[1])
            : "v"(g[0]), "v"(g[1]), "v"(pa), "v"(pb), "n"(P), "n"(P + 1));
        if constexpr (CNT > 2) fmac_chain<P, CNT - 2>(ua + 2, ub + 2, g + 2, ua[1], ub[1]);
    } else if constexpr (CNT == 1) {
        asm("s_nop 1\n\t" LBM_FMAC_DPP(0, 2, 3, 5) LBM_FMAC_DPP(1, 2, 4, 6)
            : "+&v"(ua[0]), "+&v"(ub[0])
            : "v"(g[0]), "v"(pa), "v"(pb), "n"(P), "n"(P + 1));
    }
}
#undef LBM_FMAC_DPP

__device__ __forceinline__ double row_sum(double v) { return group_sum16(v); }

// x^{-1/2} and 1 / x of normal positive x: the hardware estimate and one cubic
// correction step (y (1 + e/2 + 3 e^2/8), e = 1 - x y^2; y (1 + e + e^2), e = 1 - x y).
__device__ __forceinline__ double fast_rsqrt(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}
__device__ __forceinline__ double fast_rcp(double x) {
    const double y = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, y, 1.0);
    return fma(y, fma(e, e, e), y);
}

template <int N>
struct Direct {
    static_assert(N >= 4 && N <= 32 && N % 2 == 0, "one or two matrix rows per lane");
    static constexpr int NS = (N + 15) / 16;      // matrix rows per lane
    static constexpr int ZS = N + 1;              // stride of the LDS tables (odd)
    static constexpr int kNodeDoubles = 16 * ZS;  // per node: pole table, then the transposes
    static constexpr int kTop = (N - 1 + 3) / 4 * 4;  // first phase's width
    // the pole recurrence's values between its two passes: in registers up to N = 20,
    // beyond that in the LDS table (registers would spill)
    static constexpr bool kValLds = N > 20;
};

// Where the reflectors wait for the back transformation: a device-memory scratch with
// row n - 3 for step n (written and read by the same lanes), or LDS, step n's n - 1
// entries packed.
struct ReflGlobal {
    double* p;
    int stride;
    bool on;  // false: a lane group without a node stores nothing
    __device__ __forceinline__ void put(int n, int i, double v) const {
        if (on && i < stride) p[(size_t)(n - 3) * stride + i] = v;
    }
    __device__ __forceinline__ double get(int n, int i) const {
        return i < stride ? p[(size_t)(n - 3) * stride + i] : 0.0;
    }
};
struct ReflLds {
    double* p;
    __host__ __device__ static constexpr int doubles(int n) { return n * (n - 1) / 2; }
    __device__ __forceinline__ void put(int n, int i, double v) const {
        if (i < n - 1) p[(n - 2) * (n - 1) / 2 + i] = v;
    }
    __device__ __forceinline__ double get(int n, int i) const {
        return i < n - 1 ? p[(n - 2) * (n - 1) / 2 + i] : 0.0;
    }
};

// One phase of the tridiagonalisation: the columns n - 1 for n = min(N, W + 1) down to
// max(3, W - 2) are eliminated on rows and columns < W (n - 1 <= W).  The reflector of
// step n, H = I - v v^T on indices 0 .. n - 2 (|v|^2 = 2, or v = 0), goes to
// `vs`; d and e receive the diagonal and the coupling (i, i + 1); b
// becomes H b.  Widths in steps of four keep the code small (each phase is a loop)
// at the price of a few columns that are no longer needed.
template <int N, int W, typename R>
__device__ __forceinline__ void tri_phase(double (&A)[Direct<N>::NS][N],
                                          double (&d)[Direct<N>::NS], double (&e)[Direct<N>::NS],
                                          double (&b)[Direct<N>::NS], const R& vs, int lane) {
    constexpr int NS = Direct<N>::NS;
    constexpr int WC = W < N ? W : N;              // columns and rows of the support
    constexpr int SW = (WC + 15) / 16;             // row slots of the support
    constexpr int SX = W / 16 + 1 < NS ? W / 16 + 1 : NS;  // slots that hold a row n - 1
    constexpr int HI = W + 1 < N ? W + 1 : N;
    constexpr int LO = W - 2 > 3 ? W - 2 : 3;
    const int r = lane & 15;
#pragma unroll 1
    for (int n = HI; n >= LO; --n) {
        double x[SW], v[SW], p[SW];
#pragma unroll
        for (int h = 0; h < SX; ++h) {
            // column n - 1: a sum over the phase's columns with weights 1 and 0 (a select
            // would index the registers dynamically, through scratch memory); columns
            // beyond n - 1 hold finite values, H S H continued to all rows
            double xr = A[h][LO - 1] * (n == LO ? 1.0 : 0.0);
#pragma unroll
            for (int c = LO; c < HI; ++c) xr = fma(A[h][c], n - 1 == c ? 1.0 : 0.0, xr);
            d[h] = r + 16 * h == n - 1 ? xr : d[h];
            if (h < SW) x[h < SW ? h : 0] = r + 16 * h < n - 1 ? xr : 0.0;
        }
        double s2 = x[0] * x[0];
        if constexpr (SW > 1) s2 = fma(x[1], x[1], s2);
        constexpr int PS = (W - 1) / 16 < SW ? (W - 1) / 16 : SW - 1;  // slot of row n - 2
        const double x1 = row_bcast_dyn(x[PS], (n - 2) & 15, lane);
        s2 = row_sum(s2);
        const bool some = s2 > 1e-290;
        const double norm = s2 * fast_rsqrt(s2);
        const double rb = some ? fast_rsqrt(fma(fabs(x1), norm, s2)) : 0.0;
        const double alpha = some ? -copysign(norm, x1) : x1;
        const double shift = some ? copysign(norm, x1) : 0.0;
#pragma unroll
        for (int h = 0; h < SW; ++h) {
            const bool piv = r + 16 * h == n - 2;
            e[h] = piv ? alpha : e[h];
            v[h] = (x[h] + (piv ? shift : 0.0)) * rb;
            vs.put(n, r + 16 * h, v[h]);
        }
        double c = 0.0, cb = 0.0;
#pragma unroll
        for (int h = 0; h < SW; ++h) {
            p[h] = row_dot<WC, SW>(A[h], v);
            c = fma(v[h], p[h], c);
            cb = fma(v[h], b[h], cb);
        }
        c = row_sum(c);
        cb = row_sum(cb);
#pragma unroll
        for (int h = 0; h < SW; ++h) {
            const double w = fma(-c, v[h], p[h]);
            b[h] = fma(-cb, v[h], b[h]);
            row_axpy<WC, SW>(A[h], p, -v[h]);
            row_axpy<WC, SW>(A[h], v, -w);
        }
    }
}

// The reflectors of one phase applied from both sides, G <- H G H, in ascending n, and
// hv <- H hv.
template <int N, int W, typename R>
__device__ __forceinline__ void back_phase(double (&G)[Direct<N>::NS][N],
                                           double (&hv)[Direct<N>::NS], const R& vs, int lane) {
    constexpr int NS = Direct<N>::NS;
    constexpr int WC = W < N ? W : N;
    constexpr int SW = (WC + 15) / 16;
    constexpr int HI = W + 1 < N ? W + 1 : N;
    constexpr int LO = W - 2 > 3 ? W - 2 : 3;
    const int r = lane & 15;
#pragma unroll 1
    for (int n = LO; n <= HI; ++n) {
        double v[SW], p[NS];
#pragma unroll
        for (int h = 0; h < SW; ++h) v[h] = vs.get(n, r + 16 * h);
        double c = 0.0, ch = 0.0;
#pragma unroll
        for (int h = 0; h < NS; ++h) {
            p[h] = row_dot<WC, SW>(G[h], v);
            if (h < SW) {
                c = fma(v[h < SW ? h : 0], p[h], c);
                ch = fma(v[h < SW ? h : 0], hv[h], ch);
            }
        }
        c = row_sum(c);
        ch = row_sum(ch);
#pragma unroll
        for (int h = 0; h < NS; ++h) {
            if (h < SW) {
                const double vh = v[h < SW ? h : 0];
                hv[h] = fma(-ch, vh, hv[h]);
                row_axpy<N, NS>(G[h], p, -vh);
                row_axpy<WC, SW>(G[h], v, -fma(-c, vh, p[h]));
            } else {
                row_axpy<WC, SW>(G[h], v, -p[h]);
            }
        }
    }
}

template <int N, int W, typename R>
__device__ __forceinline__ void tri_all(double (&A)[Direct<N>::NS][N], double (&d)[Direct<N>::NS],
                                        double (&e)[Direct<N>::NS], double (&b)[Direct<N>::NS],
                                        const R& vs, int lane) {
    tri_phase<N, W>(A, d, e, b, vs, lane);
    if constexpr (W > 4) tri_all<N, W - 4>(A, d, e, b, vs, lane);
}
template <int N, int W, typename R>
__device__ __forceinline__ void back_all(double (&G)[Direct<N>::NS][N], double (&hv)[Direct<N>::NS],
                                         const R& vs, int lane) {
    if constexpr (W > 4) back_all<N, W - 4>(G, hv, vs, lane);
    back_phase<N, W>(G, hv, vs, lane);
}

// Sum over each row of 16 lanes (FP32).
__device__ __forceinline__ float row_sum_f32(float m) {
    m += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(m), 0xB1, 0xF, 0xF, true));
    m += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(m), 0x4E, 0xF, 0xF, true));
    m += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(m), 0x141, 0xF, 0xF, true));
    m += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(m), 0x140, 0xF, 0xF, true));
    return m;
}

// Adds two poles' entries of one row of the tridiagonal inverse, columns J.. of the
// slot that starts at column H: z_ii (wa, wb) on the diagonal, then z_{i,j+1} = g_j z_{i,j};
// four columns at a time (pa, pb: the column before).
template <int N, int H, int J>
__device__ __forceinline__ void row_chain(double (&a)[N], const double (&g)[N], double wa, double wb,
                                          double pa, double pb, int pr, int r) {
    constexpr int C = N - J < 4 ? N - J : 4;
    constexpr int F = J == H ? 1 : 0;  // the slot's first column has no predecessor
    double ua[4] = {0.0, 0.0, 0.0, 0.0}, ub[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < C; ++k) {
        const bool own = J + k < H + 16 && r == J + k - H;
        ua[k] = own ? wa : 0.0;
        ub[k] = own ? wb : 0.0;
    }
    if (pr == 0)
        fmac_chain<0, C - F>(ua + F, ub + F, g + (F ? J : J - 1), F ? ua[0] : pa, F ? ub[0] : pb);
    else
        fmac_chain<2, C - F>(ua + F, ub + F, g + (F ? J : J - 1), F ? ua[0] : pa, F ? ub[0] : pb);
#pragma unroll
    for (int k = 0; k < C; ++k) a[J + k] += ua[k] + ub[k];
    if constexpr (J + C < N)
        row_chain<N, H, J + C>(a, g, wa, wb, ua[C - 1], ub[C - 1], pr, r);
}

// Pole class of a wavefront: kappa = 1 + the largest norm of its four nodes (WAVE: of
// its one node), norm^2 given as a sum over the node's lanes; a NaN does not count.
template <bool WAVE>
__device__ __forceinline__ int pole_class(float part) {
    const float n2 = row_sum_f32(part);
    float w = 0.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float row = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(n2), 16 * k));
        w = WAVE ? w + row : fmaxf(w, row);
    }
    if (!(w >= 0.0f)) w = 0.0f;
    // kappa <= 2^e: the exponent of 1 + norm (a little enlarged against FP32 rounding),
    // rounded up
    const float kappa = 1.0f + 1.0001f * __builtin_amdgcn_sqrtf(w);
    const int e = ((__float_as_int(kappa) + 0x7fffff) >> 23) - 127;
    int k = 0;
    while (k < kPoleClasses - 1 && kPoleLog2[k] < e) ++k;
    return __builtin_amdgcn_readfirstlane(k);
}

// For the four nodes of a wavefront, with X = I + S/a (rows of S in A, S >= 0):
//   A <- scale * F(X)   (scale * X^{-1/2} if ROOT),   b <- X^{-1} b.
// lds: 4 * Direct<N>::kNodeDoubles doubles; vs: this node's reflector store.  Returns
// false if a node's matrix is not finite.
template <int N, bool ROOT, typename R>
__device__ __forceinline__ bool sym_direct(double (&A)[Direct<N>::NS][N],
                                           double (&b)[Direct<N>::NS], double ia, double scale,
                                           double* lds, const R& vs, int lane) {
    using D = Direct<N>;
    constexpr int NS = D::NS;
    constexpr int ZS = D::ZS;
    const int r = lane & 15;
    double* zt = lds + (size_t)(lane >> 4) * D::kNodeDoubles;  // [16][ZS]
    double d[NS], e[NS];
#pragma unroll
    for (int h = 0; h < NS; ++h) d[h] = e[h] = 0.0;
    tri_all<N, D::kTop>(A, d, e, b, vs, lane);
    // rows 0 and 1 are left: d_0, d_1, e_0
    d[0] = r == 0 ? A[0][0] : (r == 1 ? A[0][1] : d[0]);
    e[0] = r == 0 ? A[0][1] : e[0];
    // the Frobenius norm of T / a bounds its largest eigenvalue
    bool finite = true;
    float f2 = 0.0f;
#pragma unroll
    for (int h = 0; h < NS; ++h) {
        d[h] *= ia;
        e[h] *= ia;
        finite = finite && fabs(d[h]) + fabs(e[h]) < 1e300;
        const float df = (float)d[h], ef = (float)e[h];
        f2 += df * df + 2.0f * ef * ef;
    }
    const int cls = pole_class<false>(f2);
    const int p0 = kPoleOffset[cls], np = kPoleOffset[cls + 1] - p0;

#pragma unroll
    for (int h = 0; h < NS; ++h)
#pragma unroll
        for (int j = 0; j < N; ++j) A[h][j] = 0.0;
    double hv[NS];
    // fifteen poles at a time, lane r = pole (lane 15: t^2 = 0, the inverse itself):
    // X + t^2 = U Gamma U^T from the bottom row up, then its inverse's diagonal from
    // the top row down (both recurrences have positive terms only)
#pragma unroll 1
    for (int pb = 0; pb < np; pb += 15) {
        const int pi = pb + r < np && r < 15 ? p0 + pb + r : -1;
        const double t2 = pi >= 0 ? kSqrtPoles[pi < 0 ? 0 : pi].t2 : 0.0;
        double cw = pi >= 0 ? kSqrtPoles[pi < 0 ? 0 : pi].c * scale : 0.0;
        if constexpr (ROOT) cw *= 1.0 + t2;
        const double base = 1.0 + t2;
        // val_j = 1 / gamma_j, and on lane 15 y_j / gamma_j with U y = b: the same downward
        // recurrence then gives z_jj on lanes 0..14 and the solution of X h = b on lane 15
        const bool inv = r == 15;
        double g[N], val[N];
        double rg = 0.0, y = 0.0;
        auto col = [](const double (&v)[NS], auto J) {
            constexpr int j = decltype(J)::value;
            return row_bcast<j % 16>(v[j / 16]);
        };
        auto down = [&](auto self, auto J) -> void {
            constexpr int j = decltype(J)::value;
            double gam = base + col(d, J);
            if constexpr (j == N - 1) {
                g[j] = 0.0;
                y = col(b, J);
            } else {
                const double ej = col(e, J);
                g[j] = -ej * rg;
                gam = fma(g[j], ej, gam);
                y = fma(g[j], y, col(b, J));
            }
            rg = fast_rcp(gam);
            const double v = inv ? y * rg : rg;
            if constexpr (D::kValLds) zt[r * ZS + j] = v;
            else val[j] = v;
            if constexpr (j > 0) self(self, std::integral_constant<int, j - 1>());
        };
        down(down, std::integral_constant<int, N - 1>());
        if constexpr (!D::kValLds) wave_lds_sync();
        {
            const double cx = inv ? 1.0 : cw;
            double z = 0.0;
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const double v = D::kValLds ? zt[r * ZS + j] : val[j];
                const double m = j == 0 ? 0.0 : (inv ? g[j - 1] : g[j - 1] * g[j - 1]);
                z = fma(m, z, v);
                zt[r * ZS + j] = z * cx;
            }
        }
        wave_lds_sync();
#pragma unroll
        for (int h = 0; h < NS; ++h) hv[h] = r + 16 * h < N ? zt[15 * ZS + r + 16 * h] : 0.0;
        // upper triangle, row i: z_ii, then z_{i,j+1} = g_j z_{i,j}; four poles per pass,
        // after which the rows' lanes rotate by four
        const int left = np - pb < 15 ? np - pb : 15;
#pragma unroll 1
        for (int q = 0; q < left; q += 4) {
#pragma unroll
            for (int pr = 0; pr < 4; pr += 2) {
                double wa[NS], wb[NS];
#pragma unroll
                for (int h = 0; h < NS; ++h) {
                    const int i = r + 16 * h < N ? r + 16 * h : 0;
                    wa[h] = zt[(q + pr) * ZS + i];
                    wb[h] = zt[(q + pr + 1) * ZS + i];
                    if (q + pr + 1 == 15) wb[h] = 0.0;
                }
                row_chain<N, 0, 0>(A[0], g, wa[0], wb[0], 0.0, 0.0, pr, r);
                if constexpr (NS > 1)
                    row_chain<N, 16, 16>(A[NS - 1], g, wa[NS - 1], wb[NS - 1], 0.0, 0.0, pr, r);
            }
#pragma unroll
            for (int j = 0; j < N - 1; ++j) {
                const int lo = __builtin_amdgcn_mov_dpp(__double2loint(g[j]), 0x12C, 0xF, 0xF, true);
                const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(g[j]), 0x12C, 0xF, 0xF, true);
                g[j] = __hiloint2double(hi, lo);
            }
        }
        wave_lds_sync();
    }
    // lower triangle: the lower rows' columns come from rows 0..15 (one transpose), the
    // rest of rows 16.. from themselves (a second)
#pragma unroll
    for (int j = 0; j < N; ++j) zt[r * ZS + j] = A[0][j];
    if (r < N) zt[r * ZS + r] = 0.0;
    wave_lds_sync();
#pragma unroll
    for (int j = 0; j < (N < 16 ? N : 16); ++j)
#pragma unroll
        for (int h = 0; h < NS; ++h) {
            const double t = zt[j * ZS + (r + 16 * h < N ? r + 16 * h : 0)];
            A[h][j] += r + 16 * h < N ? t : 0.0;
        }
    if constexpr (NS > 1) {
        wave_lds_sync();
        if (r + 16 < N) {
#pragma unroll
            for (int j = 16; j < N; ++j) zt[r * ZS + j] = A[1][j];
            zt[r * ZS + r + 16] = 0.0;
        }
        wave_lds_sync();
#pragma unroll
        for (int j = 16; j < N; ++j) {
            const double t = zt[(j - 16) * ZS + (r + 16 < N ? r + 16 : 0)];
            A[1][j] += r + 16 < N ? t : 0.0;
        }
    }
#pragma unroll
    for (int h = 0; h < NS; ++h) b[h] = hv[h];
    back_all<N, D::kTop>(A, b, vs, lane);
    return finite;
}

// ---------------------------------------------------------------------------
// two nodes per wavefront, 32 < N <= 48
// ---------------------------------------------------------------------------
// A node owns two rows of 16 lanes.  Lane (q, r) of it (q = 0, 1) holds rows r, r + 16 and
// r + 32 and of them half the columns: of each 16 columns the 8 of index 8 q .. 8 q + 7 (of
// the last 8, N = 40, four), in all N / 2 a row: 120 or 144 registers where whole rows would
// need 240 or 288.  A vector is kept by rows in both lane rows; as broadcast operand the second
// lane row takes it rotated by those 8 (or 4) lanes, so that one row_newbcast serves both.  Only
// the products' partial sums cross the lane rows (v_permlane16_swap).  Against one node per
// wavefront (below) this leaves 2.4 times fewer instructions a node: no vector goes through
// LDS, and a step's reductions and square roots serve two nodes.
template <int N>
struct DirectP {
    static_assert(N == 40 || N == 48, "the last rows' 8 or 16 columns split evenly");
    static constexpr int NS = 3;
    static constexpr int COLS = N / 2;
    static constexpr int ZS = N + 1;
    static constexpr int kPoles = 11;             // a pass; lane 11: the solution
    static constexpr int kNodeDoubles = 24 * ZS;  // tables z, e of 12 lanes; then the transposes
    static constexpr int width(int h) { return h < 2 ? 8 : N / 2 - 16; }
    // the element of column c (0 .. COLS - 1) in lane row q
    static constexpr int elem(int c, int q) {
        return 16 * (c / 8) + width(c / 8) * q + c % 8;
    }
};

// The sum over a node's two lane rows, in both.
__device__ __forceinline__ double pair_sum(double x) {
    const unsigned lo = __double2loint(x), hi = __double2hiint(x);
    const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __hiloint2double(b[0], a[0]) + __hiloint2double(b[1], a[1]);
}

// A vector by rows as broadcast operand, slots 0 .. S.
template <int N, int S>
__device__ __forceinline__ void pair_operand(const double* x, double (&out)[3], int q) {
#pragma unroll
    for (int h = 0; h <= S; ++h) {
        int lo, hi;
        if (DirectP<N>::width(h) == 8) {
            lo = __builtin_amdgcn_mov_dpp(__double2loint(x[h]), 0x128, 0xF, 0xF, true);
            hi = __builtin_amdgcn_mov_dpp(__double2hiint(x[h]), 0x128, 0xF, 0xF, true);
        } else {
            lo = __builtin_amdgcn_mov_dpp(__double2loint(x[h]), 0x12C, 0xF, 0xF, true);
            hi = __builtin_amdgcn_mov_dpp(__double2hiint(x[h]), 0x12C, 0xF, 0xF, true);
        }
        out[h] = q ? __hiloint2double(hi, lo) : x[h];
    }
}

// a += x y and a . x over the columns of slots 0 .. S.
template <int N, int S>
__device__ __forceinline__ void pair_axpy(double* a, const double (&x)[3], double y) {
    fmac_axpy<0, 8>(a, x[0], y);
    if constexpr (S > 0) fmac_axpy<0, 8>(a + 8, x[1], y);
    if constexpr (S > 1) fmac_axpy<0, DirectP<N>::width(2)>(a + 16, x[2], y);
}
template <int N, int S>
__device__ __forceinline__ double pair_dot(const double* a, const double (&x)[3]) {
    double s0 = 0.0, s1 = 0.0;
    fmac_dot<0, 8>(a, x[0], s0, s1);
    if constexpr (S > 0) fmac_dot<0, 8>(a + 8, x[1], s0, s1);
    if constexpr (S > 1) fmac_dot<0, DirectP<N>::width(2)>(a + 16, x[2], s0, s1);
    return pair_sum(s0 + s1);
}

// tri_phase for the pivot columns n - 1 of slot S that lane row Q holds.
template <int N, int S, int Q, typename R>
__device__ __forceinline__ void pair_tri_phase(double (&A)[3][DirectP<N>::COLS], double (&d)[3],
                                               double (&e)[3], double (&b)[3], const R& vs,
                                               int lane) {
    constexpr int W = DirectP<N>::width(S);
    constexpr int BASE = 16 * S + W * Q;
    const int r = lane & 15, q = lane >> 4 & 1;
#pragma unroll 1
    for (int n = BASE + W; n > (BASE > 2 ? BASE : 2); --n) {
        double x[3] = {0.0, 0.0, 0.0}, v[3] = {0.0, 0.0, 0.0}, p[3] = {0.0, 0.0, 0.0};
        double xr[3] = {0.0, 0.0, 0.0};
        // column n - 1 (weights 1 and 0, as in tri_phase), from its lane row to both
#pragma unroll
        for (int c = 0; c < W; ++c) {
            const double w = q == Q && n - 1 == BASE + c ? 1.0 : 0.0;
#pragma unroll
            for (int h = 0; h <= S; ++h) xr[h] = fma(A[h][8 * S + c], w, xr[h]);
        }
        double s2 = 0.0;
#pragma unroll
        for (int h = 0; h <= S; ++h) {
            const double t = pair_sum(xr[h]);
            d[h] = r + 16 * h == n - 1 ? t : d[h];
            x[h] = r + 16 * h < n - 1 ? t : 0.0;
            s2 = fma(x[h], x[h], s2);
        }
        const double xp = S > 0 && n - 2 < 16 * S ? x[S > 0 ? S - 1 : 0] : x[S];
        const double x1 = row_bcast_dyn(xp, (n - 2) & 15, lane);
        s2 = row_sum(s2);
        const bool some = s2 > 1e-290;
        const double norm = s2 * fast_rsqrt(s2);
        const double rb = some ? fast_rsqrt(fma(fabs(x1), norm, s2)) : 0.0;
        const double alpha = some ? -copysign(norm, x1) : x1;
        const double shift = some ? copysign(norm, x1) : 0.0;
#pragma unroll
        for (int h = 0; h <= S; ++h) {
            const bool piv = r + 16 * h == n - 2;
            e[h] = piv ? alpha : e[h];
            v[h] = (x[h] + (piv ? shift : 0.0)) * rb;
            vs.put(n, r + 16 * h, v[h]);
        }
        double vq[3], pq[3];
        pair_operand<N, S>(v, vq, q);
        double c = 0.0, cb = 0.0;
#pragma unroll
        for (int h = 0; h <= S; ++h) {
            p[h] = pair_dot<N, S>(A[h], vq);
            c = fma(v[h], p[h], c);
            cb = fma(v[h], b[h], cb);
        }
        c = row_sum(c);
        cb = row_sum(cb);
        pair_operand<N, S>(p, pq, q);
#pragma unroll
        for (int h = 0; h <= S; ++h) {
            const double w = fma(-c, v[h], p[h]);
            b[h] = fma(-cb, v[h], b[h]);
            pair_axpy<N, S>(A[h], pq, -v[h]);
            pair_axpy<N, S>(A[h], vq, -w);
        }
    }
}

// back_phase for the reflectors of the pivot columns in slot S.
template <int N, int S, typename R>
__device__ __forceinline__ void pair_back_phase(double (&G)[3][DirectP<N>::COLS], double (&hv)[3],
                                                const R& vs, int lane) {
    const int r = lane & 15, q = lane >> 4 & 1;
    constexpr int HI = 16 * S + 16 < N ? 16 * S + 16 : N;
#pragma unroll 1
    for (int n = S > 0 ? 16 * S + 1 : 3; n <= HI; ++n) {
        double v[3] = {0.0, 0.0, 0.0}, p[3], vq[3], pq[3];
#pragma unroll
        for (int h = 0; h <= S; ++h) v[h] = vs.get(n, r + 16 * h);
        pair_operand<N, S>(v, vq, q);
        double c = 0.0, ch = 0.0;
#pragma unroll
        for (int h = 0; h < 3; ++h) {
            p[h] = pair_dot<N, S>(G[h], vq);
            if (h <= S) {
                c = fma(v[h], p[h], c);
                ch = fma(v[h], hv[h], ch);
            }
        }
        c = row_sum(c);
        ch = row_sum(ch);
        pair_operand<N, 2>(p, pq, q);
#pragma unroll
        for (int h = 0; h < 3; ++h) {
            if (h <= S) {
                hv[h] = fma(-ch, v[h], hv[h]);
                pair_axpy<N, 2>(G[h], pq, -v[h]);
                pair_axpy<N, S>(G[h], vq, -fma(-c, v[h], p[h]));
            } else {
                pair_axpy<N, S>(G[h], vq, -p[h]);
            }
        }
    }
}

// Two poles' entries of the columns of slot HC for a row of slot H: sa, sb the row's values at
// the column before them, own: this lane's diagonal column in the slot, if any.
template <int W, int K>
__device__ __forceinline__ void pair_chain(double* a, const double* g, double wa, double wb,
                                           double& pa, double& pb, int pr, int own) {
    double ua[4], ub[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const bool o = own == K + k;
        ua[k] = o ? wa : 0.0;
        ub[k] = o ? wb : 0.0;
    }
    if (pr == 0) fmac_chain<0, 4>(ua, ub, g + K, pa, pb);
    else fmac_chain<2, 4>(ua, ub, g + K, pa, pb);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        a[K + k] += ua[k] + ub[k];
        // summed here (see wave_chain)
        asm volatile("" : "+v"(a[K + k]));
    }
    pa = ua[3];
    pb = ub[3];
    if constexpr (K + 4 < W) pair_chain<W, K + 4>(a, g, wa, wb, pa, pb, pr, own);
}

// The same in the slots after the row's own.
template <int W, int K>
__device__ __forceinline__ void pair_chain_on(double* a, const double* g, double& pa, double& pb,
                                              int pr) {
    double ua[4] = {0.0, 0.0, 0.0, 0.0}, ub[4] = {0.0, 0.0, 0.0, 0.0};
    if (pr == 0) fmac_chain<0, 4>(ua, ub, g + K, pa, pb);
    else fmac_chain<2, 4>(ua, ub, g + K, pa, pb);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        a[K + k] += ua[k] + ub[k];
        asm volatile("" : "+v"(a[K + k]));
    }
    pa = ua[3];
    pb = ub[3];
    if constexpr (K + 4 < W) pair_chain_on<W, K + 4>(a, g, pa, pb, pr);
}

// ta += bcast(P, pr) sa, tb += bcast(P, pr + 1) sb
__device__ __forceinline__ void pair_scale(double& ta, double& tb, double P, double sa, double sb,
                                           int pr) {
    if (pr == 0) {
        fmac_axpy<0, 1>(&ta, P, sa);
        fmac_axpy<1, 1>(&tb, P, sb);
    } else {
        fmac_axpy<2, 1>(&ta, P, sa);
        fmac_axpy<3, 1>(&tb, P, sb);
    }
}

// sym_direct for the two nodes of a wavefront (A: half rows as above; b by rows, in both
// lane rows).  lds: 2 * DirectP<N>::kNodeDoubles doubles.
template <int N, bool ROOT, typename R>
__device__ __forceinline__ bool sym_direct_pair(double (&A)[3][DirectP<N>::COLS], double (&b)[3],
                                                double ia, double scale, double* lds, const R& vs,
                                                int lane) {
    using D = DirectP<N>;
    constexpr int ZS = D::ZS;
    const int r = lane & 15, q = lane >> 4 & 1;
    double* zt = lds + (size_t)(lane >> 5) * D::kNodeDoubles;  // [12][ZS]
    double* et = zt + 12 * ZS;
    double d[3] = {0.0, 0.0, 0.0}, e[3] = {0.0, 0.0, 0.0};
    pair_tri_phase<N, 2, 1>(A, d, e, b, vs, lane);
    pair_tri_phase<N, 2, 0>(A, d, e, b, vs, lane);
    pair_tri_phase<N, 1, 1>(A, d, e, b, vs, lane);
    pair_tri_phase<N, 1, 0>(A, d, e, b, vs, lane);
    pair_tri_phase<N, 0, 1>(A, d, e, b, vs, lane);
    pair_tri_phase<N, 0, 0>(A, d, e, b, vs, lane);
    {
        // rows 0 and 1 are left: d_0, d_1, e_0
        const double t0 = pair_sum(q == 0 ? (r == 0 ? A[0][0] : A[0][1]) : 0.0);
        const double t1 = pair_sum(q == 0 ? A[0][1] : 0.0);
        d[0] = r < 2 ? t0 : d[0];
        e[0] = r == 0 ? t1 : e[0];
    }
    bool finite = true;
    float f2 = 0.0f;
#pragma unroll
    for (int h = 0; h < 3; ++h) {
        d[h] *= ia;
        e[h] *= ia;
        finite = finite && fabs(d[h]) + fabs(e[h]) < 1e300;
        const float df = (float)d[h], ef = (float)e[h];
        f2 += df * df + 2.0f * ef * ef;
    }
    const int cls = pole_class<false>(f2);
    const int p0 = kPoleOffset[cls], np = kPoleOffset[cls + 1] - p0;
#pragma unroll
    for (int h = 0; h < 3; ++h)
#pragma unroll
        for (int c = 0; c < D::COLS; ++c) A[h][c] = 0.0;
    double hv[3] = {0.0, 0.0, 0.0};
#pragma unroll 1
    for (int pb = 0; pb < np; pb += D::kPoles) {
        const int pi = pb + r < np && r < D::kPoles ? p0 + pb + r : -1;
        const double t2 = pi >= 0 ? kSqrtPoles[pi < 0 ? 0 : pi].t2 : 0.0;
        double cw = pi >= 0 ? kSqrtPoles[pi < 0 ? 0 : pi].c * scale : 0.0;
        if constexpr (ROOT) cw *= 1.0 + t2;
        const double base = 1.0 + t2;
        const bool inv = r == D::kPoles;
        const bool keep = q == 0 && r <= D::kPoles;  // (both lane rows compute the same)
        double rg = 0.0, y = 0.0;
        // as in sym_direct: val_j = 1 / gamma_j (z table), g_j (e table), downwards
        auto down = [&](auto self, auto J) -> void {
            constexpr int j = decltype(J)::value;
            const double dj = row_bcast<j % 16>(d[j / 16]), bj = row_bcast<j % 16>(b[j / 16]);
            double gam = base + dj, gj = 0.0;
            if constexpr (j == N - 1) {
                y = bj;
            } else {
                const double ej = row_bcast<j % 16>(e[j / 16]);
                gj = -ej * rg;
                gam = fma(gj, ej, gam);
                y = fma(gj, y, bj);
            }
            rg = fast_rcp(gam);
            if (keep) {
                zt[r * ZS + j] = inv ? y * rg : rg;
                et[r * ZS + j] = gj;
            }
            if constexpr (j % 8 == 0) __builtin_amdgcn_sched_barrier(0);
            if constexpr (j > 0) self(self, std::integral_constant<int, j - 1>());
        };
        down(down, std::integral_constant<int, N - 1>());
        wave_lds_sync();
        const int row = (r <= D::kPoles ? r : 0) * ZS;
        {
            const double cx = inv ? 1.0 : cw;
            double z = 0.0, m = 0.0;
#pragma unroll 8
            for (int j = 0; j < N; ++j) {
                const double gj = et[row + j];
                z = fma(m, z, zt[row + j]);
                if (keep) zt[row + j] = z * cx;
                m = inv ? gj : gj * gj;
            }
        }
        wave_lds_sync();
        // upwards again: the factors into this lane row's columns, the value of each row at
        // the end of its own block of columns (e table), the products over the blocks between
        // two of this lane row's
        double gc[D::COLS], P[2] = {0.0, 0.0};
        {
            double sp = 1.0;  // product of the factors from column j to its block's end
            auto up = [&](auto self, auto J) -> void {
                constexpr int j = decltype(J)::value;
                constexpr int w = D::width(j / 16);
                constexpr bool last = j % 16 % w == w - 1;
                const double gj = et[row + j];  // the factor into column j + 1
                if constexpr (j + 1 < N) {
                    constexpr int h1 = (j + 1) / 16, w1 = D::width(h1), q1 = (j + 1) % 16 / w1;
                    constexpr int c1 = 8 * h1 + (j + 1) % 16 % w1;
                    if constexpr (q1 == 1) gc[c1] = gj;
                    else gc[c1] = q ? gc[c1] : gj;
                }
                // the block after this one ends its product at j = its first column - 1
                if constexpr (last && j + 1 < N) {
                    constexpr int blk = 2 * ((j + 1) / 16) + (j + 1) % 16 / D::width((j + 1) / 16);
                    const double prod = gj * sp;
                    if constexpr (blk == 1) P[0] = q ? P[0] : prod;
                    if constexpr (blk == 2) P[0] = q ? prod : P[0];
                    if constexpr (blk == 3) P[1] = q ? P[1] : prod;
                    if constexpr (blk == 4) P[1] = q ? prod : P[1];
                }
                sp = last ? 1.0 : gj * sp;
                if (keep) et[row + j] = zt[row + j] * sp;
                if constexpr (j == 0) gc[0] = q ? gc[0] : 0.0;
                if constexpr (j % 8 == 0) __builtin_amdgcn_sched_barrier(0);
                if constexpr (j > 0) self(self, std::integral_constant<int, j - 1>());
            };
            up(up, std::integral_constant<int, N - 1>());
        }
        wave_lds_sync();
#pragma unroll
        for (int h = 0; h < 3; ++h)
            hv[h] = r + 16 * h < N ? zt[D::kPoles * ZS + r + 16 * h] : 0.0;
        const int left = np - pb < D::kPoles ? np - pb : D::kPoles;
#pragma unroll 1
        for (int k = 0; k < left; k += 4) {
#pragma unroll
            for (int pr = 0; pr < 4; pr += 2) {
                const int pa = k + pr, pq = k + pr + 1;
                const bool on = pq != D::kPoles;  // (the solution's lane is no pole)
                auto rows = [&](auto self, auto H) -> void {
                    constexpr int h = decltype(H)::value, w = D::width(h);
                    const int i = r + 16 * h;
                    const int at = i < N ? i : 0;
                    const bool in = i < N;
                    double wa = zt[pa * ZS + at], wb = zt[pq * ZS + at];
                    double ea = et[pa * ZS + at], eb = et[pq * ZS + at];
                    wa = in ? wa : 0.0;
                    wb = in && on ? wb : 0.0;
                    eb = on ? eb : 0.0;
                    // the lane row's block in the rows' own slot
                    const bool enter = q == 1 && r < w;
                    double sa = enter ? ea : 0.0, sb = enter ? eb : 0.0;
                    int own = r - w * q;
                    asm volatile("" : "+v"(own));
                    pair_chain<w, 0>(A[h] + 8 * h, gc + 8 * h, wa, wb, sa, sb, pr, own);
                    if constexpr (h < 2) {
                        double ta = 0.0, tb = 0.0;
                        pair_scale(ta, tb, P[h], sa, sb, pr);
                        const bool late = q == 0 && r >= w;
                        sa = late ? ea : ta;
                        sb = late ? eb : tb;
                        pair_chain_on<D::width(h + 1), 0>(A[h] + 8 * (h + 1), gc + 8 * (h + 1), sa,
                                                          sb, pr);
                    }
                    if constexpr (h == 0) {
                        double ta = 0.0, tb = 0.0;
                        pair_scale(ta, tb, P[1], sa, sb, pr);
                        sa = ta;
                        sb = tb;
                        pair_chain_on<D::width(2), 0>(A[0] + 16, gc + 16, sa, sb, pr);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (h < 2) self(self, std::integral_constant<int, h + 1>());
                };
                rows(rows, std::integral_constant<int, 0>());
            }
            auto turn = [](double& v) {
                const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x12C, 0xF, 0xF, true);
                const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x12C, 0xF, 0xF, true);
                v = __hiloint2double(hi, lo);
            };
#pragma unroll
            for (int c = 0; c < D::COLS; ++c) turn(gc[c]);
            turn(P[0]);
            turn(P[1]);
        }
        wave_lds_sync();
    }
    // lower triangle, one slot of rows at a time through LDS
    auto mirror = [&](auto self, auto SS) -> void {
        constexpr int s = decltype(SS)::value, w = D::width(s);
#pragma unroll
        for (int c = 8 * s; c < D::COLS; ++c)
            if (16 * s + r < N) zt[r * ZS + (q ? D::elem(c, 1) : D::elem(c, 0))] = A[s][c];
        wave_lds_sync();
        if (16 * s + r < N) zt[r * ZS + 16 * s + r] = 0.0;
        wave_lds_sync();
#pragma unroll
        for (int h = s; h < 3; ++h) {
            const int i = 16 * h + r;
#pragma unroll
            for (int k = 0; k < w; ++k) {
                const double t = zt[(w * q + k) * ZS + (i < N ? i : 0)];
                A[h][8 * s + k] += i < N ? t : 0.0;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        wave_lds_sync();
        if constexpr (s < 2) self(self, std::integral_constant<int, s + 1>());
    };
    mirror(mirror, std::integral_constant<int, 0>());
#pragma unroll
    for (int h = 0; h < 3; ++h) b[h] = hv[h];
    pair_back_phase<N, 0>(A, b, vs, lane);
    pair_back_phase<N, 1>(A, b, vs, lane);
    pair_back_phase<N, 2>(A, b, vs, lane);
    return finite;
}

// ---------------------------------------------------------------------------
// one node per wavefront, 32 < N <= 64
// ---------------------------------------------------------------------------
// Lane (g, r) = (lane / 16, lane % 16) holds columns 16 g .. 16 g + 15 of the rows 16 h + r,
// h < NS: NS x 16 doubles, half the registers of whole rows two to a lane, and still
// every broadcast is a row_newbcast inside the lane's own row of 16.  A vector lives
// "by element" (element = lane) as the broadcast operand and "by row" (element 16 h + r
// in register h) as the lane's own factor; the two forms, and the sum of the four
// column blocks' partial products, go through LDS.
template <int N>
struct DirectW {
    static_assert(N > 32 && N <= 64 && N % 8 == 0, "three or four rows of 16");
    static constexpr int NS = (N + 15) / 16;
    static constexpr int ZS = 16 * NS + 1;
    static constexpr int kTab = 16 * ZS;
    // tables g, z, e; block products [16][4]; partial products [4][64]; two vectors
    static constexpr int kDoubles = 3 * kTab + 64 + 256 + 128;
};

// x (element = lane) as rows: out[h] = element 16 h + r, through the LDS vector vec.
template <int S>
__device__ __forceinline__ void to_rows(double x, double (&out)[S], double* vec, int lane) {
    wave_lds_sync();
    vec[lane] = x;
    wave_lds_sync();
#pragma unroll
    for (int h = 0; h < S; ++h) out[h] = vec[16 * h + (lane & 15)];
}

// Element lane of A v: the partial products over this lane's W columns, summed over
// the first GR column blocks (the others' v is zero).
template <int NS, int SP, int GR, int W>
__device__ __forceinline__ double wave_matvec(const double (&A)[NS][16], double v, double* part,
                                              int lane) {
    double pr[SP];
#pragma unroll
    for (int h = 0; h < SP; ++h) {
        double s0 = 0.0, s1 = 0.0;
        fmac_dot<0, W>(A[h], v, s0, s1);
        pr[h] = s0 + s1;
    }
    const int g = lane >> 4, r = lane & 15;
    wave_lds_sync();
    if (g < GR) {
#pragma unroll
        for (int h = 0; h < SP; ++h) part[64 * g + 16 * h + r] = pr[h];
    }
    wave_lds_sync();
    double p = 0.0;
    if (lane < 16 * SP) {
#pragma unroll
        for (int k = 0; k < GR; ++k) p += part[64 * k + lane];
    }
    return p;
}

// The steps n - 1 = HI .. LO of the tridiagonalisation, pivot rows in slot S (supports
// within slots 0 .. S); W columns per block (less than 16 only for S = 0).
template <int N, int S, int HI, int LO, int W, typename R>
__device__ __forceinline__ void wtri_phase(double (&A)[DirectW<N>::NS][16], double& d, double& e,
                                           double& b, double* lds, const R& vs, int lane) {
    using D = DirectW<N>;
    constexpr int NS = D::NS;
    double* part = lds + 3 * D::kTab + 64;
    double* vec = part + 256;
    const int g = lane >> 4, r = lane & 15;
#pragma unroll 1
    for (int n = HI + 1; n > LO; --n) {
        // row n - 1 (by symmetry column n - 1): its 16-column pieces sit in the lanes
        // (g, (n - 1) % 16)
        wave_lds_sync();
        if (r == ((n - 1) & 15) && g <= S) {
#pragma unroll
            for (int k = 0; k < 16; k += 2)
                *reinterpret_cast<double2*>(vec + 16 * g + k) = make_double2(A[S][k], A[S][k + 1]);
        }
        wave_lds_sync();
        const double raw = lane < n ? vec[lane] : 0.0;
        d = lane == n - 1 ? raw : d;
        const double x = lane < n - 1 ? raw : 0.0;
        const double s2 = wave_sum(x * x);
        const double x1 = lane_value(x, n - 2);
        const bool some = s2 > 1e-290;
        const double norm = s2 * fast_rsqrt(s2);
        const double rb = some ? fast_rsqrt(fma(fabs(x1), norm, s2)) : 0.0;
        const double alpha = some ? -copysign(norm, x1) : x1;
        const double shift = some ? copysign(norm, x1) : 0.0;
        const bool piv = lane == n - 2;
        e = piv ? alpha : e;
        const double v = (x + (piv ? shift : 0.0)) * rb;
        vs.put(n, lane, v);
        double vr[S + 1], p_r[S + 1];
        to_rows<S + 1>(v, vr, vec + 64, lane);
        const double p = wave_matvec<NS, S + 1, S + 1, W>(A, v, part, lane);
        const double c = wave_sum(v * p);
        b = fma(-wave_sum(v * b), v, b);
        to_rows<S + 1>(p, p_r, vec, lane);
#pragma unroll
        for (int h = 0; h <= S; ++h) {
            fmac_axpy<0, W>(A[h], p, -vr[h]);
            fmac_axpy<0, W>(A[h], v, -fma(-c, vr[h], p_r[h]));
        }
    }
}

// The same steps of the back transformation, ascending.
template <int N, int S, int HI, int LO, int W, typename R>
__device__ __forceinline__ void wback_phase(double (&G)[DirectW<N>::NS][16], double& hv, double* lds,
                                            const R& vs, int lane) {
    using D = DirectW<N>;
    constexpr int NS = D::NS;
    double* part = lds + 3 * D::kTab + 64;
    double* vec = part + 256;
#pragma unroll 1
    for (int n = LO + 1; n <= HI + 1; ++n) {
        const double v = vs.get(n, lane);
        double vr[S + 1], p_r[NS];
        to_rows<S + 1>(v, vr, vec + 64, lane);
        const double p = wave_matvec<NS, NS, S + 1, W>(G, v, part, lane);
        const double c = wave_sum(v * p);
        hv = fma(-wave_sum(v * hv), v, hv);
        to_rows<NS>(p, p_r, vec, lane);
#pragma unroll
        for (int h = 0; h < NS; ++h) {
            if (h <= S) {
                const double vh = vr[h <= S ? h : 0];
                fmac_axpy<0, 16>(G[h], p, -vh);
                fmac_axpy<0, W>(G[h], v, -fma(-c, vh, p_r[h]));
            } else {
                fmac_axpy<0, W>(G[h], v, -p_r[h]);
            }
        }
    }
}

template <int N, int S, typename R>
__device__ __forceinline__ void wtri_all(double (&A)[DirectW<N>::NS][16], double& d, double& e,
                                         double& b, double* lds, const R& vs, int lane) {
    constexpr int HI = 16 * S + 15 < N - 1 ? 16 * S + 15 : N - 1;
    if constexpr (S > 0) {
        wtri_phase<N, S, HI, 16 * S, 16>(A, d, e, b, lds, vs, lane);
        wtri_all<N, S - 1>(A, d, e, b, lds, vs, lane);
    } else {
        wtri_phase<N, 0, 15, 8, 16>(A, d, e, b, lds, vs, lane);
        wtri_phase<N, 0, 7, 2, 8>(A, d, e, b, lds, vs, lane);
    }
}
template <int N, int S, typename R>
__device__ __forceinline__ void wback_all(double (&G)[DirectW<N>::NS][16], double& hv, double* lds,
                                          const R& vs, int lane) {
    constexpr int HI = 16 * S + 15 < N - 1 ? 16 * S + 15 : N - 1;
    if constexpr (S > 0) {
        wback_all<N, S - 1>(G, hv, lds, vs, lane);
        wback_phase<N, S, HI, 16 * S, 16>(G, hv, lds, vs, lane);
    } else {
        wback_phase<N, 0, 7, 2, 8>(G, hv, lds, vs, lane);
        wback_phase<N, 0, 15, 8, 16>(G, hv, lds, vs, lane);
    }
}

// row_chain for one 16-column block: columns K.., `own`: the column of the row's diagonal in
// this block, if 0..15; pa, pb: the previous column (for K = 0 the block's start value).
template <int K>
__device__ __forceinline__ void wave_chain(double (&a)[16], const double (&g)[16], double wa,
                                           double wb, double pa, double pb, int pr, int own) {
    double ua[4], ub[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const bool o = own == K + k;
        ua[k] = o ? wa : (K + k == 0 ? pa : 0.0);
        ub[k] = o ? wb : (K + k == 0 ? pb : 0.0);
    }
    constexpr int F = K == 0 ? 1 : 0;
    if (pr == 0)
        fmac_chain<0, 4 - F>(ua + F, ub + F, g + K - 1 + F, F ? ua[0] : pa, F ? ub[0] : pb);
    else
        fmac_chain<2, 4 - F>(ua + F, ub + F, g + K - 1 + F, F ? ua[0] : pa, F ? ub[0] : pb);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        a[K + k] += ua[k] + ub[k];
        // summed here: otherwise the additions of all slots and poles are left to the end of
        // the pass and their operands spill
        asm volatile("" : "+v"(a[K + k]));
    }
    if constexpr (K < 12) wave_chain<K + 4>(a, g, wa, wb, ua[3], ub[3], pr, own);
}

// sym_direct for the one node of a wavefront (b: element = lane).  lds:
// DirectW<N>::kDoubles doubles.
template <int N, bool ROOT, typename R>
__device__ __forceinline__ bool sym_direct_wave(double (&A)[DirectW<N>::NS][16], double& b,
                                                double ia, double scale, double* lds, const R& vs,
                                                int lane) {
    using D = DirectW<N>;
    constexpr int NS = D::NS;
    constexpr int ZS = D::ZS;
    double* gt = lds;                // [16 poles][ZS] g_j
    double* zt = gt + D::kTab;       // 1 / gamma_j, then z_jj c (row 15: the solution of X h = b)
    double* et = zt + D::kTab;       // products of g to the end of j's block, then z_jj c times them
    double* pb = et + D::kTab;       // [16 poles][4] block products
    const int g = lane >> 4, r = lane & 15;
    double d = 0.0, e = 0.0;
    wtri_all<N, NS - 1>(A, d, e, b, lds, vs, lane);
    if (g == 0) {
        d = r == 0 ? A[0][0] : (r == 1 ? A[0][1] : d);
        e = r == 0 ? A[0][1] : e;
    }
    d *= ia;
    e *= ia;
    const bool finite = __all(fabs(d) + fabs(e) < 1e300);
    const float df = (float)d, ef = (float)e;
    const int cls = pole_class<true>(df * df + 2.0f * ef * ef);
    const int p0 = kPoleOffset[cls], np = kPoleOffset[cls + 1] - p0;
#pragma unroll
    for (int h = 0; h < NS; ++h)
#pragma unroll
        for (int k = 0; k < 16; ++k) A[h][k] = 0.0;
    double hv = 0.0;
#pragma unroll 1
    for (int pc = 0; pc < np; pc += 15) {
        const int pi = pc + r < np && r < 15 ? p0 + pc + r : -1;
        const double t2 = pi >= 0 ? kSqrtPoles[pi < 0 ? 0 : pi].t2 : 0.0;
        double cw = pi >= 0 ? kSqrtPoles[pi < 0 ? 0 : pi].c * scale : 0.0;
        if constexpr (ROOT) cw *= 1.0 + t2;
        const double base = 1.0 + t2;
        wave_lds_sync();
        {
            // as in sym_direct: 1 / gamma_j, on the lanes of pole 15 y_j / gamma_j
            double rg = 0.0, y = 0.0, sp = 0.0;
#pragma unroll 4
            for (int j = N - 1; j >= 0; --j) {
                const double ej = j == N - 1 ? 0.0 : lane_value(e, j);
                const double gj = -ej * rg;
                y = fma(gj, y, lane_value(b, j));
                rg = fast_rcp(fma(gj, ej, base + lane_value(d, j)));
                sp = (j & 15) == 15 ? gj : gj * sp;
                if (g == 0) {
                    gt[r * ZS + j] = gj;
                    zt[r * ZS + j] = r == 15 ? y * rg : rg;
                    et[r * ZS + j] = sp;
                    if ((j & 15) == 0) pb[4 * r + (j >> 4)] = sp;
                }
            }
        }
        wave_lds_sync();
        if (g == 0) {
            double z = 0.0, m = 0.0;
            const double cx = r == 15 ? 1.0 : cw;
#pragma unroll 4
            for (int j = 0; j < N; ++j) {
                const double gj = gt[r * ZS + j];
                z = fma(m, z, zt[r * ZS + j]);
                et[r * ZS + j] *= z * cx;
                zt[r * ZS + j] = z * cx;
                m = r == 15 ? gj : gj * gj;
            }
        }
        wave_lds_sync();
        hv = lane < N ? zt[15 * ZS + lane] : 0.0;
        double gc[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const double v = gt[r * ZS + 16 * (g < NS ? g : 0) + k];
            gc[k] = 16 * g + k < N ? v : 0.0;
        }
        const int left = np - pc < 15 ? np - pc : 15;
#pragma unroll 1
        for (int q = 0; q < left; q += 4) {
#pragma unroll
            for (int pr = 0; pr < 4; pr += 2) {
                const int pa = q + pr, pq = q + pr + 1;
                // row 15 is the solution for b, not a pole (and may hold a NaN of b's)
                const bool on = pq != 15;
                const int el = lane < N ? lane : 0;
                const double wa = zt[pa * ZS + el];
                const double wq = zt[pq * ZS + el], wb = on ? wq : 0.0;
#pragma unroll
                for (int h = 0; h < NS; ++h) {
                    // block g > h starts from row i's value at the end of its own block
                    // times the products of the blocks in between
                    double sa = 0.0, sb = 0.0;
                    if (h + 1 < NS) {
                        sa = et[pa * ZS + 16 * h + r];
                        sb = et[pq * ZS + 16 * h + r];
                        sb = on ? sb : 0.0;
#pragma unroll
                        for (int k = h + 1; k + 1 < NS; ++k) {
                            sa *= g > k ? pb[4 * pa + k] : 1.0;
                            sb *= g > k ? pb[4 * pq + k] : 1.0;
                        }
                    }
                    const bool later = h + 1 < NS && g > h;
                    double pa_ = later ? sa : 0.0, pb_ = later ? sb : 0.0;
                    // (opaque, so that the sixteen lane masks are formed where they are used
                    // instead of being kept in 128 scalar registers)
                    int own = lane - 16 * h;
                    asm volatile("" : "+v"(own));
                    wave_chain<0>(A[h], gc, wa, wb, pa_, pb_, pr, own);
                }
            }
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int lo = __builtin_amdgcn_mov_dpp(__double2loint(gc[k]), 0x12C, 0xF, 0xF, true);
                const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(gc[k]), 0x12C, 0xF, 0xF, true);
                gc[k] = __hiloint2double(hi, lo);
            }
        }
    }
    // lower triangle, one slot of rows at a time: rows 16 s + r to LDS, their columns back
    // to the lanes of group s
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        wave_lds_sync();
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if (g >= s && g < NS) zt[r * ZS + 16 * g + k] = A[s][k];
        if (g == s) zt[r * ZS + lane] = 0.0;
        wave_lds_sync();
#pragma unroll
        for (int h = s; h < NS; ++h) {
            double t[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) t[k] = zt[k * ZS + 16 * h + r];
#pragma unroll
            for (int k = 0; k < 16; ++k) A[h][k] += g == s ? t[k] : 0.0;
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    b = hv;
    wback_all<N, NS - 1>(A, b, lds, vs, lane);
    return finite;
}

}  // namespace dev
}  // namespace lbmletkf
