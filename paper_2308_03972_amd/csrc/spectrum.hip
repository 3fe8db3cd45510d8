// Energy spectrum of an ensemble (Sec. 4.1 shell definition; the ensemble's
// spectrum is the mean of the members' spectra, Sec. 4.3.2):
//   E(k) = M^-1 sum_m sum_{k - 1/2 <= |k'| < k + 1/2} (|u_hat_m(k')|^2 + |v_hat_m(k')|^2) / 2,
//   u_hat(k') = n^-2 sum_xi u(xi) exp(-2 pi i k'.xi / n),  u = j / rho per member.
// u and v are transformed together as z = u + i v: for real u, v
//   |z_hat(k)|^2 + |z_hat(-k)|^2 = 2 (|u_hat(k)|^2 + |v_hat(k)|^2),
// and a shell holds -k with every k, so E(k) sums |z_hat|^2 / 2 over the full plane.
//
// Each 1D transform of length n = n1 n2 (n1 the largest divisor <= sqrt n) goes in two
// passes through LDS (Cooley-Tukey): for x = n2 a + b, k = c + n1 d,
//   Y_b(c) = sum_a z(n2 a + b) e^{-2 pi i a c / n1},
//   Z(k)   = sum_b Y_b(c) e^{-2 pi i b k / n},
// n (n1 + n2) products instead of n^2; a prime n has n1 = 1, the direct sum.  The
// row pass reads a row for a group of members (whole cache lines), the column pass
// sums |Z|^2 over its group of members in member order, the groups are added in order,
// and the shells sum in a fixed order (deterministic).  Passes of any n: 256^2 x 64 FP64 rows
// 637 -> 136 us, columns 880 -> 116 us against direct sums with one member per block (shells
// 38 -> 14), bound by LDS reads (one 16-byte value per four multiply-adds) and latency;
// with factors of 8 and 16 in registers, see below.
// Off the hot path: called at report times.  Scratch comes from the
// context's ping-pong buffer.
#include "common.h"
#include "device_util.h"

namespace lbmletkf {
namespace {
using namespace dev;

constexpr int kSpecBlock = 256;
constexpr int kSpecLds = 72 * 1024;  // line buffers: two blocks per CU

// Stride of a line in LDS: n values, or n1 pieces of n2 + 1 (a padding value each, so that
// 16 lanes reading different pieces hit different banks), and one more.
__host__ __device__ inline int spec_stride(int n, int n1) { return n + n1 + 1; }

// Lines (members of a row, columns of a member) a block transforms at a time.
inline int spec_lines(int n, int n1, int most) {
    int l = 1;
    while (l * 2 <= most && 2 * (l * 2) * spec_stride(n, n1) * (int)sizeof(double2) <= kSpecLds) l *= 2;
    return l;
}
// LDS: two line buffers and the twiddle table.
inline size_t spec_lds(int n, int n1, int lines) {
    return ((size_t)2 * lines * spec_stride(n, n1) + n) * sizeof(double2);
}

inline int spec_factor(int n) {
    int f = 1;
    for (int d = 1; d * d <= n; ++d)
        if (n % d == 0) f = d;
    return f;
}

// Members of one column-pass block, and the number of such groups.
constexpr int kColMembers = 2;
inline int col_groups(int members) { return (members + kColMembers - 1) / kColMembers; }

__device__ __forceinline__ void fill_twiddles(double2* tw, int n) {
    for (int j = threadIdx.x; j < n; j += kSpecBlock) {
        double s, c;
        sincospi(2.0 * (double)j / (double)n, &s, &c);
        tw[j] = make_double2(c, -s);
    }
}

__device__ __forceinline__ void mac(double2& acc, double2 z, double2 w) {
    acc.x = fma(z.x, w.x, fma(-z.y, w.y, acc.x));
    acc.y = fma(z.x, w.y, fma(z.y, w.x, acc.y));
}

// The transform of `lines` lines z[line][n] (LDS): Y in y[line][n], then emit(line, k, Z).
// L lines at a time share each twiddle factor; a thread past the last line repeats it, so that
// the loops have no branches (all passes, us, with a branch per line / without: 97^2 x 8 85 / 28,
// 254^2 x 8 209 / 86).  A prime n takes k and n - k from the same four sums (251^2 x 64, both:
// 1026 / 318).
template <int L, typename Emit>
__device__ __forceinline__ void transform(const double2* z, double2* y, const double2* tw, int n,
                                          int n1, int n2, int lines, Emit emit) {
    const int lb = (lines + L - 1) / L, ls = spec_stride(n, n1);
    __syncthreads();
    if (n1 == 1) {
        // k and n - k together: the sums of x c, y s, y c and x s (twiddle c - i s) give both
        const int half = n / 2 + 1;
        for (int t = threadIdx.x; t < lb * half; t += kSpecBlock) {
            const int q = t / half, k = t - q * half;
            const double2* at[L];
            double2 even[L], odd[L];  // (sum x c, sum y c), (sum y s, sum x s)
#pragma unroll
            for (int l = 0; l < L; ++l) {
                at[l] = z + min(L * q + l, lines - 1) * ls;
                even[l] = odd[l] = make_double2(0.0, 0.0);
            }
            int p = 0;
#pragma unroll 4
            for (int b = 0; b < n; ++b) {
                const double2 w = tw[p];
#pragma unroll
                for (int l = 0; l < L; ++l) {
                    const double2 v = at[l][b];
                    even[l].x = fma(v.x, w.x, even[l].x);
                    even[l].y = fma(v.y, w.x, even[l].y);
                    odd[l].x = fma(v.y, -w.y, odd[l].x);
                    odd[l].y = fma(v.x, -w.y, odd[l].y);
                }
                p += k;
                if (p >= n) p -= n;
            }
#pragma unroll
            for (int l = 0; l < L; ++l) {
                if (L * q + l >= lines) break;
                emit(L * q + l, k, make_double2(even[l].x + odd[l].x, even[l].y - odd[l].y));
                if (k > 0 && 2 * k < n)
                    emit(L * q + l, n - k,
                         make_double2(even[l].x - odd[l].x, even[l].y + odd[l].y));
            }
        }
        __syncthreads();
        return;
    }
    for (int t = threadIdx.x; t < lb * n; t += kSpecBlock) {
        const int q = t / n, i = t - q * n;  // i = c n2 + b
        const int c = i / n2, b = i - c * n2;
        const double2* at[L];
        double2 acc[L];
#pragma unroll
        for (int l = 0; l < L; ++l) {
            at[l] = z + min(L * q + l, lines - 1) * ls + b;
            acc[l] = make_double2(0.0, 0.0);
        }
        int p = 0;
        const int dp = c * n2;  // < n
#pragma unroll 4
        for (int a = 0; a < n1; ++a) {
            const double2 w = tw[p];
#pragma unroll
            for (int l = 0; l < L; ++l) mac(acc[l], at[l][n2 * a], w);
            p += dp;
            if (p >= n) p -= n;
        }
#pragma unroll
        for (int l = 0; l < L; ++l)
            if (L * q + l < lines) y[(L * q + l) * ls + i + c] = acc[l];
    }
    __syncthreads();
    for (int t = threadIdx.x; t < lb * n; t += kSpecBlock) {
        const int q = t / n, k = t - q * n;
        const int c = k % n1;
        const double2* at[L];
        double2 acc[L];
#pragma unroll
        for (int l = 0; l < L; ++l) {
            at[l] = y + min(L * q + l, lines - 1) * ls + c * (n2 + 1);
            acc[l] = make_double2(0.0, 0.0);
        }
        int p = 0;
#pragma unroll 4
        for (int b = 0; b < n2; ++b) {
            const double2 w = tw[p];
#pragma unroll
            for (int l = 0; l < L; ++l) mac(acc[l], at[l][b], w);
            p += k;
            if (p >= n) p -= n;
        }
#pragma unroll
        for (int l = 0; l < L; ++l)
            if (L * q + l < lines) emit(L * q + l, k, acc[l]);
    }
    __syncthreads();
}

// Row pass: block = (row y, group of `lines` members); out[m][y][kx].
template <typename T, int L>
__global__ __launch_bounds__(kSpecBlock) void spectrum_rows_kernel(const T* __restrict__ f, int n,
                                                                   int n1, int members, int lines,
                                                                   double2* __restrict__ out) {
    extern __shared__ double2 spec[];
    double2* z = spec;
    const int ls = spec_stride(n, n1);
    double2* y2 = z + (size_t)lines * ls;
    double2* tw = y2 + (size_t)lines * ls;
    const int groups = (members + lines - 1) / lines;
    const int blk = xcd_remap(blockIdx.x, gridDim.x);  // a row's groups share cache lines
    const int y = blk / groups, m0 = (blk - y * groups) * lines;
    const int nm = min(lines, members - m0);
    fill_twiddles(tw, n);
    for (int t = threadIdx.x; t < n * nm; t += kSpecBlock) {
        const int x = t / nm, m = t - x * nm;
        double rho = 0.0, jx = 0.0, jy = 0.0;
#pragma unroll
        for (int a = 0; a < 9; ++a) {
            const double fa =
                PopIO<T>::load(f + slot(src_node(x, y, a, n, n), a, m0 + m, members), a);
            rho += fa;
            jx += cx_of(a) * fa;
            jy += cy_of(a) * fa;
        }
        z[m * ls + x] = make_double2(jx / rho, jy / rho);
    }
    transform<L>(z, y2, tw, n, n1, n / n1, nm, [&](int l, int k, double2 v) {
        out[((size_t)(m0 + l) * n + y) * n + k] = v;
    });
}

// Column pass: block = (tile of `lines` kx, group of kColMembers members);
// e[group][ky][kx] = sum over the group's members of |Z|^2 / 2.
template <int L>
__global__ __launch_bounds__(kSpecBlock) void spectrum_cols_kernel(const double2* __restrict__ rows,
                                                                   int n, int n1, int members,
                                                                   int lines,
                                                                   double* __restrict__ e) {
    extern __shared__ double2 spec[];
    double2* z = spec;
    const int ls = spec_stride(n, n1);
    double2* y2 = z + (size_t)lines * ls;
    double2* tw = y2 + (size_t)lines * ls;
    const int tiles = (n + lines - 1) / lines;
    const int group = blockIdx.x / tiles, kx0 = (blockIdx.x - group * tiles) * lines;
    const int nl = min(lines, n - kx0);
    fill_twiddles(tw, n);
    double* const eg = e + (size_t)group * n * n;
    const int mend = min(members, (group + 1) * kColMembers);
    for (int m = group * kColMembers; m < mend; ++m) {
        for (int t = threadIdx.x; t < n * nl; t += kSpecBlock) {
            const int y = t / nl, l = t - y * nl;
            z[l * ls + y] = rows[((size_t)m * n + y) * n + kx0 + l];
        }
        const bool first = m == group * kColMembers;
        transform<L>(z, y2, tw, n, n1, n / n1, nl, [&](int l, int k, double2 v) {
            // (the same thread visits (l, k) for every member)
            double* p = eg + (size_t)k * n + kx0 + l;
            const double w = 0.5 * (v.x * v.x + v.y * v.y);
            *p = first ? w : *p + w;
        });
    }
}

// The same passes for n = n1 n2 with factors of 8 and 16 (64, 128, 256): a thread holds one
// sub-transform of 8 or 16 values in registers, radix 4 x 4 or 2 x 4, so that a value crosses
// LDS three times instead of 2 (n1 + n2) / 4 and the line buffer is used in place, which
// leaves room for sixteen lines: whole 128-byte lines of members in the row pass, and of columns
// in the column pass, whose sums over its members stay in registers.  256^2 x 64 FP64: rows
// 136 -> 71 us, columns 116 -> 20 us.  Bound by HBM (the state once, the row transforms
// written and read).
__device__ __forceinline__ double2 cmul(double2 a, double c, double s) {  // a (c - i s)
    return make_double2(fma(a.x, c, a.y * s), fma(a.y, c, -a.x * s));
}
__device__ __forceinline__ void dft4(double2& a, double2& b, double2& c, double2& d) {
    const double2 p = make_double2(a.x + c.x, a.y + c.y), m = make_double2(a.x - c.x, a.y - c.y);
    const double2 q = make_double2(b.x + d.x, b.y + d.y), r = make_double2(b.x - d.x, b.y - d.y);
    a = make_double2(p.x + q.x, p.y + q.y);
    b = make_double2(m.x + r.y, m.y - r.x);
    c = make_double2(p.x - q.x, p.y - q.y);
    d = make_double2(m.x - r.y, m.y + r.x);
}
// v <- its R-point transform, in order: index 4 a + b, a < R / 4, then c + (R / 4) d.
template <int R>
__device__ __forceinline__ void dft(double2 (&v)[R]) {
    static_assert(R == 8 || R == 16, "radix 2 x 4 or 4 x 4");
    constexpr int Q = R / 4;
    constexpr double kCos[10] = {1.0, 0.92387953251128675613, 0.70710678118654752440,
                                 0.38268343236508977173, 0.0, -0.38268343236508977173,
                                 -0.70710678118654752440, -0.92387953251128675613, -1.0,
                                 -0.92387953251128675613};  // cos(pi k / 8)
    constexpr double kSin[10] = {0.0, 0.38268343236508977173, 0.70710678118654752440,
                                 0.92387953251128675613, 1.0, 0.92387953251128675613,
                                 0.70710678118654752440, 0.38268343236508977173, 0.0,
                                 -0.38268343236508977173};
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        if constexpr (R == 16) {
            dft4(v[b], v[4 + b], v[8 + b], v[12 + b]);
        } else {
            const double2 p = v[b], q = v[4 + b];
            v[b] = make_double2(p.x + q.x, p.y + q.y);
            v[4 + b] = make_double2(p.x - q.x, p.y - q.y);
        }
#pragma unroll
        for (int c = 1; c < Q; ++c)
            if (b > 0) v[4 * c + b] = cmul(v[4 * c + b], kCos[b * c * (16 / R)], kSin[b * c * (16 / R)]);
    }
    double2 u[R];
#pragma unroll
    for (int c = 0; c < Q; ++c) {
        dft4(v[4 * c], v[4 * c + 1], v[4 * c + 2], v[4 * c + 3]);
#pragma unroll
        for (int d = 0; d < 4; ++d) u[c + Q * d] = v[4 * c + d];
    }
#pragma unroll
    for (int j = 0; j < R; ++j) v[j] = u[j];
}

constexpr int kRegLines = 16;

template <int N1, int N2>
constexpr size_t reg_lds() {
    return ((size_t)kRegLines * (N1 * N2 + N1 + 1) + N1 * N2) * sizeof(double2);
}

// transform() in place on z[line][n], line < lines <= 16; emit(line, c, u) gets
// Z(c + N1 d) = u[d], threads with consecutive line (LINE) or c together.
template <int N1, int N2, bool LINE, typename Emit>
__device__ __forceinline__ void transform_regs(double2* z, const double2* tw, int lines, Emit emit) {
    constexpr int ls = N1 * N2 + N1 + 1;
    const int t = threadIdx.x;
    const int l = t / N2, b = t % N2;
    const bool on = l < lines;
    __syncthreads();
    double2 v[N1];
    if (on) {
#pragma unroll
        for (int a = 0; a < N1; ++a) v[a] = z[l * ls + N2 * a + b];
        dft<N1>(v);
#pragma unroll
        for (int c = 1; c < N1; ++c) {
            const double2 w = tw[b * c];
            v[c] = cmul(v[c], w.x, -w.y);
        }
    }
    __syncthreads();
    if (on) {
#pragma unroll
        for (int c = 0; c < N1; ++c) z[l * ls + c * (N2 + 1) + b] = v[c];
    }
    __syncthreads();
    const int l2 = LINE ? t % kRegLines : t / N1, c2 = LINE ? t / kRegLines : t % N1;
    if (c2 < N1 && l2 < lines) {
        double2 u[N2];
#pragma unroll
        for (int d = 0; d < N2; ++d) u[d] = z[l2 * ls + c2 * (N2 + 1) + d];
        dft<N2>(u);
        emit(l2, c2, u);
    }
    __syncthreads();
}

template <typename T, int N1, int N2>
__global__ __launch_bounds__(kSpecBlock) void spectrum_rows_regs_kernel(const T* __restrict__ f,
                                                                        int members,
                                                                        double2* __restrict__ out) {
    extern __shared__ double2 spec[];
    constexpr int n = N1 * N2, ls = n + N1 + 1;
    double2* z = spec;
    double2* tw = z + kRegLines * ls;
    const int groups = (members + kRegLines - 1) / kRegLines;
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const int y = blk / groups, m0 = (blk - y * groups) * kRegLines;
    const int nm = min(kRegLines, members - m0);
    fill_twiddles(tw, n);
    const int m = threadIdx.x % kRegLines;
    if (m < nm) {
#pragma unroll 2
        for (int x = threadIdx.x / kRegLines; x < n; x += kSpecBlock / kRegLines) {
            double rho = 0.0, jx = 0.0, jy = 0.0;
#pragma unroll
            for (int a = 0; a < 9; ++a) {
                const double fa =
                    PopIO<T>::load(f + slot(src_node(x, y, a, n, n), a, m0 + m, members), a);
                rho += fa;
                jx += cx_of(a) * fa;
                jy += cy_of(a) * fa;
            }
            z[m * ls + x] = make_double2(jx / rho, jy / rho);
        }
    }
    transform_regs<N1, N2, false>(z, tw, nm, [&](int l, int c, const double2 (&u)[N2]) {
        double2* o = out + ((size_t)(m0 + l) * n + y) * n + c;
#pragma unroll
        for (int d = 0; d < N2; ++d) o[N1 * d] = u[d];
    });
}

template <int N1, int N2>
__global__ __launch_bounds__(kSpecBlock) void spectrum_cols_regs_kernel(
    const double2* __restrict__ rows, int members, double* __restrict__ e) {
    extern __shared__ double2 spec[];
    constexpr int n = N1 * N2, ls = n + N1 + 1, tiles = n / kRegLines;
    double2* z = spec;
    double2* tw = z + kRegLines * ls;
    const int group = blockIdx.x / tiles, kx0 = (blockIdx.x - group * tiles) * kRegLines;
    fill_twiddles(tw, n);
    double* const eg = e + (size_t)group * n * n;
    const int mend = min(members, (group + 1) * kColMembers);
    double acc[N2];
#pragma unroll
    for (int d = 0; d < N2; ++d) acc[d] = 0.0;
    for (int m = group * kColMembers; m < mend; ++m) {
        const int l = threadIdx.x % kRegLines;
#pragma unroll 4
        for (int y = threadIdx.x / kRegLines; y < n; y += kSpecBlock / kRegLines)
            z[l * ls + y] = rows[((size_t)m * n + y) * n + kx0 + l];
        transform_regs<N1, N2, true>(z, tw, kRegLines, [&](int, int, const double2 (&u)[N2]) {
#pragma unroll
            for (int d = 0; d < N2; ++d) acc[d] += 0.5 * (u[d].x * u[d].x + u[d].y * u[d].y);
        });
    }
    // (the thread of line l and residue c, as transform_regs deals them out)
    const int l = threadIdx.x % kRegLines, c = threadIdx.x / kRegLines;
    if (c < N1) {
#pragma unroll
        for (int d = 0; d < N2; ++d) eg[(size_t)(c + N1 * d) * n + kx0 + l] = acc[d];
    }
}

// The groups' sums added up, in group order, into the first.
__global__ __launch_bounds__(kSpecBlock) void spectrum_fold_kernel(double* __restrict__ e, int modes,
                                                                   int groups) {
    const int i = blockIdx.x * kSpecBlock + threadIdx.x;
    if (i >= modes) return;
    double acc = e[i];
#pragma unroll 8
    for (int g = 1; g < groups; ++g) acc += e[(size_t)g * modes + i];
    e[i] = acc;
}

// Shell pass: block k.  E[k] = sum over the modes of shell k, floor(|k'| + 1/2) = k, of e,
// / (M n^4): a thread takes one sign of ky and the columns kx = t, t + 128, ..., whose
// modes of the shell lie within two of sqrt((k +- 1/2)^2 - kx^2), in ascending |ky|.
// e: the sums of `groups` groups of members, added up here in group order.
__global__ __launch_bounds__(kSpecBlock) void spectrum_shell_kernel(const double* __restrict__ e,
                                                                    int n, int groups, int members,
                                                                    double* __restrict__ E) {
    __shared__ double red[kSpecBlock];
    const int k = blockIdx.x;
    double acc = 0.0;
    const bool neg = threadIdx.x >= kSpecBlock / 2;
    const int top = neg ? (n - 1) / 2 : n / 2;  // largest |ky| of this sign
    for (int kx = threadIdx.x % (kSpecBlock / 2); kx < n; kx += kSpecBlock / 2) {
        const int kxs = 2 * kx > n ? kx - n : kx;
        if (abs(kxs) > k + 1) continue;
        const double in2 = (k - 0.5) * (k - 0.5) - (double)kxs * kxs;
        const double out2 = (k + 0.5) * (k + 0.5) - (double)kxs * kxs;
        const int hi = min(out2 > 0.0 ? (int)sqrtf((float)out2) + 2 : 1, top);
        const int lo = max(k > 0 && in2 > 0.0 ? (int)sqrtf((float)in2) - 2 : 0, neg ? 1 : 0);
        // floor(|k'| + 1/2) = k in whole numbers: k^2 - k < |k'|^2 <= k^2 + k (0 for k = 0)
#pragma unroll 4
        for (int s = lo; s <= hi; ++s) {
            const int r2 = kxs * kxs + s * s;
            const double* at = e + (size_t)(neg ? n - s : s) * n + kx;
            double mode = at[0];
            for (int g = 1; g < groups; ++g) mode += at[(size_t)g * n * n];
            acc += r2 <= k * k + k && (k == 0 || r2 > k * k - k) ? mode : 0.0;
        }
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = kSpecBlock / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double n2 = (double)n * (double)n;
        E[k] = red[0] / ((double)members * n2 * n2);
    }
}

template <typename K>
hipError_t allow_spec_lds(K kernel, size_t bytes) {
    if (bytes <= 65536) return hipSuccess;
    return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)bytes);
}

template <typename T, int L>
hipError_t launch_rows_any(const void* f, int n, int n1, int members, int lines, double2* rows,
                           hipStream_t s) {
    const size_t lds = spec_lds(n, n1, lines);
    hipError_t err = allow_spec_lds(spectrum_rows_kernel<T, L>, lds);
    if (err != hipSuccess) return err;
    spectrum_rows_kernel<T, L><<<n * ((members + lines - 1) / lines), kSpecBlock, lds, s>>>(
        (const T*)f, n, n1, members, lines, rows);
    return hipGetLastError();
}

template <int L>
hipError_t launch_cols_any(const double2* rows, int n, int n1, int members, int lines, double* e,
                           hipStream_t s) {
    const size_t lds = spec_lds(n, n1, lines);
    hipError_t err = allow_spec_lds(spectrum_cols_kernel<L>, lds);
    if (err != hipSuccess) return err;
    spectrum_cols_kernel<L><<<col_groups(members) * ((n + lines - 1) / lines), kSpecBlock, lds, s>>>(
        rows, n, n1, members, lines, e);
    return hipGetLastError();
}

// Row and column passes: e[group][ky][kx] from the state.
hipError_t launch_passes_any(const void* f, int n, int members, int storage, double2* rows, double* e,
                             hipStream_t s) {
    const int n1 = spec_factor(n);
    int most = 1;
    while (most < members && most < 16) most *= 2;
    int rl = spec_lines(n, n1, most), cl = spec_lines(n, n1, 8);
    // (lines shared by a block save LDS reads, but few members leave few blocks: then fewer
    // lines each until two blocks per CU have work.  us, all passes, 16 and 8
    // lines / this: 251^2 x 1 161 / 76)
    while (rl > 1 && n * ((members + rl - 1) / rl) < 512) rl /= 2;
    while (cl > 1 && col_groups(members) * ((n + cl - 1) / cl) < 512) cl /= 2;
    hipError_t err =
        storage == kStoreF32Dev
            ? (rl >= 4   ? launch_rows_any<float, 4>(f, n, n1, members, rl, rows, s)
               : rl == 2 ? launch_rows_any<float, 2>(f, n, n1, members, rl, rows, s)
                         : launch_rows_any<float, 1>(f, n, n1, members, rl, rows, s))
            : (rl >= 4   ? launch_rows_any<double, 4>(f, n, n1, members, rl, rows, s)
               : rl == 2 ? launch_rows_any<double, 2>(f, n, n1, members, rl, rows, s)
                         : launch_rows_any<double, 1>(f, n, n1, members, rl, rows, s));
    if (err != hipSuccess) return err;
    return cl >= 4   ? launch_cols_any<4>(rows, n, n1, members, cl, e, s)
           : cl == 2 ? launch_cols_any<2>(rows, n, n1, members, cl, e, s)
                     : launch_cols_any<1>(rows, n, n1, members, cl, e, s);
}

template <typename T, int N1, int N2>
hipError_t launch_passes_t(const T* f, int members, double2* rows, double* e, hipStream_t s) {
    constexpr int n = N1 * N2;
    constexpr size_t lds = reg_lds<N1, N2>();
    hipError_t err = allow_spec_lds(spectrum_rows_regs_kernel<T, N1, N2>, lds);
    if (err == hipSuccess) err = allow_spec_lds(spectrum_cols_regs_kernel<N1, N2>, lds);
    if (err != hipSuccess) return err;
    spectrum_rows_regs_kernel<T, N1, N2>
        <<<n * ((members + kRegLines - 1) / kRegLines), kSpecBlock, lds, s>>>(f, members, rows);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    spectrum_cols_regs_kernel<N1, N2>
        <<<col_groups(members) * (n / kRegLines), kSpecBlock, lds, s>>>(rows, members, e);
    return hipGetLastError();
}

template <int N1, int N2>
hipError_t launch_passes(const void* f, int members, int storage, double2* rows, double* e,
                         hipStream_t s) {
    return storage == kStoreF32Dev
               ? launch_passes_t<float, N1, N2>((const float*)f, members, rows, e, s)
               : launch_passes_t<double, N1, N2>((const double*)f, members, rows, e, s);
}

}  // namespace

size_t spectrum_scratch_bytes(int n, int members) {
    const size_t rows = (size_t)members * n * n * sizeof(double2);
    const size_t need = rows + (size_t)col_groups(members) * n * n * sizeof(double);
    // the documented requirement (half-plane transforms of u and v, one energy plane)
    const size_t ncol = (size_t)n / 2 + 1;
    const size_t stated = (size_t)members * n * ncol * 32 + n * ncol * sizeof(double) + 256;
    return need > stated ? need : stated;
}

hipError_t launch_energy_spectrum(const void* f, int n, int members, int storage, int kmax,
                                  void* scratch, double* E, hipStream_t s) {
    double2* rows = reinterpret_cast<double2*>(scratch);
    double* e = reinterpret_cast<double*>(rows + (size_t)members * n * n);
    int groups = col_groups(members);
    // (the sizes whose two factors are 8 or 16 transform in registers, 252 -> 91 us for both passes
    // at 256^2 x 64; same results to rounding)
    hipError_t err = n == 256   ? launch_passes<16, 16>(f, members, storage, rows, e, s)
                     : n == 128 ? launch_passes<8, 16>(f, members, storage, rows, e, s)
                     : n == 64  ? launch_passes<8, 8>(f, members, storage, rows, e, s)
                                : launch_passes_any(f, n, members, storage, rows, e, s);
    if (err != hipSuccess) return err;
    // (few modes in few groups: the shells add them up themselves, a launch less: 16^2 x 8
    // 20.6 -> 18.2 us; 31^2 x 64 in 32 groups 38 -> 80)
    if (groups > 4 || (groups > 1 && n * n * groups > 32768)) {
        spectrum_fold_kernel<<<(n * n + kSpecBlock - 1) / kSpecBlock, kSpecBlock, 0, s>>>(e, n * n,
                                                                                          groups);
        if ((err = hipGetLastError()) != hipSuccess) return err;
        groups = 1;
    }
    spectrum_shell_kernel<<<kmax + 1, kSpecBlock, 0, s>>>(e, n, groups, members, E);
    return hipGetLastError();
}

}  // namespace lbmletkf
