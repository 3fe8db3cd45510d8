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
// and the shells sum in a fixed order (deterministic).  256^2 x 64 FP64: rows 637 -> 136 us, columns
// 880 -> 116 us, shells 38 -> 14 us against direct sums with one member per block.
// Bound by LDS reads (one 16-byte value per four multiply-adds) and latency.
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
// Four lines at a time share each twiddle factor.
template <typename Emit>
__device__ __forceinline__ void transform(const double2* z, double2* y, const double2* tw, int n,
                                          int n1, int n2, int lines, Emit emit) {
    const int lb = (lines + 3) / 4, ls = spec_stride(n, n1);
    __syncthreads();
    if (n1 > 1) {
        for (int t = threadIdx.x; t < lb * n; t += kSpecBlock) {
            const int q = t / n, i = t - q * n;  // i = c n2 + b
            const int c = i / n2, b = i - c * n2;
            double2 acc[4];
#pragma unroll
            for (int l = 0; l < 4; ++l) acc[l] = make_double2(0.0, 0.0);
            int p = 0;
            const int dp = c * n2;  // < n
            for (int a = 0; a < n1; ++a) {
                const double2 w = tw[p];
#pragma unroll
                for (int l = 0; l < 4; ++l)
                    if (4 * q + l < lines) mac(acc[l], z[(4 * q + l) * ls + n2 * a + b], w);
                p += dp;
                if (p >= n) p -= n;
            }
#pragma unroll
            for (int l = 0; l < 4; ++l)
                if (4 * q + l < lines) y[(4 * q + l) * ls + i + c] = acc[l];
        }
        __syncthreads();
    }
    const double2* src = n1 > 1 ? y : z;
    for (int t = threadIdx.x; t < lb * n; t += kSpecBlock) {
        const int q = t / n, k = t - q * n;
        const int c = n1 > 1 ? k % n1 : 0;
        double2 acc[4];
#pragma unroll
        for (int l = 0; l < 4; ++l) acc[l] = make_double2(0.0, 0.0);
        int p = 0;
        for (int b = 0; b < n2; ++b) {
            const double2 w = tw[p];
#pragma unroll
            for (int l = 0; l < 4; ++l)
                if (4 * q + l < lines) mac(acc[l], src[(4 * q + l) * ls + c * (n2 + 1) + b], w);
            p += k;
            if (p >= n) p -= n;
        }
#pragma unroll
        for (int l = 0; l < 4; ++l)
            if (4 * q + l < lines) emit(4 * q + l, k, acc[l]);
    }
    __syncthreads();
}

// Row pass: block = (row y, group of `lines` members); out[m][y][kx].
template <typename T>
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
    transform(z, y2, tw, n, n1, n / n1, nm, [&](int l, int k, double2 v) {
        out[((size_t)(m0 + l) * n + y) * n + k] = v;
    });
}

// Column pass: block = (tile of `lines` kx, group of kColMembers members);
// e[group][ky][kx] = sum over the group's members of |Z|^2 / 2.
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
        transform(z, y2, tw, n, n1, n / n1, nl, [&](int l, int k, double2 v) {
            // (the same thread visits (l, k) for every member)
            double* p = eg + (size_t)k * n + kx0 + l;
            const double w = 0.5 * (v.x * v.x + v.y * v.y);
            *p = first ? w : *p + w;
        });
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
__global__ __launch_bounds__(kSpecBlock) void spectrum_shell_kernel(const double* __restrict__ e,
                                                                    int n, int members,
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
        const int hi = min(out2 > 0.0 ? (int)sqrt(out2) + 2 : 1, top);
        const int lo = max(k > 0 && in2 > 0.0 ? (int)sqrt(in2) - 2 : 0, neg ? 1 : 0);
        for (int s = lo; s <= hi; ++s) {
            if ((int)floor(sqrt((double)(kxs * kxs + s * s)) + 0.5) != k) continue;
            acc += e[(size_t)(neg ? n - s : s) * n + kx];
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
    const int n1 = spec_factor(n);
    int most = 1;
    while (most < members && most < 16) most *= 2;
    const int rl = spec_lines(n, n1, most), cl = spec_lines(n, n1, 8);
    const size_t row_lds = spec_lds(n, n1, rl), col_lds = spec_lds(n, n1, cl);
    const int row_blocks = n * ((members + rl - 1) / rl);
    hipError_t err;
    if (storage == kStoreF32Dev) {
        if ((err = allow_spec_lds(spectrum_rows_kernel<float>, row_lds)) != hipSuccess) return err;
        spectrum_rows_kernel<float><<<row_blocks, kSpecBlock, row_lds, s>>>((const float*)f, n, n1,
                                                                            members, rl, rows);
    } else {
        if ((err = allow_spec_lds(spectrum_rows_kernel<double>, row_lds)) != hipSuccess) return err;
        spectrum_rows_kernel<double><<<row_blocks, kSpecBlock, row_lds, s>>>((const double*)f, n, n1,
                                                                             members, rl, rows);
    }
    if ((err = hipGetLastError()) != hipSuccess) return err;
    if ((err = allow_spec_lds(spectrum_cols_kernel, col_lds)) != hipSuccess) return err;
    const int groups = col_groups(members);
    spectrum_cols_kernel<<<groups * ((n + cl - 1) / cl), kSpecBlock, col_lds, s>>>(rows, n, n1,
                                                                                   members, cl, e);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    if (groups > 1) {
        spectrum_fold_kernel<<<(n * n + kSpecBlock - 1) / kSpecBlock, kSpecBlock, 0, s>>>(e, n * n,
                                                                                          groups);
        if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    spectrum_shell_kernel<<<kmax + 1, kSpecBlock, 0, s>>>(e, n, members, E);
    return hipGetLastError();
}

}  // namespace lbmletkf
