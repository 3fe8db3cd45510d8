// The observation route's update of the nine populations, from the solver's G and h
// (letkf_obs.hip, letkf_direct.hip):
//   B = dX Z^T (9 x l),  x_m = x_bar + sqrt(beta) dX_m + B h + (B G) Z_m.
//
// Four nodes per wavefront, a row of 16 lanes each; lane r holds the members r, r + 16,
// .. of its node's populations, and observations (of B and C = B G) r, r + 16, ..  All
// three contractions run on v_fmac_f64_dpp with the row_newbcast operand:
//   B: lane = observation, the member's dX broadcast, the lane's own row of dY streamed;
//   C: lane = column of G (streamed, coalesced), B broadcast;
//   Z: lane = member, C broadcast, the members' dY streamed, added into dX in place.
// Where one node per wavefront spent an LDS read per multiply-add of B and ran C on 18 of
// 64 lanes, this takes 3900 vector instructions per four nodes of 18 observations and 64
// members against 8400.  Bound by FP64 issue (9 (M ceil(l / 16) + l ceil(l / 16) +
// l ceil(M / 16)) multiply-adds per four nodes, 40% of the time) and by the latencies of
// about 16 dependent loads at two wavefronts per SIMD, which the populations' registers
// allow.  256^2 nodes, 64 members, FP64: analysis 750 -> 600 us; 512^2, FP32: 2.8 -> 2.1 ms.
// Measured and left out: rows of dY through LDS (as fast; 40% fewer cache accesses) and
// three wavefronts per SIMD with 19 registers spilled (1% slower).
#include <type_traits>

#include "common.h"
#include "device_util.h"
#include "sym_direct.h"

namespace lbmletkf {
namespace {
using namespace dev;

// acc[a] += bcast(x[a], L) * y for the nine populations (hazard: see fmac_axpy).
#define LBM_F9(a, x) \
    "v_fmac_f64_dpp %" #a ", %" #x ", %18 row_newbcast:%19 row_mask:0xf bank_mask:0xf\n\t"
template <int L>
__device__ __forceinline__ void fmac9(double (&acc)[9], const double (&x)[9], double y) {
    asm("s_nop 1\n\t" LBM_F9(0, 9) LBM_F9(1, 10) LBM_F9(2, 11) LBM_F9(3, 12) LBM_F9(4, 13)
            LBM_F9(5, 14) LBM_F9(6, 15) LBM_F9(7, 16) LBM_F9(8, 17)
        : "+&v"(acc[0]), "+&v"(acc[1]), "+&v"(acc[2]), "+&v"(acc[3]), "+&v"(acc[4]),
          "+&v"(acc[5]), "+&v"(acc[6]), "+&v"(acc[7]), "+&v"(acc[8])
        : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(x[6]), "v"(x[7]),
          "v"(x[8]), "v"(y), "n"(L));
}
#undef LBM_F9

template <int K>
using Int = std::integral_constant<int, K>;

// f(Int<0>()) .. f(Int<N - 1>()); the scheduling barrier after each keeps the compiler from
// hoisting the loads of all chunks to the front (twice the registers and more).
template <int N, int C = 0, typename F>
__device__ __forceinline__ void chunks(F& f) {
    if constexpr (C < N) {
        f(Int<C>());
        __builtin_amdgcn_sched_barrier(0);
        chunks<N, C + 1>(f);
    }
}

// acc[h] += bcast(x, L + t) * y[t][h], t < W, h < NS
template <int L, int W, int NS, int T = 0>
__device__ __forceinline__ void fmac9xw(double (&acc)[NS][9], const double (&x)[9],
                                        const double (&y)[W][NS]) {
    if constexpr (T < W) {
#pragma unroll
        for (int h = 0; h < NS; ++h) fmac9<L + T>(acc[h], x, y[T][h]);
        fmac9xw<L, W, NS, T + 1>(acc, x, y);
    }
}

typedef double double2u __attribute__((ext_vector_type(2), aligned(8)));

// The address in lane L of each row of 16.
template <int L>
__device__ __forceinline__ const double* row_bcast_ptr(const double* v) {
    return reinterpret_cast<const double*>(
        __builtin_bit_cast(long, row_bcast<L>(__builtin_bit_cast(double, v))));
}

// Nodes nodes[item0 .. end - 1] (at most four), problem size n <= 16 NS, M <= 16 MS.  A row
// past the end repeats the first node and stores nothing.
template <int NS, int MS, typename T>
__device__ __forceinline__ void apply_rows(const AnalysisParams& p, const int* nodes, int item0,
                                           int end, int n, const double* __restrict__ gin,
                                           double (*__restrict__ mean)[12]) {
    T* __restrict__ fs = reinterpret_cast<T*>(p.f);
    const int lane = threadIdx.x;
    const int r = lane & 15, row = lane >> 4;
    const bool valid = item0 + row < end;
    const int node = nodes[item0 + (valid ? row : 0)];
    const int nx = p.nx, ny = p.ny, M = p.members;
    const int x = node % nx, y = node / nx;
    const int sz = n * n + n;
    const double* __restrict__ g = gin + (size_t)item0 * sz;  // uniform
    const int grow = valid ? row * sz : 0;

    // independent loads first: the populations, this lane's observations and h
    // (only the last slot can reach past the ensemble: it repeats the last member)
    const bool tail = r + 16 * (MS - 1) < M;
    const int rlast = tail ? r + 16 * (MS - 1) : M - 1;
    double f[MS][9];
    {
        const PullSlots<const T> src(fs, x, wrap(x - 1, nx), wrap(x + 1, nx), y, wrap(y - 1, ny),
                                     wrap(y + 1, ny), nx, M, r);
#pragma unroll
        for (int a = 0; a < 9; ++a) {
            const T* at = src.at(a);
#pragma unroll
            for (int s = 0; s + 1 < MS; ++s) f[s][a] = PopIO<T>::load(at + 16 * s, a);
            f[MS - 1][a] = PopIO<T>::load(at + (rlast - r), a);
        }
    }
    int q[NS];
    double w[NS], hv[NS];
#pragma unroll
    for (int h = 0; h < NS; ++h) {
        q[h] = 0;
        w[h] = 0.0;
        const int j = r + 16 * h;
        if (j < n) local_obs(p, node, j, &q[h], &w[h], nullptr);
        hv[h] = j < n ? g[grow + n * n + j] : 0.0;
    }
    // (so that a zero weight meets no other node's values below)
    const bool any = weighted_indices<NS>(q, w, lane);
    const double* yr[NS];
#pragma unroll
    for (int h = 0; h < NS; ++h) yr[h] = p.dY + (size_t)q[h] * M;

    bool mem[MS];
#pragma unroll
    for (int s = 0; s < MS; ++s) mem[s] = s + 1 < MS || tail;
#pragma unroll
    for (int a = 0; a < 9; ++a) f[MS - 1][a] = tail ? f[MS - 1][a] : 0.0;
    if (p.diag_node)
        row_diag_record<MS>(f, mem, M, node, nx * ny, p.truth_uv,
                            p.diag_node + (size_t)node * kDiagFieldCount, valid, r);
    // (the means wait in LDS: in registers they would cost B a wavefront per SIMD)
    wave_lds_sync();  // (a queue's previous nodes are done with theirs)
    const double rm = 1.0 / M;
#pragma unroll
    for (int a = 0; a < 9; ++a) {
        double s1 = f[0][a];
#pragma unroll
        for (int s = 1; s < MS; ++s) s1 += f[s][a];
        const double xb = row_sum(s1) * rm;
        if (r == a) mean[row][a] = xb;
#pragma unroll
        for (int s = 0; s + 1 < MS; ++s) f[s][a] -= xb;
        f[MS - 1][a] = tail ? f[MS - 1][a] - xb : 0.0;
    }

    // (a row of lanes whose node has no weighted observation sits this out as a whole)
    double B[NS][9];
#pragma unroll
    for (int h = 0; h < NS; ++h)
#pragma unroll
        for (int a = 0; a < 9; ++a) B[h][a] = 0.0;
    if (any) {
        // B[h][a] of observation 16 h + r, unweighted: eight members at a time
        auto b_part = [&](auto Q) {
            constexpr int m = 8 * decltype(Q)::value, s = m / 16, k = m % 16;
            double z[8][NS];
            if (m + 8 <= 16 * (MS - 1) || m + 8 <= M) {  // uniform
#pragma unroll
                for (int t = 0; t < 8; t += 2)
#pragma unroll
                    for (int h = 0; h < NS; ++h) {
                        const double2u v = *reinterpret_cast<const double2u*>(yr[h] + m + t);
                        z[t][h] = v.x;
                        z[t + 1][h] = v.y;
                    }
            } else {
                if (m >= M) return;
                // (a member past the ensemble reads the last one again: dX is 0 there)
#pragma unroll
                for (int t = 0; t < 8; ++t)
#pragma unroll
                    for (int h = 0; h < NS; ++h) z[t][h] = yr[h][min(m + t, M - 1)];
            }
            fmac9xw<k, 8>(B, f[s], z);
        };
        chunks<2 * MS>(b_part);
#pragma unroll
        for (int h = 0; h < NS; ++h)
#pragma unroll
            for (int a = 0; a < 9; ++a) B[h][a] *= w[h];
    }
    // x_bar plus the mean increment B h waits with the means; the members' part of the update
    // replaces dX and stays at the size of dX until the end (summed into the populations
    // themselves, each of its n terms would round at their size: 3 to 10 ulps against 1)
    wave_lds_sync();
#pragma unroll
    for (int a = 0; a < 9; ++a) {
        double d = B[0][a] * hv[0];
#pragma unroll
        for (int h = 1; h < NS; ++h) d = fma(B[h][a], hv[h], d);
        d = row_sum(d);
        if (r == a) mean[row][a] += d;
#pragma unroll
        for (int s = 0; s < MS; ++s) f[s][a] *= p.sqrt_beta;
    }
    if (any) {
        // C = B G, column 16 h + r, then weighted for the unweighted dY below
        double C[NS][9];
#pragma unroll
        for (int h = 0; h < NS; ++h)
#pragma unroll
            for (int a = 0; a < 9; ++a) C[h][a] = 0.0;
        int col[NS];
#pragma unroll
        for (int h = 0; h < NS; ++h) col[h] = grow + (r + 16 * h < n ? r + 16 * h : 0);
        auto c_part = [&](auto Q) {
            constexpr int j = 4 * decltype(Q)::value, hb = j / 16, k = j % 16;
            if (j >= n) return;  // uniform
            // (columns past n collect values nobody reads, rows past n meet B = 0)
            double v[4][NS];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const double* gr = g + min(j + t, n - 1) * n;
#pragma unroll
                for (int h = 0; h < NS; ++h) v[t][h] = gr[(unsigned)col[h]];
            }
            fmac9xw<k, 4>(C, B[hb], v);
        };
        chunks<4 * NS>(c_part);
#pragma unroll
        for (int h = 0; h < NS; ++h)
#pragma unroll
            for (int a = 0; a < 9; ++a) C[h][a] *= w[h];
        // the transform, four observations per chunk
        auto z_part = [&](auto Q) {
            constexpr int j = 4 * decltype(Q)::value, hb = j / 16, k = j % 16;
            if (j >= n) return;  // uniform
            double z[4][MS];
            auto load = [&](auto U) {
                constexpr int t = decltype(U)::value;
                const double* yt = row_bcast_ptr<k + t>(yr[hb]);
#pragma unroll
                for (int s = 0; s + 1 < MS; ++s) z[t][s] = (yt + r)[16 * s];
                z[t][MS - 1] = yt[rlast];
            };
            load(Int<0>());
            load(Int<1>());
            load(Int<2>());
            load(Int<3>());
#pragma unroll
            for (int s = 0; s < MS; ++s) fmac9<k>(f[s], C[hb], z[0][s]);
#pragma unroll
            for (int s = 0; s < MS; ++s) fmac9<k + 1>(f[s], C[hb], z[1][s]);
#pragma unroll
            for (int s = 0; s < MS; ++s) fmac9<k + 2>(f[s], C[hb], z[2][s]);
#pragma unroll
            for (int s = 0; s < MS; ++s) fmac9<k + 3>(f[s], C[hb], z[3][s]);
        };
        chunks<4 * NS>(z_part);
    }
    wave_lds_sync();
#pragma unroll
    for (int a = 0; a < 9; ++a) {
        const double c0 = mean[row][a];
#pragma unroll
        for (int s = 0; s < MS; ++s) f[s][a] += c0;
    }
    {
        // (the slots' addresses anew: kept from the loads they would hold 18 registers)
        int xs = x;
        asm volatile("" : "+v"(xs));
        const PullSlots<T> dst(fs, xs, wrap(xs - 1, nx), wrap(xs + 1, nx), y, wrap(y - 1, ny),
                               wrap(y + 1, ny), nx, M, r);
#pragma unroll
        for (int s = 0; s < MS; ++s) {
            if (valid && mem[s]) {
#pragma unroll
                for (int a = 0; a < 9; ++a) PopIO<T>::store(dst.at(a) + 16 * s, a, f[s][a]);
            }
        }
    }
    if (p.diag_node) {
#pragma unroll
        for (int s = 0; s < MS; ++s)
#pragma unroll
            for (int a = 0; a < 9; ++a) f[s][a] = PopIO<T>::round(f[s][a], a);
        row_diag_record<MS>(f, mem, M, node, nx * ny, p.truth_uv,
                            p.diag_node + ((size_t)nx * ny + node) * kDiagFieldCount, valid, r);
    }
}

// Wavefronts per SIMD (four slots of observations with three or four of members keep 20 and 60
// registers in scratch memory).
template <int NS>
constexpr int apply_waves() { return 2; }

template <int NS, int MS, typename T>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(apply_waves<NS>())))
void analysis_apply_rows_kernel(AnalysisParams p, const int* nodes, int count, int n,
                                const double* __restrict__ gin) {
    __shared__ double mean[4][12];
    apply_rows<NS, MS, T>(p, nodes, xcd_remap(blockIdx.x, gridDim.x) * 4, count, n, gin, mean);
}

// Batched form: waves[w] = (4 problem + items - 1, first item).
template <int NS, int MS, typename T>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(apply_waves<NS>())))
void analysis_apply_rows_batch_kernel(const AnalysisParams* P, const int2* waves, int nwaves,
                                      const int* nodes, int n, const double* __restrict__ gin) {
    const int w = xcd_remap(blockIdx.x, gridDim.x);
    if (w >= nwaves) return;
    __shared__ double mean[4][12];
    const int2 d = waves[w];
    apply_rows<NS, MS, T>(P[d.x >> 2], nodes, d.y, d.y + (d.x & 3) + 1, n, gin, mean);
}

template <int NS, int MS, typename T>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(apply_waves<NS>())))
void analysis_apply_rows_queue_kernel(const AnalysisParams* P, const int2* waves, int nwaves,
                                      const int* nodes, int n, const double* __restrict__ gin,
                                      int* counters) {
    __shared__ int next;
    __shared__ double mean[4][12];
    const int per = (nwaves + 7) / 8;
    const int lo = (int)(blockIdx.x % 8) * per;
    const int hi = min(nwaves, lo + per);
    for (;;) {
        const int w0 = queue_take(counters, &next, lo);
        if (w0 >= hi) return;  // uniform over the block
        const int w1 = min(hi, w0 + kQueueChunk);
        for (int w = w0; w < w1; ++w) {
            const int2 d = waves[w];
            apply_rows<NS, MS, T>(P[d.x >> 2], nodes, d.y, d.y + (d.x & 3) + 1, n, gin, mean);
        }
    }
}

template <int NS, int MS, typename T>
hipError_t launch_t(const ApplyLaunch& l, hipStream_t s) {
    if (!l.waves)
        analysis_apply_rows_kernel<NS, MS, T><<<(l.count + 3) / 4, 64, 0, s>>>(*l.p, l.nodes, l.count,
                                                                               l.n, l.gbuf);
    else if (!l.counters)
        analysis_apply_rows_batch_kernel<NS, MS, T><<<l.count, 64, 0, s>>>(
            l.d_params, l.waves, l.count, l.nodes, l.n, l.gbuf);
    else
        analysis_apply_rows_queue_kernel<NS, MS, T><<<persistent_blocks(64, l.count), 64, 0, s>>>(
            l.d_params, l.waves, l.count, l.nodes, l.n, l.gbuf, l.counters);
    return hipGetLastError();
}

template <int NS, int MS>
hipError_t launch_s(const ApplyLaunch& l, hipStream_t s) {
    return l.storage == kStoreF32Dev ? launch_t<NS, MS, float>(l, s) : launch_t<NS, MS, double>(l, s);
}

template <int NS>
hipError_t launch_m(const ApplyLaunch& l, hipStream_t s) {
    switch ((l.members + 15) / 16) {
        case 1: return launch_s<NS, 1>(l, s);
        case 2: return launch_s<NS, 2>(l, s);
        case 3: return launch_s<NS, 3>(l, s);
        case 4: return launch_s<NS, 4>(l, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_apply_rows(const ApplyLaunch& l, hipStream_t s) {
    if (l.count == 0) return hipSuccess;
    switch ((l.n + 15) / 16) {
        case 1: return launch_m<1>(l, s);
        case 2: return launch_m<2>(l, s);
        case 3: return launch_m<3>(l, s);
        case 4: return launch_m<4>(l, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace lbmletkf
