// The analysis without iteration (sym_direct.h), for both routes.
//
// Observation route: with X = I + S / a, S = Z Z^T (l x l) and a = (M - 1) / beta,
//   G = U phi(Lambda) U^T = -sqrt(beta) / a  F(X),   h = U psi U^T d~ = X^{-1} d~ / a
// (phi, psi and how G and h enter the update: letkf_obs.hip).
// Ensemble route: with X = A / a = I + Z^T Z / a (M x M),
//   dW = sqrt((M - 1)) A^{-1/2} = sqrt(beta) X^{-1/2},   w_bar = X^{-1} Z^T d~ / a,
// and the update x_m = x_bar + dX (w_bar + dW[:, m]) of the nine populations follows in the
// same wavefront, the rows of dW still in registers.
//
// Sizes up to 32 take four nodes per wavefront (a row of 16 lanes each), the observation
// route's 40 and 48 two, larger ones (and the ensemble route's 48) one.
// What bounds it: FP64 issue and the latency of the reflector chain (two reductions and
// two reciprocal square roots per step); LDS and memory traffic are minor.  Measured
// per node (S resident, 39,232 nodes at N <= 32, 16,384 beyond; before: the Jacobi
// solver): N = 8 1.0 ns (6), 16 2.4 (19), 18 3.8 (15), 24 7.3 (65), 32 11.5 (109),
// 40 32 (404; one node per wavefront: 62), 48 43 (687; 75), 64 178 (1466).
#include <type_traits>

#include "common.h"
#include "device_util.h"
#include "sym_direct.h"

namespace lbmletkf {
namespace {
using namespace dev;

template <int N>
constexpr bool kRows16 = N <= 32;  // four nodes per wavefront
template <int N>
constexpr bool kPairs = N > 32 && N <= 48;  // two (observation route)

// Adds the wavefront's failed nodes (SEG lanes each, any of them `bad`) to *count.
template <int SEG>
__device__ __forceinline__ void count_failed(bool bad, int* count, int lane) {
    const unsigned long long lanes = __ballot(bad);
    if (lanes == 0) return;  // uniform
    int nodes = 0;
#pragma unroll
    for (int k = 0; k < kWave; k += SEG) nodes += (lanes >> k & ((1ull << SEG) - 1)) != 0;
    if (lane == 0) atomicAdd(count, nodes);
}

// ---------------------------------------------------------------------------
// observation route
// ---------------------------------------------------------------------------
// (An observation without weight takes the index of one that counts, so that the products
// with K meet no other node's values; a node without any reads finite localization
// weights in place of K.)

// Four nodes nodes[item0 + 0 .. 3] (item < end) of one problem.
template <int N>
__device__ __forceinline__ void direct_body(const AnalysisParams p, const int* nodes, int item0,
                                            int end, double* gout) {
    constexpr int NS = Direct<N>::NS;
    extern __shared__ double lds[];
    const int lane = threadIdx.x;
    const int r = lane & 15;
    const int item = item0 + (lane >> 4);
    const bool valid = item < end;
    const int node = valid ? nodes[item] : 0;
    int q[NS];
    double w[NS], b[NS];
#pragma unroll
    for (int h = 0; h < NS; ++h) {
        q[h] = 0;
        w[h] = b[h] = 0.0;
        if (valid && r + 16 * h < N) local_obs(p, node, r + 16 * h, &q[h], &w[h], &b[h]);
    }
    const bool any = weighted_indices<NS>(q, w, lane);
    const double* krow[NS];
#pragma unroll
    for (int h = 0; h < NS; ++h) krow[h] = any ? p.K + (size_t)q[h] * p.nobs : p.loc_g;
    // S = diag(w) K diag(w): all loads in flight together, then the weights
    double A[NS][N];
    auto load = [&](auto self, auto J) -> void {
        constexpr int j = decltype(J)::value;
        const int qj = __builtin_amdgcn_mov_dpp(q[j / 16], 0x150 + j % 16, 0xF, 0xF, true);
#pragma unroll
        for (int h = 0; h < NS; ++h) A[h][j] = krow[h][qj];
        if constexpr (j + 1 < N) self(self, std::integral_constant<int, j + 1>());
    };
    load(load, std::integral_constant<int, 0>());
    auto weigh = [&](auto self, auto J) -> void {
        constexpr int j = decltype(J)::value;
        const double wj = row_bcast<j % 16>(w[j / 16]);
#pragma unroll
        for (int h = 0; h < NS; ++h) A[h][j] *= w[h] * wj;
        if constexpr (j + 1 < N) self(self, std::integral_constant<int, j + 1>());
    };
    weigh(weigh, std::integral_constant<int, 0>());
    const double ia = 1.0 / p.a;
    double* out = gout + (size_t)(valid ? item : item0) * (N * N + N);
    const ReflGlobal vs{out, N, valid};
    const bool finite = sym_direct<N, false>(A, b, ia, -p.sqrt_beta * ia, lds, vs, lane);
    count_failed<16>(valid && !finite, p.eig_fail, lane);
    if (valid) {
#pragma unroll
        for (int h = 0; h < NS; ++h) {
            const int i = r + 16 * h;
            if (i >= N) continue;
#pragma unroll
            for (int j = 0; j < N; ++j) out[(size_t)j * N + i] = A[h][j];
            out[(size_t)N * N + i] = b[h] * ia;
        }
    }
}

// Two nodes nodes[item0], nodes[item0 + 1] (item < end), N = 40 or 48.
template <int N>
__device__ __forceinline__ void direct_body_pair(const AnalysisParams p, const int* nodes, int item0,
                                                 int end, double* gout) {
    using D = DirectP<N>;
    extern __shared__ double lds[];
    const int lane = threadIdx.x;
    const int r = lane & 15, half = lane >> 4 & 1;
    const int item = item0 + (lane >> 5);
    const bool valid = item < end;
    const int node = valid ? nodes[item] : 0;
    int q[3];
    double w[3], b[3];
#pragma unroll
    for (int h = 0; h < 3; ++h) {
        q[h] = 0;
        w[h] = b[h] = 0.0;
        if (valid && r + 16 * h < N) local_obs(p, node, r + 16 * h, &q[h], &w[h], &b[h]);
    }
    const bool any = weighted_indices<3>(q, w, lane);
    const double* krow[3];
#pragma unroll
    for (int h = 0; h < 3; ++h) krow[h] = any ? p.K + (size_t)q[h] * p.nobs : p.loc_g;
    // S = diag(w) K diag(w): all loads in flight together, then the weights
    double A[3][D::COLS];
    auto load = [&](auto self, auto C) -> void {
        constexpr int c = decltype(C)::value, j0 = D::elem(c, 0), j1 = D::elem(c, 1);
        const int q0 = __builtin_amdgcn_mov_dpp(q[j0 / 16], 0x150 + j0 % 16, 0xF, 0xF, true);
        const int q1 = __builtin_amdgcn_mov_dpp(q[j1 / 16], 0x150 + j1 % 16, 0xF, 0xF, true);
        const int qj = half ? q1 : q0;
#pragma unroll
        for (int h = 0; h < 3; ++h) A[h][c] = krow[h][qj];
        if constexpr (c + 1 < D::COLS) self(self, std::integral_constant<int, c + 1>());
    };
    load(load, std::integral_constant<int, 0>());
    auto weigh = [&](auto self, auto C) -> void {
        constexpr int c = decltype(C)::value, j0 = D::elem(c, 0), j1 = D::elem(c, 1);
        const double w0 = row_bcast<j0 % 16>(w[j0 / 16]), w1 = row_bcast<j1 % 16>(w[j1 / 16]);
        const double wj = half ? w1 : w0;
#pragma unroll
        for (int h = 0; h < 3; ++h) A[h][c] *= w[h] * wj;
        if constexpr (c + 1 < D::COLS) self(self, std::integral_constant<int, c + 1>());
    };
    weigh(weigh, std::integral_constant<int, 0>());
    const double ia = 1.0 / p.a;
    double* out = gout + (size_t)(valid ? item : item0) * (N * N + N);
    const ReflGlobal vs{out, N, valid};
    const bool finite = sym_direct_pair<N, false>(A, b, ia, -p.sqrt_beta * ia, lds, vs, lane);
    count_failed<32>(valid && !finite, p.eig_fail, lane);
    if (valid) {
#pragma unroll
        for (int h = 0; h < 3; ++h) {
            const int i = r + 16 * h;
            if (i >= N) continue;
#pragma unroll
            for (int c = 0; c < D::COLS; ++c)
                out[(size_t)(half ? D::elem(c, 1) : D::elem(c, 0)) * N + i] = A[h][c];
            if (half == 0) out[(size_t)N * N + i] = b[h] * ia;
        }
    }
}

// One node nodes[item] (item < end), 48 < N <= 64.
template <int N>
__device__ __forceinline__ void direct_body_wave(const AnalysisParams p, const int* nodes, int item,
                                                 int end, double* gout) {
    constexpr int NS = DirectW<N>::NS;
    extern __shared__ double lds[];
    const int lane = threadIdx.x;
    const int g = lane >> 4, r = lane & 15;
    if (item >= end) return;  // uniform over the wavefront
    const int node = nodes[item];
    int q = 0;
    double w = 0.0, b = 0.0;
    if (lane < N) local_obs(p, node, lane, &q, &w, &b);
    const unsigned long long on = __ballot(w != 0.0);
    const int qf = on ? __builtin_amdgcn_readlane(q, __ffsll(on) - 1) : 0;
    if (w == 0.0) q = qf;
    const double* kbase = on ? p.K : p.loc_g;
    double A[NS][16];
    double wr[NS];
#pragma unroll
    for (int h = 0; h < NS; ++h) {
        const int src = 16 * h + r;
        const int qr = __shfl(q, src, kWave);
        wr[h] = __shfl(w, src, kWave);
        const double* krow = kbase + (on ? (size_t)qr * p.nobs : 0);
        auto load = [&](auto self, auto J) -> void {
            constexpr int k = decltype(J)::value;
            A[h][k] = krow[__builtin_amdgcn_mov_dpp(q, 0x150 + k, 0xF, 0xF, true)];
            if constexpr (k + 1 < 16) self(self, std::integral_constant<int, k + 1>());
        };
        load(load, std::integral_constant<int, 0>());
    }
    auto weigh = [&](auto self, auto J) -> void {
        constexpr int k = decltype(J)::value;
        const double wk = row_bcast<k>(w);
#pragma unroll
        for (int h = 0; h < NS; ++h) A[h][k] *= wr[h] * wk;
        if constexpr (k + 1 < 16) self(self, std::integral_constant<int, k + 1>());
    };
    weigh(weigh, std::integral_constant<int, 0>());
    const double ia = 1.0 / p.a;
    double* out = gout + (size_t)item * (N * N + N);
    const ReflGlobal vs{out, N, true};
    const bool finite = sym_direct_wave<N, false>(A, b, ia, -p.sqrt_beta * ia, lds, vs, lane);
    if (!finite && lane == 0) atomicAdd(p.eig_fail, 1);
#pragma unroll
    for (int h = 0; h < NS; ++h) {
        const int i = 16 * h + r;
        if (i >= N) continue;
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if (16 * g + k < N) out[(size_t)(16 * g + k) * N + i] = A[h][k];
    }
    if (lane < N) out[(size_t)N * N + lane] = b * ia;
}

template <int N>
__device__ __forceinline__ void direct_node(const AnalysisParams p, const int* nodes, int item0,
                                            int end, double* gout) {
    if constexpr (kRows16<N>) direct_body<N>(p, nodes, item0, end, gout);
    else if constexpr (kPairs<N>) direct_body_pair<N>(p, nodes, item0, end, gout);
    else direct_body_wave<N>(p, nodes, item0, end, gout);
}

template <int N>
constexpr int direct_segs() { return kRows16<N> ? 4 : (kPairs<N> ? 2 : 1); }

// Wavefronts per SIMD.  At these N = 20 and 30 and 32 members keep two to four registers in
// scratch memory, the queue forms of 14 to 48 up to 73, and N = 56 and 64 about 180 (their queue
// forms 215 and 231): those hold NS x 16 matrix entries of two registers each beside
// the pole sums.  One wavefront per SIMD, with twice the registers, is not measured.
template <int N>
constexpr int direct_waves() { return N <= 16 ? 4 : (N <= 20 ? 3 : 2); }

template <int N>
constexpr size_t direct_lds_bytes() {
    if constexpr (kRows16<N>) return 4 * Direct<N>::kNodeDoubles * sizeof(double);
    else if constexpr (kPairs<N>) return 2 * DirectP<N>::kNodeDoubles * sizeof(double);
    else return DirectW<N>::kDoubles * sizeof(double);
}

template <int N>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(direct_waves<N>())))
void analysis_direct_kernel(AnalysisParams p, const int* nodes, int count, double* gout) {
    direct_node<N>(p, nodes, xcd_remap(blockIdx.x, gridDim.x) * direct_segs<N>(), count, gout);
}

// Batched form: wavefront w takes waves[w] = (problem, first item, end of the
// problem's items).
template <int N>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(direct_waves<N>())))
void analysis_direct_batch_kernel(const AnalysisParams* P, const int4* waves, int nwaves,
                                  const int* nodes, double* gout) {
    const int w = xcd_remap(blockIdx.x, gridDim.x);
    if (w >= nwaves) return;
    const int4 d = waves[w];
    const AnalysisParams p = P[d.x];
    direct_node<N>(p, nodes, d.y, d.z, gout);
}

template <int N>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(direct_waves<N>())))
void analysis_direct_queue_kernel(const AnalysisParams* P, const int4* waves, int nwaves,
                                  const int* nodes, double* gout, int* counters) {
    __shared__ int next;
    const int per = (nwaves + 7) / 8;
    const int lo = (int)(blockIdx.x % 8) * per;
    const int hi = min(nwaves, lo + per);
    for (;;) {
        const int w0 = queue_take(counters, &next, lo);
        if (w0 >= hi) return;  // uniform over the block
        const int w1 = min(hi, w0 + kQueueChunk);
        for (int w = w0; w < w1; ++w) {
            if (w > w0) __syncthreads();
            const int4 d = waves[w];
            const AnalysisParams p = P[d.x];
            direct_node<N>(p, nodes, d.y, d.z, gout);
        }
    }
}

// ---------------------------------------------------------------------------
// ensemble route
// ---------------------------------------------------------------------------
// Nodes node0 .. node0 + 3 (those < nx * ny), M <= N <= 32 members, lane r of a row =
// members r and r + 16.
template <int N, typename T>
__device__ __forceinline__ void ens_direct_body(const AnalysisParams& p, int node0) {
    constexpr int NS = Direct<N>::NS;
    extern __shared__ double lds[];
    T* __restrict__ fs = reinterpret_cast<T*>(p.f);
    const int lane = threadIdx.x;
    const int seg = lane >> 4, r = lane & 15;
    const int nx = p.nx, ny = p.ny, M = p.members;
    const int plane = nx * ny;
    const int node = node0 + seg;
    const bool here = node < plane;
    int mi[NS];
    bool mem[NS];
#pragma unroll
    for (int h = 0; h < NS; ++h) {
        mem[h] = here && r + 16 * h < M;
        mi[h] = r + 16 * h < M ? r + 16 * h : 0;
    }
    // S = Z^T Z and Z^T d~, eight observations at a time: lane r < 8 of the row looks
    // observation j0 + r up, every lane loads its members' perturbations of all eight
    double A[NS][N], b[NS];
#pragma unroll
    for (int h = 0; h < NS; ++h) {
        b[h] = 0.0;
#pragma unroll
        for (int j = 0; j < N; ++j) A[h][j] = 0.0;
    }
    const int nz = p.nvar * p.lmax;
#pragma unroll 1
    for (int j0 = 0; j0 < nz; j0 += 8) {
        int q = 0;
        double w = 0.0, d = 0.0;
        if (here && r < 8) local_obs(p, node, j0 + r, &q, &w, &d);
        if (!__any(w != 0.0)) continue;
        double y[8][NS];
        auto load = [&](auto self, auto K) -> void {
            constexpr int k = decltype(K)::value;
            const int qk = __builtin_amdgcn_mov_dpp(q, 0x150 + k, 0xF, 0xF, true);
#pragma unroll
            for (int h = 0; h < NS; ++h) y[k][h] = p.dY[(size_t)qk * M + mi[h]];
            if constexpr (k < 7) self(self, std::integral_constant<int, k + 1>());
        };
        load(load, std::integral_constant<int, 0>());
        auto add = [&](auto self, auto K) -> void {
            constexpr int k = decltype(K)::value;
            const double wk = row_bcast<k>(w), dk = row_bcast<k>(d);
            double z[NS];
#pragma unroll
            for (int h = 0; h < NS; ++h) {
                z[h] = mem[h] && wk != 0.0 ? wk * y[k][h] : 0.0;
                if (wk != 0.0) b[h] = fma(z[h], dk, b[h]);
            }
#pragma unroll
            for (int h = 0; h < NS; ++h) row_axpy<N, NS>(A[h], z, z[h]);
            if constexpr (k < 7) self(self, std::integral_constant<int, k + 1>());
        };
        add(add, std::integral_constant<int, 0>());
    }
    const double ia = 1.0 / p.a;
    const ReflLds vs{lds + 4 * Direct<N>::kNodeDoubles + seg * ReflLds::doubles(N)};
    const bool finite = sym_direct<N, true>(A, b, ia, p.sqrt_beta, lds, vs, lane);
    count_failed<16>(here && !finite, p.eig_fail, lane);

    // the populations, read only now: nothing above needs them, and they would hold
    // 18 registers per member slot through the solver
    const int x = here ? node % nx : 0, y = here ? node / nx : 0;
    double f[NS][9];
#pragma unroll
    for (int a = 0; a < 9; ++a)
#pragma unroll
        for (int h = 0; h < NS; ++h)
            f[h][a] = PopIO<T>::load(fs + slot(src_node(x, y, a, nx, ny), a, mi[h], M), a);
#pragma unroll
    for (int h = 0; h < NS; ++h)
#pragma unroll
        for (int a = 0; a < 9; ++a) f[h][a] = mem[h] ? f[h][a] : 0.0;
    if (p.diag_node)
        row_diag_record<NS>(f, mem, M, node, plane, p.truth_uv,
                            p.diag_node + (size_t)(here ? node : 0) * kDiagFieldCount, here, r);
#pragma unroll
    for (int a = 0; a < 9; ++a) {
        double s = 0.0, wm = 0.0;
#pragma unroll
        for (int h = 0; h < NS; ++h) s += f[h][a];
        const double xbar = row_sum(s) / M;
        double dx[NS];
#pragma unroll
        for (int h = 0; h < NS; ++h) {
            dx[h] = mem[h] ? f[h][a] - xbar : 0.0;
            wm = fma(dx[h], b[h] * ia, wm);
        }
        const double xm = xbar + row_sum(wm);
#pragma unroll
        for (int h = 0; h < NS; ++h) {
            const double v = xm + row_dot<N, NS>(A[h], dx);
            if (mem[h]) PopIO<T>::store(fs + slot(src_node(x, y, a, nx, ny), a, mi[h], M), a, v);
            f[h][a] = mem[h] ? PopIO<T>::round(v, a) : 0.0;
        }
    }
    if (p.diag_node)
        row_diag_record<NS>(f, mem, M, node, plane, p.truth_uv,
                            p.diag_node + (size_t)(plane + (here ? node : 0)) * kDiagFieldCount,
                            here, r);
}

// One node, 32 < M <= N <= 64 members, lane = member.
template <int N, typename T>
__device__ __forceinline__ void ens_direct_wave(const AnalysisParams& p, int node) {
    constexpr int NS = DirectW<N>::NS;
    extern __shared__ double lds[];
    T* __restrict__ fs = reinterpret_cast<T*>(p.f);
    const int lane = threadIdx.x;
    const int r = lane & 15;
    const int nx = p.nx, ny = p.ny, M = p.members;
    const int plane = nx * ny;
    const bool mem = lane < M;
    const int ml = mem ? lane : 0;
    double A[NS][16], b = 0.0;
#pragma unroll
    for (int h = 0; h < NS; ++h)
#pragma unroll
        for (int k = 0; k < 16; ++k) A[h][k] = 0.0;
    const int nz = p.nvar * p.lmax;
#pragma unroll 1
    for (int j0 = 0; j0 < nz; j0 += kWave) {
        int q = 0;
        double w = 0.0, d = 0.0;
        local_obs(p, node, j0 + lane, &q, &w, &d);
        const int left = min(kWave, nz - j0);
        for (int k = 0; k < left; ++k) {
            const double wk = lane_value(w, k);
            if (wk == 0.0) continue;  // uniform over the wavefront
            const double* yrow = p.dY + (size_t)__builtin_amdgcn_readlane(q, k) * M;
            const double yl = yrow[ml];
            double zr[NS];
#pragma unroll
            for (int h = 0; h < NS; ++h) zr[h] = yrow[16 * h + r < M ? 16 * h + r : 0];
            const double z = mem ? wk * yl : 0.0;
            b = fma(z, lane_value(d, k), b);
#pragma unroll
            for (int h = 0; h < NS; ++h)
                fmac_axpy<0, 16>(A[h], z, 16 * h + r < M ? wk * zr[h] : 0.0);
        }
    }
    const double ia = 1.0 / p.a;
    const ReflLds vs{lds + DirectW<N>::kDoubles};
    const bool finite = sym_direct_wave<N, true>(A, b, ia, p.sqrt_beta, lds, vs, lane);
    if (!finite && lane == 0) atomicAdd(p.eig_fail, 1);

    const int x = node % nx, y = node / nx;
    double f[9];
#pragma unroll
    for (int a = 0; a < 9; ++a)
        f[a] = PopIO<T>::load(fs + slot(src_node(x, y, a, nx, ny), a, ml, M), a);
#pragma unroll
    for (int a = 0; a < 9; ++a) f[a] = mem ? f[a] : 0.0;
    if (p.diag_node)
        node_diag_record(f, mem, M, node, plane, p.truth_uv,
                         p.diag_node + (size_t)node * kDiagFieldCount);
    double* part = lds + 3 * DirectW<N>::kTab + 64;
#pragma unroll 1
    for (int a = 0; a < 9; ++a) {
        double fa = 0.0;
#pragma unroll
        for (int c = 0; c < 9; ++c) fa = a == c ? f[c] : fa;
        const double xbar = wave_sum(fa) / M;
        const double dx = mem ? fa - xbar : 0.0;
        const double v = xbar + wave_sum(dx * (b * ia)) + wave_matvec<NS, NS, NS, 16>(A, dx, part, lane);
#pragma unroll
        for (int c = 0; c < 9; ++c) f[c] = a == c ? v : f[c];
    }
    double xa[9];
#pragma unroll
    for (int a = 0; a < 9; ++a) {
        xa[a] = 0.0;
        if (mem) {
            PopIO<T>::store(fs + slot(src_node(x, y, a, nx, ny), a, lane, M), a, f[a]);
            xa[a] = PopIO<T>::round(f[a], a);
        }
    }
    if (p.diag_node)
        node_diag_record(xa, mem, M, node, plane, p.truth_uv,
                         p.diag_node + ((size_t)plane + node) * kDiagFieldCount);
}

template <int N, typename T>
__device__ __forceinline__ void ens_direct_node(const AnalysisParams& p, int node0) {
    if (node0 >= p.nx * p.ny) return;  // uniform over the wavefront
    if constexpr (N == 8) {
        // (half the size for ensembles of up to four members)
        if (p.members <= 4) ens_direct_body<4, T>(p, node0);
        else ens_direct_body<8, T>(p, node0);
    } else if constexpr (kRows16<N>) ens_direct_body<N, T>(p, node0);
    else ens_direct_wave<N, T>(p, node0);
}

template <int N>
constexpr int ens_direct_segs() { return kRows16<N> ? 4 : 1; }

template <int N>
constexpr size_t ens_direct_lds_bytes() {
    if constexpr (kRows16<N>)
        return 4 * (Direct<N>::kNodeDoubles + ReflLds::doubles(N)) * sizeof(double);
    else
        return (DirectW<N>::kDoubles + ReflLds::doubles(N)) * sizeof(double);
}

template <int N, typename T>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(direct_waves<N>())))
void analysis_ens_direct_kernel(AnalysisParams p) {
    ens_direct_node<N, T>(p, xcd_remap(blockIdx.x, gridDim.x) * ens_direct_segs<N>());
}

template <int N, typename T>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(direct_waves<N>())))
void analysis_ens_direct_batch_kernel(const AnalysisParams* P, const int2* waves, int nwaves) {
    const int w = xcd_remap(blockIdx.x, gridDim.x);
    if (w >= nwaves) return;
    const int2 d = waves[w];  // (problem, first node)
    ens_direct_node<N, T>(P[d.x], d.y);
}

// ---------------------------------------------------------------------------
// launches
// ---------------------------------------------------------------------------
template <int N>
hipError_t launch_direct_n(const AnalysisParams& p, const int* nodes, int count, double* gbuf,
                           hipStream_t s) {
    constexpr int segs = direct_segs<N>();
    analysis_direct_kernel<N><<<(count + segs - 1) / segs, 64, direct_lds_bytes<N>(), s>>>(
        p, nodes, count, gbuf);
    return hipGetLastError();
}

template <int N>
hipError_t launch_direct_batch_n(const AnalysisParams* P, const int4* waves, int n, const int* nodes,
                                 double* gbuf, int* counters, hipStream_t s) {
    if (counters)
        analysis_direct_queue_kernel<N><<<persistent_blocks(64, n), 64, direct_lds_bytes<N>(), s>>>(
            P, waves, n, nodes, gbuf, counters);
    else
        analysis_direct_batch_kernel<N><<<n, 64, direct_lds_bytes<N>(), s>>>(P, waves, n, nodes,
                                                                             gbuf);
    return hipGetLastError();
}

template <int N, typename T>
hipError_t launch_ens_direct_t(const AnalysisParams& p, hipStream_t s) {
    constexpr int segs = ens_direct_segs<N>();
    analysis_ens_direct_kernel<N, T><<<(p.nx * p.ny + segs - 1) / segs, 64,
                                       ens_direct_lds_bytes<N>(), s>>>(p);
    return hipGetLastError();
}

template <int N, typename T>
hipError_t launch_ens_direct_batch_t(const AnalysisParams* P, const int2* waves, int n,
                                     hipStream_t s) {
    analysis_ens_direct_batch_kernel<N, T><<<n, 64, ens_direct_lds_bytes<N>(), s>>>(P, waves, n);
    return hipGetLastError();
}

}  // namespace

#define LBMLETKF_OBS_SIZES(X) X(8) X(10) X(12) X(14) X(16) X(18) X(20) X(22) X(24) X(26) \
    X(28) X(30) X(32) X(40) X(48) X(56) X(64)
#define LBMLETKF_ENS_SIZES(X) X(8) X(16) X(24) X(32) X(48) X(64)

int direct_segments(int n) { return n <= 32 ? 4 : (n <= 48 ? 2 : 1); }

hipError_t launch_eig_direct(const AnalysisParams& p, const int* nodes, int count, int n,
                             double* gbuf, hipStream_t s) {
    switch (n) {
#define X(v) case v: return launch_direct_n<v>(p, nodes, count, gbuf, s);
        LBMLETKF_OBS_SIZES(X)
#undef X
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_eig_direct_batch(const AnalysisParams* d_params, const int4* d_eig_waves,
                                   int n_eig, const int* d_nodes, int n, double* gbuf,
                                   int* counters, hipStream_t s) {
    switch (n) {
#define X(v)                                                                               \
    case v:                                                                                \
        return launch_direct_batch_n<v>(d_params, d_eig_waves, n_eig, d_nodes, gbuf, counters, s);
        LBMLETKF_OBS_SIZES(X)
#undef X
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_ens_direct(const AnalysisParams& p, int n, hipStream_t s) {
    switch (n) {
#define X(v)                                                              \
    case v:                                                               \
        return p.storage == kStoreF32Dev ? launch_ens_direct_t<v, float>(p, s) \
                                         : launch_ens_direct_t<v, double>(p, s);
        LBMLETKF_ENS_SIZES(X)
#undef X
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_ens_direct_batch(const AnalysisParams* d_params, const int2* d_waves, int nwaves,
                                   int n, int storage, hipStream_t s) {
    if (nwaves == 0) return hipSuccess;
    switch (n) {
#define X(v)                                                                              \
    case v:                                                                               \
        return storage == kStoreF32Dev                                                    \
                   ? launch_ens_direct_batch_t<v, float>(d_params, d_waves, nwaves, s)    \
                   : launch_ens_direct_batch_t<v, double>(d_params, d_waves, nwaves, s);
        LBMLETKF_ENS_SIZES(X)
#undef X
        default: return hipErrorInvalidValue;
    }
}

}  // namespace lbmletkf
