// Forecast kernels: the D2Q9 lattice Boltzmann equation with BGK relaxation,
// Smagorinsky eddy viscosity and a body force (Sec. 2), advanced for every
// ensemble member in one launch (one step, or two steps on spatial tiles).
//
// Layout: f[node][a][member], node = y * nx + x, members fastest (FP64, or
// FP32 deviations).  One thread per (node, member), a block of
// (members x nodes) threads.  The kernels pull: the thread of node (x, y)
// gathers f_a from the slot of node (x - c_ax, y - c_ay), which holds the
// pre-collision population f_a(x, y, t), collides, and writes f*_a to its own
// slot (node, a).  Between steps a buffer therefore holds post-collision
// values, and the canonical f_a(x, y) lives at the slot of node
// (x - c_ax, y - c_ay); import/export convert.  With 64 members every load
// and store of a wavefront is 512 contiguous, aligned bytes.
//
// Relaxation time: the strain rate is taken from the local non-equilibrium
// momentum flux Pi = sum_a c_a c_a (f_a - f_a^eq) through the Chapman-Enskog
// relation S = -3 Pi / (2 rho tau); with nu + nu_SGS = (tau - 1/2)/3 and
// nu_SGS = C_s^2 |S| (Sec. 2) tau solves
//     tau^2 - tau0 tau - 9 sqrt(2) C_s^2 |Pi| / (2 rho) = 0,
// |Pi| = sqrt(Pi_xx^2 + Pi_yy^2 + 2 Pi_xy^2), whose positive root is used.
// The momentum flux of f^eq is rho/3 I + rho u u, so Pi needs no f^eq.
#include <algorithm>

#include "common.h"
#include "device_util.h"

namespace lbmletkf {
namespace {

constexpr int kBlock = 256;

__device__ __forceinline__ int wrap_dec(int i, int n) { return i == 0 ? n - 1 : i - 1; }
__device__ __forceinline__ int wrap_inc(int i, int n) { return i == n - 1 ? 0 : i + 1; }

// c_a . (x, y) for the D2Q9 velocity a (a constant after unrolling) as the one
// addition or sign change it needs: a multiplication by 0 or +-1 would cost an
// instruction and, without fast-math, is not dropped by the compiler.
__device__ __forceinline__ double cdot(int a, double x, double y) {
    const int cx = cx_of(a), cy = cy_of(a);
    const double tx = cx > 0 ? x : (cx < 0 ? -x : 0.0);
    if (cy == 0) return tx;
    if (cx == 0) return cy > 0 ? y : -y;
    return cy > 0 ? tx + y : tx - y;
}

// Relax one node: f[9] in (pre-collision), f*[9] out.  The multiply-adds are
// written out as fma() and the compiler may fuse nothing else, so the result
// does not depend on the code the function is inlined into: the one-step and
// the two-step kernels give the same bits.
__device__ __forceinline__ void collide_node(double (&f)[9], double tau0, double smag,
                                             double fx_ext, double fy_ext, double mu) {
#pragma clang fp contract(off)
    const double rho = ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7])) + f[8];
    const double jx = (f[1] - f[2]) + (f[5] - f[6]) + (f[7] - f[8]);
    const double jy = (f[3] - f[4]) + (f[5] - f[6]) + (f[8] - f[7]);
    const double inv_rho = 1.0 / rho;
    const double u = jx * inv_rho, v = jy * inv_rho;
    const double uu = u * u, vv = v * v, uv = u * v;
    // non-equilibrium momentum flux: sum c c f - rho/3 I - rho u u
    const double pxx = fma(-rho, 1.0 / 3.0 + uu, f[1] + f[2] + f[5] + f[6] + f[7] + f[8]);
    const double pyy = fma(-rho, 1.0 / 3.0 + vv, f[3] + f[4] + f[5] + f[6] + f[7] + f[8]);
    const double pxy = fma(-rho, uv, f[5] + f[6] - f[7] - f[8]);
    const double pn = sqrt(fma(pxx, pxx, fma(pyy, pyy, (2.0 * pxy) * pxy)));
    const double tau = 0.5 * (tau0 + sqrt(fma(tau0, tau0, (smag * pn) * inv_rho)));
    const double omega = 1.0 / tau;
    // acceleration: external field plus linear friction
    const double gx = fma(-mu, u, fx_ext), gy = fma(-mu, v, fy_ext);
    const double one_usq = 1.0 - 1.5 * (uu + vv);
#pragma unroll
    for (int a = 0; a < 9; ++a) {
        const double cu = cdot(a, u, v);
        // f^eq = rho w (1 + 3 cu + 4.5 cu^2 - 1.5 u.u)
        const double feq = (rho * w_of(a)) * fma(cu, fma(4.5, cu, 3.0), one_usq);
        const double Fa = (3.0 * w_of(a) * rho) * cdot(a, gx, gy);
        f[a] = fma(-omega, f[a] - feq, f[a] + Fa);
    }
}

// The same relaxation in FP32 on the deviations g_a = f_a - w_a that FP32
// storage keeps (the precision form): the lattice sums of the weights are
// exact constants (sum w = 1, sum w c = 0, sum w c c = I/3), so every moment
// is a sum of small numbers, rho = 1 + sum g,
//   Pi_xx = sum c_x^2 g - (rho - 1)/3 - rho u^2,  Pi_xy = sum c_x c_y g - rho u v,
//   g^eq_a = w_a [(rho - 1) + rho (3 cu + 4.5 cu^2 - 1.5 u.u)],
// and FP32 keeps ~7 significant digits of quantities of size |g| <~ 0.02.
__device__ __forceinline__ float cdotf(int a, float x, float y) {
    const int cx = cx_of(a), cy = cy_of(a);
    const float tx = cx > 0 ? x : (cx < 0 ? -x : 0.0f);
    if (cy == 0) return tx;
    if (cx == 0) return cy > 0 ? y : -y;
    return cy > 0 ? tx + y : tx - y;
}

__device__ __forceinline__ void collide_node_dev(float (&g)[9], float tau0, float smag,
                                                 float fx_ext, float fy_ext, float mu) {
#pragma clang fp contract(off)
    const float drho = ((g[0] + g[1]) + (g[2] + g[3])) + ((g[4] + g[5]) + (g[6] + g[7])) + g[8];
    const float rho = 1.0f + drho;
    const float jx = (g[1] - g[2]) + (g[5] - g[6]) + (g[7] - g[8]);
    const float jy = (g[3] - g[4]) + (g[5] - g[6]) + (g[8] - g[7]);
    // 1 / rho: the hardware reciprocal (1 ulp) refined by one Newton step, three
    // instructions instead of the correctly rounded division's ten (the bare
    // reciprocal biases u enough to move a 200-step misfit by 4e-6 relative);
    // the square roots below are the hardware ones (|Pi| and R only need their
    // own relative accuracy)
    float inv_rho = __builtin_amdgcn_rcpf(rho);
    inv_rho = fmaf(inv_rho, fmaf(-rho, inv_rho, 1.0f), inv_rho);
    const float u = jx * inv_rho, v = jy * inv_rho;
    const float uu = u * u, vv = v * v, uv = u * v;
    const float d3 = drho * (1.0f / 3.0f);
    const float pxx = fmaf(-rho, uu, (g[1] + g[2] + g[5] + g[6] + g[7] + g[8]) - d3);
    const float pyy = fmaf(-rho, vv, (g[3] + g[4] + g[5] + g[6] + g[7] + g[8]) - d3);
    const float pxy = fmaf(-rho, uv, g[5] + g[6] - g[7] - g[8]);
    const float pn = __builtin_amdgcn_sqrtf(fmaf(pxx, pxx, fmaf(pyy, pyy, (2.0f * pxy) * pxy)));
    // omega = 1 / tau = 2 / (tau0 + R), R = sqrt(tau0^2 + x), x = 18 sqrt(2) C_s^2 |Pi| / rho,
    // taken as the molecular 1 / tau0 minus the eddy part x / (tau0 (tau0 + R)^2),
    // which FP32 then carries to its own relative accuracy (as 1 / tau the eddy
    // part, often 1e-4 of omega, would keep only a few bits)
    const float x = (smag * pn) * inv_rho;
    const float tr = tau0 + __builtin_amdgcn_sqrtf(fmaf(tau0, tau0, x));
    const float omega = 1.0f / tau0 - x * __builtin_amdgcn_rcpf(tau0 * tr * tr);
    const float gx = fmaf(-mu, u, fx_ext), gy = fmaf(-mu, v, fy_ext);
    const float usq = -1.5f * (uu + vv);
#pragma unroll
    for (int a = 0; a < 9; ++a) {
        const float w = (float)w_of(a);
        const float cu = cdotf(a, u, v);
        const float geq = w * fmaf(rho, fmaf(cu, fmaf(4.5f, cu, 3.0f), usq), drho);
        const float Fa = (3.0f * w * rho) * cdotf(a, gx, gy);
        g[a] = fmaf(-omega, g[a] - geq, g[a] + Fa);
    }
}

// V consecutive members per thread: FP32 deviations move 4 bytes per member,
// and one 8-byte access per population for two members keeps the wavefront's
// requests as wide as in FP64.
typedef float float2v __attribute__((ext_vector_type(2)));

// Pull, collide and store one node for members m .. m + V - 1.
template <typename T, int V>
__device__ __forceinline__ void lbm_update(const T* __restrict__ fin, T* __restrict__ fout,
                                           const double* __restrict__ force, int nx, int ny,
                                           int members, int node, int m, double tau0,
                                           double smag, double mu) {
    static_assert(V == 1 || (V == 2 && sizeof(T) == 4), "two members per thread: FP32 only");
    const int plane = nx * ny;
    const int y = node / nx, x = node - y * nx;
    const int xm = wrap_dec(x, nx), xp = wrap_inc(x, nx);
    const int ym = wrap_dec(y, ny), yp = wrap_inc(y, ny);
    // slots holding the canonical f_a(x, y): node (x - c_ax, y - c_ay)
    const PullSlots<const T> src(fin, x, xm, xp, y, ym, yp, nx, members, m);
    T* const dst = fout + (size_t)node * 9 * members + m;
    double fx = 0.0, fy = 0.0;
    if (force) {
        fx = force[node];
        fy = force[plane + node];
    }
    // every population is read once and written once per step: stream it
    // past the caches (nontemporal loads and stores)
    if constexpr (sizeof(T) == 8) {
        double f[9];
#pragma unroll
        for (int a = 0; a < 9; ++a) f[a] = PopIO<T>::load_nt(src.at(a), a);
        collide_node(f, tau0, smag, fx, fy, mu);
#pragma unroll
        for (int a = 0; a < 9; ++a) PopIO<T>::store_nt(dst + (uint32_t)a * members, a, f[a]);
    } else {
        // FP32 deviations: the FP32 relaxation on g = f - w, no conversion
        float g[V][9];
        if constexpr (V == 1) {
#pragma unroll
            for (int a = 0; a < 9; ++a)
                g[0][a] = __builtin_nontemporal_load(src.at(a));
        } else {
#pragma unroll
            for (int a = 0; a < 9; ++a) {
                const float2v p = __builtin_nontemporal_load(
                    reinterpret_cast<const float2v*>(src.at(a)));
                g[0][a] = p.x;
                g[1][a] = p.y;
            }
        }
#pragma unroll
        for (int k = 0; k < V; ++k)
            collide_node_dev(g[k], (float)tau0, (float)smag, (float)fx, (float)fy, (float)mu);
        if constexpr (V == 1) {
#pragma unroll
            for (int a = 0; a < 9; ++a)
                __builtin_nontemporal_store(g[0][a], dst + (uint32_t)a * members);
        } else {
#pragma unroll
            for (int a = 0; a < 9; ++a) {
                float2v p;
                p.x = g[0][a];
                p.y = g[1][a];
                __builtin_nontemporal_store(p, reinterpret_cast<float2v*>(dst + (uint32_t)a * members));
            }
        }
    }
}

// Members per thread of the forecast kernels: 2 for FP32 storage with an even
// ensemble, else 1 (the single and the batched step use the same choice, so
// they round identically).
__host__ __device__ constexpr int members_per_thread(int elem_bytes, int members) {
    return (elem_bytes == 4 && members % 2 == 0) ? 2 : 1;
}

template <typename T, int V>
__global__ __launch_bounds__(kBlock) void stream_collide_kernel(
    const T* __restrict__ fin, T* __restrict__ fout, const double* __restrict__ force, int nx,
    int ny, int members, double tau0, double smag, double mu) {
    const int node = blockIdx.x * blockDim.y + threadIdx.y;
    if (node >= nx * ny) return;
    lbm_update<T, V>(fin, fout, force, nx, ny, members, node, threadIdx.x * V, tau0, smag, mu);
}

// Many problems in one persistent launch: blocks of 256 threads walk the
// concatenated tile list (problem k owns tiles [tile0_k, tile0_{k+1})); a
// tile is `tile_nodes` consecutive nodes of one problem, processed as rows of
// (256 / M) nodes x M members.  The schedule is static (block b takes tiles
// b, b + gridDim.x, ...), so every launch does the same work in the same order.
template <typename T>
__global__ __launch_bounds__(kBlock) void stream_collide_batch_kernel(const LbmTask* __restrict__ tasks,
                                                                      int ntasks, int ntiles) {
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        int k = 0;
        while (k + 1 < ntasks && tasks[k + 1].tile0 <= t) ++k;
        const LbmTask& tk = tasks[k];
        const int M = tk.members;
        const int V = members_per_thread((int)sizeof(T), M);
        const int tpn = M / V;  // threads per node
        const int npb = kBlock / tpn;
        const int plane = tk.nx * tk.ny;
        const int node0 = (t - tk.tile0) * tk.tile_nodes;
        const int m = (threadIdx.x % tpn) * V, nl = threadIdx.x / tpn;
        if (nl >= npb) continue;
        for (int r = nl; r < tk.tile_nodes; r += npb) {
            const int node = node0 + r;
            if (node >= plane) break;
            if (V == 2)
                lbm_update<T, members_per_thread((int)sizeof(T), 2)>(
                    static_cast<const T*>(tk.fin), static_cast<T*>(tk.fout), tk.force, tk.nx,
                    tk.ny, M, node, m, tk.tau0, tk.smag, tk.mu);
            else
                lbm_update<T, 1>(static_cast<const T*>(tk.fin), static_cast<T*>(tk.fout), tk.force,
                                 tk.nx, tk.ny, M, node, m, tk.tau0, tk.smag, tk.mu);
        }
    }
}

// Two steps per launch on spatial tiles.  A block takes kTwoMG members of a
// kTwoT x kTwoT tile of nodes: its first step covers the tile and a one-node
// ring around it (kTwoR x kTwoR nodes, one thread per node and member, exactly
// the single step's arithmetic on the same inputs) and keeps the results in
// LDS, rounded as a store and reload would round them; its second step pulls
// from there for the tile's nodes and writes them.  HBM traffic per two steps
// is kTwoR^2 / kTwoT^2 reads plus one write of the tile instead of two reads
// and two writes (0.69x for 6 x 6 tiles).
constexpr int kTwoMG = 16;
constexpr int kTwoT = 6;
constexpr int kTwoR = kTwoT + 2;

__host__ __device__ constexpr int two_step_lds_doubles() { return kTwoR * kTwoR * 9 * kTwoMG; }

// Block b of a two-step launch over one problem (FP64 storage): member group
// b % (members / kTwoMG) of tile b / (members / kTwoMG).
__device__ __forceinline__ void two_step_body(const double* __restrict__ fin,
                                              double* __restrict__ fout,
                                              const double* __restrict__ force, int nx, int ny,
                                              int members, double tau0, double smag, double mu,
                                              int b, double* __restrict__ fmid) {
    extern __shared__ double mid[];  // [kTwoR * kTwoR][9][kTwoMG]
    using T = double;
    const int groups = members / kTwoMG;
    const int tiles_x = (nx + kTwoT - 1) / kTwoT;
    const int mg = b % groups, tile = b / groups;
    const int x0 = (tile % tiles_x) * kTwoT, y0 = (tile / tiles_x) * kTwoT;
    const int m = mg * kTwoMG + threadIdx.x;
    const int r = threadIdx.y, rx = r % kTwoR, ry = r / kTwoR;
    // this thread's region node, periodic (a ragged edge tile computes a few
    // nodes nobody reads)
    const int gx = (x0 - 1 + rx + nx) % nx, gy = (y0 - 1 + ry + ny) % ny;
    const int plane = nx * ny;
    const int node = gy * nx + gx;
    double fx = 0.0, fy = 0.0;
    if (force) {
        fx = force[node];
        fy = force[plane + node];
    }
    const PullSlots<const T> src(fin, gx, wrap_dec(gx, nx), wrap_inc(gx, nx), gy, wrap_dec(gy, ny),
                                 wrap_inc(gy, ny), nx, members, m);
    const size_t own_slot = (size_t)node * 9 * members + m;
    // first step: the single step's pull and collision
    double f[9];
#pragma unroll
    for (int a = 0; a < 9; ++a) f[a] = PopIO<T>::load_nt(src.at(a), a);
    collide_node(f, tau0, smag, fx, fy, mu);
#pragma unroll
    for (int a = 0; a < 9; ++a) mid[(r * 9 + a) * kTwoMG + threadIdx.x] = PopIO<T>::round(f[a], a);
    const int ix = rx - 1, iy = ry - 1;
    const bool own = ix >= 0 && ix < kTwoT && iy >= 0 && iy < kTwoT && x0 + ix < nx && y0 + iy < ny;
    // the first step's state of the tile's own nodes, when asked for
    if (fmid && own) {
#pragma unroll
        for (int a = 0; a < 9; ++a)
            PopIO<T>::store_nt(fmid + own_slot + (uint32_t)a * members, a, f[a]);
    }
    __syncthreads();
    // second step for the tile's own nodes
    if (!own) return;
#pragma unroll
    for (int a = 0; a < 9; ++a)
        f[a] = mid[(((ry - cy_of(a)) * kTwoR + rx - cx_of(a)) * 9 + a) * kTwoMG + threadIdx.x];
    collide_node(f, tau0, smag, fx, fy, mu);
#pragma unroll
    for (int a = 0; a < 9; ++a) PopIO<T>::store_nt(fout + own_slot + (uint32_t)a * members, a, f[a]);
}

__global__ __launch_bounds__(kTwoMG * kTwoR * kTwoR) void stream_collide2_kernel(
    const double* __restrict__ fin, double* __restrict__ fout, const double* __restrict__ force,
    int nx, int ny, int members, double tau0, double smag, double mu, double* __restrict__ fmid) {
    two_step_body(fin, fout, force, nx, ny, members, tau0, smag, mu, blockIdx.x, fmid);
}

// The two-step kernel for FP32 storage: the FP32 relaxation on deviations
// (collide_node_dev), MG members per block as MG / 2 threads of two adjacent
// members each (8-byte accesses, as in the single step), the intermediate
// deviations kept in LDS as FP32 -- exactly the values a single step would
// store -- so that a launch equals two single-step launches bit for bit.
// Block b of a two-step launch over one problem (FP32 storage) holds MG / gsize units of
// gsize members; unit u is member group u % (members / gsize) of tile u / (members / gsize).
// (A batch runs ensembles that 32 does not divide as two units of 16 per block; with one,
// half of each block's threads idled: batch of 128^2 x 16, 128^2 x 32, 192^2 x 16, 192^2 x 64,
// us per launch 87 -> 82.)
template <int MG>
__device__ __forceinline__ void two_step_dev_body(const float* __restrict__ fin,
                                                  float* __restrict__ fout,
                                                  const double* __restrict__ force, int nx, int ny,
                                                  int members, float tau0, float smag, float mu,
                                                  int b, int gsize, float* __restrict__ fmid) {
    extern __shared__ float mids[];  // [kTwoR * kTwoR][9][MG]
    typedef float f2 __attribute__((ext_vector_type(2)));
    const int groups = members / gsize;
    const int tiles_x = (nx + kTwoT - 1) / kTwoT;
    const int units = tiles_x * ((ny + kTwoT - 1) / kTwoT) * groups;
    const int mp = 2 * threadIdx.x;          // first member of the pair within the block
    // a block of one unit (uniform: its divisions stay on the scalar unit; per thread they cost
    // a single problem's launch 6% at 68^2 x 64) or of several
    int mg = b % groups, tile = b / groups, m = mp;
    bool on = true;
    if (gsize != MG) {
        const int u = b * (MG / gsize) + mp / gsize;
        on = u < units;  // (the last block may hold one unit)
        mg = on ? u % groups : 0;
        tile = on ? u / groups : 0;
        m = mp % gsize;
    }
    m += mg * gsize;
    const int x0 = (tile % tiles_x) * kTwoT, y0 = (tile / tiles_x) * kTwoT;
    const int r = threadIdx.y, rx = r % kTwoR, ry = r / kTwoR;
    const int gx = (x0 - 1 + rx + nx) % nx, gy = (y0 - 1 + ry + ny) % ny;
    const int plane = nx * ny;
    const int node = gy * nx + gx;
    float fx = 0.0f, fy = 0.0f;
    if (force) {
        fx = (float)force[node];
        fy = (float)force[plane + node];
    }
    const PullSlots<const float> src(fin, gx, wrap_dec(gx, nx), wrap_inc(gx, nx), gy,
                                     wrap_dec(gy, ny), wrap_inc(gy, ny), nx, members, m);
    const size_t own_slot = (size_t)node * 9 * members + m;
    float g0[9], g1[9];
#pragma unroll
    for (int a = 0; a < 9; ++a) {
        const f2 v = __builtin_nontemporal_load(reinterpret_cast<const f2*>(src.at(a)));
        g0[a] = v.x;
        g1[a] = v.y;
    }
    collide_node_dev(g0, tau0, smag, fx, fy, mu);
    collide_node_dev(g1, tau0, smag, fx, fy, mu);
#pragma unroll
    for (int a = 0; a < 9; ++a) {
        f2 v;
        v.x = g0[a];
        v.y = g1[a];
        *reinterpret_cast<f2*>(mids + (r * 9 + a) * MG + mp) = v;
    }
    const int ix = rx - 1, iy = ry - 1;
    const bool own = on && ix >= 0 && ix < kTwoT && iy >= 0 && iy < kTwoT && x0 + ix < nx &&
                     y0 + iy < ny;
    // the first step's state of the tile's own nodes, when asked for
    if (fmid && own) {
#pragma unroll
        for (int a = 0; a < 9; ++a) {
            f2 v;
            v.x = g0[a];
            v.y = g1[a];
            __builtin_nontemporal_store(
                v, reinterpret_cast<f2*>(fmid + own_slot + (uint32_t)a * members));
        }
    }
    __syncthreads();
    if (!own) return;
#pragma unroll
    for (int a = 0; a < 9; ++a) {
        const f2 v = *reinterpret_cast<const f2*>(
            mids + (((ry - cy_of(a)) * kTwoR + rx - cx_of(a)) * 9 + a) * MG + mp);
        g0[a] = v.x;
        g1[a] = v.y;
    }
    collide_node_dev(g0, tau0, smag, fx, fy, mu);
    collide_node_dev(g1, tau0, smag, fx, fy, mu);
#pragma unroll
    for (int a = 0; a < 9; ++a) {
        f2 v;
        v.x = g0[a];
        v.y = g1[a];
        __builtin_nontemporal_store(v, reinterpret_cast<f2*>(fout + own_slot + (uint32_t)a * members));
    }
}

template <int MG>
__global__ __launch_bounds__(MG / 2 * kTwoR * kTwoR) void stream_collide2_dev_kernel(
    const float* __restrict__ fin, float* __restrict__ fout, const double* __restrict__ force,
    int nx, int ny, int members, float tau0, float smag, float mu, float* __restrict__ fmid) {
    two_step_dev_body<MG>(fin, fout, force, nx, ny, members, tau0, smag, mu, blockIdx.x, MG, fmid);
}

// Two steps of many problems in one launch: block b belongs to the task k
// with block0_k <= b < block0_{k+1} (a problem's blocks are its tiles x member
// groups: 16 members for FP64 storage, 32 -- or two units of 16 where 32 does not divide M --
// for FP32 storage), and runs that problem's two-step block b - block0_k.
constexpr int kTwoMG32 = 32;  // members per block of the FP32 batched launch

template <typename T>
__global__ __launch_bounds__((sizeof(T) == 8 ? kTwoMG : kTwoMG32 / 2) * kTwoR * kTwoR) void
stream_collide2_batch_kernel(const LbmTask* __restrict__ tasks, int ntasks) {
    const int b = blockIdx.x;
    int k = 0;
    while (k + 1 < ntasks && tasks[k + 1].block0 <= b) ++k;
    const LbmTask& tk = tasks[k];
    if constexpr (sizeof(T) == 8)
        two_step_body(static_cast<const double*>(tk.fin), static_cast<double*>(tk.fout), tk.force,
                      tk.nx, tk.ny, tk.members, tk.tau0, tk.smag, tk.mu, b - tk.block0, nullptr);
    else
        two_step_dev_body<kTwoMG32>(static_cast<const float*>(tk.fin),
                                    static_cast<float*>(tk.fout), tk.force, tk.nx, tk.ny,
                                    tk.members, (float)tk.tau0, (float)tk.smag, (float)tk.mu,
                                    b - tk.block0, tk.members % kTwoMG32 == 0 ? kTwoMG32 : kTwoMG,
                                    nullptr);
}

// ---------------------------------------------------------------------------
// Several steps per launch on regions of any size and any member count: a block
// takes MG members of a region of RX x RY nodes, pulls the first step from HBM and keeps
// the results in LDS; each further step loses the region's outer ring, and after k steps
// the inner nodes (RX - 2 (k - 1) by RY - 2 (k - 1)) are written.  For ensembles that the 128-byte
// member blocks above do not fit, and for problems so small that a step's launch costs
// more than its work: 72 M bytes per node leave room for regions of 12-24 nodes, so that
// k = 3-6 steps cost one read of the region and one write of its inner nodes, one launch and k barriers.
// One thread holds I items (a node, V members) through all steps, LDS is updated in place
// between two barriers.  Same arithmetic and rounding as single steps, bit for bit.
// Bound by latency (a launch, one round of loads, k barriers) on small problems and by
// L2 requests of 32-byte pieces and FP64 issue on large ones (4.0 TB/s of the kernel's own
// bytes at 400^2 x 24).  Shapes: step_plans below.
// ---------------------------------------------------------------------------
template <typename T, int V, int I>
__global__ __launch_bounds__(1024) void stream_collide_tile_kernel(
    const T* __restrict__ fin, T* __restrict__ fout, const double* __restrict__ force, int nx,
    int ny, int members, double tau0, double smag, double mu, int RX, int RY, int MG,
    int steps,
    T* __restrict__ fmid, size_t mid_stride) {
    extern __shared__ char lds_raw[];
    T* const mid = reinterpret_cast<T*>(lds_raw);  // [9][RX * RY][MG]
    typedef T vec __attribute__((ext_vector_type(V)));
    const int halo = steps - 1, tile_x = RX - 2 * halo, tile_y = RY - 2 * halo;
    const int groups = (members + MG - 1) / MG;
    const int tiles_x = (nx + tile_x - 1) / tile_x;
    const int b = dev::xcd_remap(blockIdx.x, gridDim.x);  // the groups of a tile share lines
    const int t = b / groups, m0 = (b - t * groups) * MG;
    const int x0 = (t % tiles_x) * tile_x, y0 = (t / tiles_x) * tile_y;
    const int per = MG / V;  // items per node
    const int plane = nx * ny, rr = RX * RY;
    int rx[I], ry[I], m[I];
    bool on[I];
    size_t own[I];
    double fx[I], fy[I];
    T f[I][V][9];
#pragma unroll
    for (int i = 0; i < I; ++i) {
        const int it = threadIdx.x + i * blockDim.x;
        const int node_r = it / per;
        m[i] = (it - node_r * per) * V;
        ry[i] = node_r / RX;
        rx[i] = node_r - ry[i] * RX;
        on[i] = node_r < rr && m0 + m[i] < members;
        int gx = (x0 - halo + rx[i]) % nx, gy = (y0 - halo + ry[i]) % ny;
        gx = gx < 0 ? gx + nx : gx;
        gy = gy < 0 ? gy + ny : gy;
        const int node = gy * nx + gx;
        own[i] = (size_t)node * 9 * members + m0 + m[i];
        fx[i] = fy[i] = 0.0;
        if (!on[i]) continue;
        if (force) {
            fx[i] = force[node];
            fy[i] = force[plane + node];
        }
        const PullSlots<const T> src(fin, gx, wrap_dec(gx, nx), wrap_inc(gx, nx), gy,
                                     wrap_dec(gy, ny), wrap_inc(gy, ny), nx, members, m0 + m[i]);
#pragma unroll
        for (int a = 0; a < 9; ++a) {
            const vec v = *reinterpret_cast<const vec*>(src.at(a));
#pragma unroll
            for (int k = 0; k < V; ++k) f[i][k][a] = v[k];
        }
    }
    for (int s = 1;; ++s) {
        const int lo = s - 1, hx = RX - lo, hy = RY - lo;  // this step's nodes
#pragma unroll
        for (int i = 0; i < I; ++i) {
            on[i] = on[i] && rx[i] >= lo && rx[i] < hx && ry[i] >= lo && ry[i] < hy;
            if (!on[i]) continue;
#pragma unroll
            for (int k = 0; k < V; ++k) {
                if constexpr (sizeof(T) == 8)
                    collide_node(f[i][k], tau0, smag, fx[i], fy[i], mu);
                else
                    collide_node_dev(f[i][k], (float)tau0, (float)smag, (float)fx[i], (float)fy[i],
                                     (float)mu);
            }
            const bool inner = rx[i] >= halo && rx[i] < halo + tile_x && ry[i] >= halo &&
                               ry[i] < halo + tile_y && x0 + rx[i] - halo < nx &&
                               y0 + ry[i] - halo < ny;
            T* const dst = s == steps ? fout : (fmid ? fmid + (size_t)(s - 1) * mid_stride : nullptr);
            if (inner && dst) {
#pragma unroll
                for (int a = 0; a < 9; ++a) {
                    vec v;
#pragma unroll
                    for (int k = 0; k < V; ++k) v[k] = f[i][k][a];
                    *reinterpret_cast<vec*>(dst + own[i] + (uint32_t)a * members) = v;
                }
            }
        }
        if (s == steps) return;
        if (s > 1) __syncthreads();  // the previous step's values have been read
#pragma unroll
        for (int i = 0; i < I; ++i) {
            if (!on[i]) continue;
#pragma unroll
            for (int a = 0; a < 9; ++a) {
                vec v;
#pragma unroll
                for (int k = 0; k < V; ++k) v[k] = f[i][k][a];
                *reinterpret_cast<vec*>(mid + ((size_t)a * rr + ry[i] * RX + rx[i]) * MG + m[i]) = v;
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < I; ++i) {
            // the next step's nodes: their neighbours are this step's
            const bool next = on[i] && rx[i] > lo && rx[i] < hx - 1 && ry[i] > lo &&
                              ry[i] < hy - 1;
            if (!next) continue;
#pragma unroll
            for (int a = 0; a < 9; ++a) {
                const vec v = *reinterpret_cast<const vec*>(
                    mid + ((size_t)a * rr + (ry[i] - cy_of(a)) * RX + rx[i] - cx_of(a)) * MG + m[i]);
#pragma unroll
                for (int k = 0; k < V; ++k) f[i][k][a] = v[k];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// conversions between the member-fastest storage and x-fastest fields.  A block takes
// `tile` consecutive nodes (across the ends of lattice rows) for `mg` members (128 bytes of one
// population where the ensemble has that many) and all nine populations through an LDS
// tile [9][mg][tile + 1], so that both sides move whole cache lines: HBM-bound.  (One
// thread per element with one side strided by 9 M elements fetched every line once
// per member: 256^2 x 64 FP64 import 391 us, export 715, moments 645.)  The member groups of a
// tile follow each other on one XCD: where a group is no whole number of lines they share
// some, which its L2 then completes.
// ---------------------------------------------------------------------------
struct ConvTile {
    int nx, ny, members;
    int log_tile, mg, groups, tiles;  // tile = 1 << log_tile nodes
    // block -> (first node, first member, members and nodes of this block)
    __device__ __forceinline__ void at(int b, int blocks, int* i0, int* m0, int* nm,
                                       int* nn) const {
        b = dev::xcd_remap(b, blocks);
        const int t = b / groups;
        *i0 = t << log_tile;
        *m0 = (b - t * groups) * mg;
        *nm = min(mg, members - *m0);
        *nn = min(1 << log_tile, nx * ny - *i0);
    }
};

// Threads 0 .. 255 step through (row = a * nm + m, x) with x fastest, a thread's x fixed ...
template <typename F>
__device__ __forceinline__ void for_rows(int rows, int log_tile, int nn, F f) {
    const int x = threadIdx.x & ((1 << log_tile) - 1);
    if (x >= nn) return;
#pragma unroll 6
    for (int row = threadIdx.x >> log_tile; row < rows; row += kBlock >> log_tile) f(row, x);
}
// ... and through (row = x * na + a, m) with m fastest.
template <typename F>
__device__ __forceinline__ void for_members(int rows, int nm, F f) {
    const int per = kBlock / nm;  // rows at a time
    const int m = threadIdx.x % nm, r0 = threadIdx.x / nm;
    if (r0 >= per) return;
#pragma unroll 6
    for (int row = r0; row < rows; row += per) f(row, m);
}

// storage slot (node (x, y), a, m) <- canonical [m][a][y + c_ay][x + c_ax]
template <typename T>
__global__ __launch_bounds__(kBlock) void import_kernel(const double* __restrict__ canon,
                                                        T* __restrict__ f, ConvTile c) {
    extern __shared__ char lds_raw[];
    T* tile = reinterpret_cast<T*>(lds_raw);
    int i0, m0, nm, nn;
    c.at(blockIdx.x, gridDim.x, &i0, &m0, &nm, &nn);
    const int ts = (1 << c.log_tile) + 1;
    const size_t plane = (size_t)c.nx * c.ny;
    const int node = i0 + (threadIdx.x & (ts - 2)), ny = node / c.nx, nx = node - ny * c.nx;
    for_rows(9 * nm, c.log_tile, nn, [&](int row, int x) {
        const int a = row / nm, m = row - a * nm;
        const int xs = wrap1(nx + cx_dyn(a), c.nx), ys = wrap1(ny + cy_dyn(a), c.ny);
        tile[(size_t)row * ts + x] = PopIO<T>::pack(
            canon[((size_t)(m0 + m) * 9 + a) * plane + (size_t)ys * c.nx + xs], w_dyn(a));
    });
    __syncthreads();
    T* const out = f + (size_t)i0 * 9 * c.members + m0;
    for_members(9 * nn, nm, [&](int row, int m) {
        const int x = row / 9, a = row - 9 * x;
        out[(size_t)row * c.members + m] = tile[(size_t)(a * nm + m) * ts + x];
    });
}

// canonical [m][a][y + c_ay][x + c_ax] <- storage slot (node (x, y), a, m)
template <typename T>
__global__ __launch_bounds__(kBlock) void export_kernel(const T* __restrict__ f,
                                                        double* __restrict__ canon, ConvTile c) {
    extern __shared__ char lds_raw[];
    T* tile = reinterpret_cast<T*>(lds_raw);
    int i0, m0, nm, nn;
    c.at(blockIdx.x, gridDim.x, &i0, &m0, &nm, &nn);
    const int ts = (1 << c.log_tile) + 1;
    const size_t plane = (size_t)c.nx * c.ny;
    const T* const in = f + (size_t)i0 * 9 * c.members + m0;
    for_members(9 * nn, nm, [&](int row, int m) {
        const int x = row / 9, a = row - 9 * x;
        tile[(size_t)(a * nm + m) * ts + x] = in[(size_t)row * c.members + m];
    });
    __syncthreads();
    const int node = i0 + (threadIdx.x & (ts - 2)), ny = node / c.nx, nx = node - ny * c.nx;
    for_rows(9 * nm, c.log_tile, nn, [&](int row, int x) {
        const int a = row / nm, m = row - a * nm;
        const int xs = wrap1(nx + cx_dyn(a), c.nx), ys = wrap1(ny + cy_dyn(a), c.ny);
        canon[((size_t)(m0 + m) * 9 + a) * plane + (size_t)ys * c.nx + xs] =
            PopIO<T>::unpack(tile[(size_t)row * ts + x], w_dyn(a));
    });
}

// f^eq(rho, u) of node (x, y), written to the slots that hold its canonical populations
// (velocities come in x-fastest: through the LDS tile [2 or 3][mg][tile + 1]).
template <typename T>
__global__ __launch_bounds__(kBlock) void init_equilibrium_kernel(
    const double* __restrict__ rho_in, const double* __restrict__ uv, T* __restrict__ f,
    ConvTile c) {
    extern __shared__ char lds_raw[];
    double* tile = reinterpret_cast<double*>(lds_raw);
    int i0, m0, nm, nn;
    c.at(blockIdx.x, gridDim.x, &i0, &m0, &nm, &nn);
    const int ts = (1 << c.log_tile) + 1;
    const size_t plane = (size_t)c.nx * c.ny;
    for_rows((rho_in ? 3 : 2) * nm, c.log_tile, nn, [&](int row, int x) {
        const int k = row / nm, m = m0 + row - k * nm;
        const double* src = k == 2 ? rho_in + (size_t)m * plane : uv + ((size_t)m * 2 + k) * plane;
        tile[(size_t)row * ts + x] = src[i0 + x];
    });
    __syncthreads();
    for_members(nn, nm, [&](int i, int m) {
        const int y = (i0 + i) / c.nx, x = i0 + i - y * c.nx;
        const double u = tile[(size_t)m * ts + i], v = tile[(size_t)(nm + m) * ts + i];
        const double rho = rho_in ? tile[(size_t)(2 * nm + m) * ts + i] : 1.0;
        const double usq = 1.5 * (u * u + v * v);
#pragma unroll
        for (int a = 0; a < 9; ++a) {
            const double cu = cx_of(a) * u + cy_of(a) * v;
            PopIO<T>::store(f + slot(src_node(x, y, a, c.nx, c.ny), a, m0 + m, c.members), a,
                            rho * w_of(a) * (1.0 + 3.0 * cu + 4.5 * cu * cu - usq));
        }
    });
}

// rho, u, v of every node from the canonical populations: out[m][3][y][x].
template <typename T>
__global__ __launch_bounds__(kBlock) void moments_kernel(const T* __restrict__ f,
                                                         double* __restrict__ out, ConvTile c) {
    extern __shared__ char lds_raw[];
    double* tile = reinterpret_cast<double*>(lds_raw);
    int i0, m0, nm, nn;
    c.at(blockIdx.x, gridDim.x, &i0, &m0, &nm, &nn);
    const int ts = (1 << c.log_tile) + 1;
    const size_t plane = (size_t)c.nx * c.ny;
    for_members(nn, nm, [&](int i, int m) {
        const int y = (i0 + i) / c.nx, x = i0 + i - y * c.nx;
        double rho = 0.0, jx = 0.0, jy = 0.0;
#pragma unroll
        for (int a = 0; a < 9; ++a) {
            const double fa = PopIO<T>::load(
                f + slot(src_node(x, y, a, c.nx, c.ny), a, m0 + m, c.members), a);
            rho += fa;
            jx += cx_of(a) * fa;
            jy += cy_of(a) * fa;
        }
        tile[(size_t)m * ts + i] = rho;
        tile[(size_t)(nm + m) * ts + i] = jx / rho;
        tile[(size_t)(2 * nm + m) * ts + i] = jy / rho;
    });
    __syncthreads();
    for_rows(3 * nm, c.log_tile, nn, [&](int row, int x) {
        const int k = row / nm, m = row - k * nm;
        out[((size_t)(m0 + m) * 3 + k) * plane + i0 + x] = tile[(size_t)row * ts + x];
    });
}

// Tiling of a conversion: up to 128 bytes of members (balanced over the groups), and as
// many nodes as keep the LDS tile near 37 KB (four blocks per CU).
ConvTile conv_tile(LbmDims d, int elem_bytes) {
    ConvTile c{d.nx, d.ny, d.members, 5, 0, 0, 0};
    const int most = 128 / elem_bytes;
    c.groups = (d.members + most - 1) / most;
    c.mg = (d.members + c.groups - 1) / c.groups;
    while (c.log_tile < 8 && (c.mg * elem_bytes << (c.log_tile + 1)) <= 128 * 32) ++c.log_tile;
    c.tiles = (d.nx * d.ny + (1 << c.log_tile) - 1) >> c.log_tile;
    return c;
}

}  // namespace

hipError_t launch_stream_collide(const void* fin, void* fout, const double* force, LbmDims d,
                                 double tau0, double cs, double mu, int storage, hipStream_t s) {
    const int plane = d.nx * d.ny;
    const int V = members_per_thread((int)state_elem_bytes(storage), d.members);
    const int tpn = d.members / V;
    const int npb = nodes_per_block(tpn);
    const dim3 block(tpn, npb);
    const dim3 grid((plane + npb - 1) / npb);
    const double smag = 18.0 * sqrt(2.0) * cs * cs;
    if (storage == kStoreF32Dev && V == 2)
        stream_collide_kernel<float, 2><<<grid, block, 0, s>>>(
            (const float*)fin, (float*)fout, force, d.nx, d.ny, d.members, tau0, smag, mu);
    else if (storage == kStoreF32Dev)
        stream_collide_kernel<float, 1><<<grid, block, 0, s>>>(
            (const float*)fin, (float*)fout, force, d.nx, d.ny, d.members, tau0, smag, mu);
    else
        stream_collide_kernel<double, 1><<<grid, block, 0, s>>>(
            (const double*)fin, (double*)fout, force, d.nx, d.ny, d.members, tau0, smag, mu);
    return hipGetLastError();
}

bool two_step_supported(LbmDims d, int storage) {
    // FP64: blocks of 16 members; FP32 deviations: 32 (or 16) members as pairs
    return d.members % kTwoMG == 0;
}

namespace {
// Time (us) of a multi-step launch, fitted to 6,700 timed shapes on problems of 24^2 .. 512 x 400
// nodes and 1 .. 64 members (median error 8%): a launch, a step of a round of blocks (two
// per CU where LDS and the 16 wavefronts of 128 registers allow), the wavefronts a CU runs in
// all rounds once and per step, in thousands the 64-byte and 128-byte lines a CU touches
// and the bytes it moves, and in MB all blocks' bytes and 128-byte lines.
struct TileFit {
    double launch, round_step, wave, wave_step, lines64, lines128, bytes, all_bytes, all_lines;
};
constexpr TileFit kTileFit[3][2] = {  // FP64, FP32, FP32 pairs of members; items per thread
    {{3.15, 0.436, 0.0, 0.0688, 0.207, 0.0676, 0.00418, 0.0565, 0.0062},
     {4.38, 0.602, 0.0, 0.0558, 0.279, 0.0, 0.0, 0.0546, 0.0112}},
    {{4.48, 0.322, 0.0, 0.0240, 0.0307, 0.0, 0.0296, 0.0135, 0.00352},
     {2.86, 0.940, 0.0, 0.0240, 0.136, 0.0, 0.0288, 0.0346, 0.00241}},
    {{4.73, 0.252, 0.0, 0.0690, 0.202, 0.0, 0.0, 0.0485, 0.00822},
     {3.78, 1.19, 0.0339, 0.0396, 0.245, 0.0, 0.0, 0.0399, 0.0126}}};
constexpr int kMostTileLds = 80 * 1024;  // two blocks per CU

// Lines of 1 << log_line bytes that a block's members of one population touch, mean over the
// rows' alignments (they repeat after a line's worth of elements) and the member groups.
double lines_touched(int members, int mg, int elem, int log_line) {
    int rows = 1;
    while ((rows * members * elem) & ((1 << log_line) - 1)) rows *= 2;
    int total = 0, n = 0;
    for (int row = 0; row < rows; ++row)
        for (int m0 = 0; m0 < members; m0 += mg, ++n) {
            const int first = (row * members + m0) * elem;
            const int last = first + (members - m0 < mg ? members - m0 : mg) * elem - 1;
            total += (last >> log_line) - (first >> log_line) + 1;
        }
    return (double)total / n;
}

struct TileCost {
    int members, elem, V, mg, groups;
    const TileFit* fit;  // [items per thread - 1]
    double l64, l128;
    TileCost(LbmDims d, int storage, int V_, int mg_)
        : members(d.members), elem((int)state_elem_bytes(storage)), V(V_), mg(mg_),
          groups((d.members + mg_ - 1) / mg_),
          fit(kTileFit[V_ == 2 ? 2 : (storage == kStoreF32Dev ? 1 : 0)]),
          l64(lines_touched(d.members, mg_, elem, 6)),
          l128(lines_touched(d.members, mg_, elem, 7)) {}
    int lds(int rx, int ry) const { return 9 * rx * ry * mg * elem; }
    int threads(int rx, int ry, int items) const {
        const int n = rx * ry * mg >> (V - 1);  // (V, items: 1 or 2)
        return (((n + items - 1) >> (items - 1)) + kWave - 1) / kWave * kWave;
    }
    // us per step of a launch of pl.steps on `tiles` tiles, or a large number where it does
    // not fit
    double operator()(LbmDims d, const StepPlan& pl) const {
        const int tx = pl.rx - 2 * (pl.steps - 1), ty = pl.ry - 2 * (pl.steps - 1);
        return (*this)(pl, ((d.nx + tx - 1) / tx) * ((d.ny + ty - 1) / ty));
    }
    // (or takes more than `limit` us per step)
    double operator()(const StepPlan& pl, int tiles, double limit = 1e30) const {
        const int tx = pl.rx - 2 * (pl.steps - 1), ty = pl.ry - 2 * (pl.steps - 1);
        const int bytes = lds(pl.rx, pl.ry);
        const int thr = threads(pl.rx, pl.ry, pl.items);
        if (bytes > kMostTileLds || thr > 1024) return 1e30;
        const int blocks = tiles * groups;
        const double rows = (double)(pl.rx * pl.ry + tx * ty) * 9;  // of one block
        const double mb = rows * blocks / 1e6;
        const TileFit& f = fit[pl.items - 1];
        const double wave = (double)thr / kWave * pl.items * (f.wave + f.wave_step * pl.steps);
        const double lines = f.lines64 * l64 + f.lines128 * l128 + f.bytes * mg * elem;
        const double all = mb * (f.all_bytes * mg * elem + f.all_lines * l128 * 128);
        // (a CU has at least blocks / 256 blocks, in one round or more)
        if (f.launch + f.round_step * pl.steps + all + blocks / 256.0 * (wave + rows / 1e3 * lines) >
            1.000001 * limit * pl.steps)
            return 1e30;
        const int per_cu = std::min(160 * 1024 / bytes, 1024 / thr);
        const int round = 256 * per_cu;
        const int full = blocks / round, rest = blocks - full * round;
        const int rounds = full + (rest > 0);
        const int mine = full * per_cu + (rest + 255) / 256;
        return (f.launch + f.round_step * rounds * pl.steps + mine * (wave + rows / 1e3 * lines) + all) /
               pl.steps;
    }
};

// A plan by size alone, from a sweep of every (members per block, square region, steps,
// items per thread): small problems take few members and long chains, large ones four
// members (32 bytes, eight in FP32) and k = 3, where a longer chain's halo costs more than
// it saves.
StepPlan square_plan(int M, double P, bool pairs) {
    auto balanced = [&](int most) { return (M + (M + most - 1) / most - 1) / ((M + most - 1) / most); };
    auto square = [](int k, int r, int mg, int items) { return StepPlan{k, r, r, mg, items}; };
    if (pairs) {
        if (M == 2) return P <= 1e5 ? square(6, 16, 2, 1) : square(4, 22, 2, 1);
        if (P <= 2e4) return square(6, 16, 2, 1);
        if (P <= 6.4e4) return square(5, 16, 4, 1);
        if (P <= 1e5) return square(4, 16, 4, 1);
        if (M % 8 == 0 && P <= 9e5) return square(P <= 2e5 ? 4 : 3, 16, 8, 1);
        return square(4, 22, 4, 1);
    }
    if (P <= 1e4 || (M == 1 && P <= 2e4)) return square(6, 16, 1, 1);
    if (M == 1) return P <= 1e5 ? square(5, 24, 1, 1) : square(4, 22, 1, 1);
    if (P <= 3.2e4 || (M <= 3 && P <= 6.4e4)) return square(5, 16, M == 3 ? 3 : 2, 1);
    if (M <= 3) return square(4, M == 2 ? 22 : 16, M, 1);
    const int mg = balanced(4);
    if (P <= 6.4e4) return square(5, 16, mg, 1);
    if (P <= 1e5) return square(4, 16, mg, 1);
    return square(3, 16, mg, P <= 2.2e5 ? 1 : 2);
}
}  // namespace

// The tiled multi-step launches of an ensemble, or none where pairs of steps on 128-byte
// member blocks are as fast or faster: 16 | M from P = 1e5 node-members on, except FP32
// with 16 members (us per step, single / pair / tiles: 96^2 x 16 5.8 / 3.7 / 3.7, 160^2 x 32
// 20.4 / 15.3 / 16, but 24^2 x 16 3.9 / 3.0 / 1.6 and FP32 256^2 x 16 17.8 / 14.2 / 10.6).
// Square regions leave to chance how full the last round of blocks is, so a launch of n
// steps takes the shape of the least fitted time, if that is 8% (the fit's error) below the
// square one's.  Searched at the square plan's members and, but for FP32 pairs, among the
// member counts and steps that were ever best: one member and long chains for ensembles of up
// to three and small problems (not the smallest, one block on every other CU at most); four
// members (or five, or half the ensemble) and up to three steps else; two in between.  us per
// step, square / this: 32^2 x 8 1.8 / 1.5, 149 x 143 x 1 1.7 / 1.3, 150 x 97 x 20 9.0 / 8.5,
// 170 x 110 x 6 5.0 / 3.5, 333 x 300 x 5 16 / 10.5; FP32 101 x 122 x 20 5.3 / 4.1, 201 x 249 x 3
// 4.1 / 2.9.
StepPlans step_plans(LbmDims d, int storage) {
    const double P = (double)d.nx * d.ny * d.members;
    const int M = d.members;
    const bool pairs = members_per_thread((int)state_elem_bytes(storage), M) == 2;
    StepPlans out{};
    if (M % kTwoMG == 0 && P > 1e5 && !(pairs && M == 16)) return out;
    const int V = pairs ? 2 : 1;
    StepPlan base = square_plan(M, P, pairs);
    double guard[kMostSteps + 1];
    {
        const TileCost cost(d, storage, V, base.members);
        for (int n = 1; n <= kMostSteps; ++n) {
            out.us[n] = guard[n] = 1e30;
            if (n > base.steps) continue;
            out.p[n] = base;
            out.p[n].steps = n;
            out.us[n] = n * cost(d, out.p[n]);
            guard[n] = 0.92 * out.us[n];
        }
    }
    constexpr int kLeastTile = 4, kMostTile = 32;
    int tiles_x[kMostTile + 1], tiles_y[kMostTile + 1];
    for (int t = kLeastTile; t <= kMostTile; ++t) {
        tiles_x[t] = (d.nx + t - 1) / t;
        tiles_y[t] = (d.ny + t - 1) / t;
    }
    auto search = [&](int mg, int k0, int k1) {
        if (mg > M || mg % V) return;
        const TileCost cost(d, storage, V, mg);
        for (int k = k0; k <= k1; ++k)
            for (int tx = kLeastTile; tx <= kMostTile; ++tx) {
                // (a wider tile costs more unless it saves one)
                if (tx > kLeastTile && tiles_x[tx] == tiles_x[tx - 1]) continue;
                for (int ty = kLeastTile; ty <= kMostTile; ++ty) {
                    if (ty > kLeastTile && tiles_y[ty] == tiles_y[ty - 1]) continue;
                    StepPlan pl{k, tx + 2 * (k - 1), ty + 2 * (k - 1), mg, 1};
                    // (both grow with ty)
                    if (cost.lds(pl.rx, pl.ry) > kMostTileLds ||
                        cost.threads(pl.rx, pl.ry, 2) > 1024)
                        break;
                    for (; pl.items <= 2; ++pl.items) {
                        const double t = k * cost(pl, tiles_x[tx] * tiles_y[ty], guard[k] / k);
                        if (t < guard[k]) {
                            guard[k] = out.us[k] = t;
                            out.p[k] = pl;
                        }
                    }
                }
            }
    };
    if (P > 5e3) search(base.members, 2, base.steps);
    if (pairs) {
        if (M % 10 == 0 && P > 1e6) search(10, 3, 3);
    } else if (P > 5e3) {
        if (M <= 3 || P < 2e4) search(1, 5, 6);
        if (P < 2e5) search(2, 3, 5);
        if (M == 3) search(3, 2, 3);
        search(4, 2, 3);
        search(5, 2, 3);
        if (M >= 12 && M <= 24) search((M + 1) / 2, 2, 2);
    }
    for (int n = 1; n <= kMostSteps; ++n)
        if (out.us[n] < 1e29) out.most = n;
    // Launches too short to gain from the tiles, which split a line's members: single steps
    // for all but small ensembles, pairs for 16 FP32 members.  us of two single steps, plain /
    // tiled: 1 member 21 / 16 at P = 6.6e4, 5 members 28 / 19 at 3e5 but 10.6 / 11.8 at 3e3, FP64 50 members 900 / 1329 at 1.3e7, 33 members 143 / 212 at 2.2e6; FP32 12 members
    // 1.17 times at 4e6, 0.73 at 1e5; four steps of 16 FP32 members as pairs / tiled 167 / 190 at 4e6.
    const bool tiled = (M <= 2 && P >= 2e4) || (M <= 5 && P >= 1e5) ||
                       (M <= 12 && M * (int)state_elem_bytes(storage) <= 56 && P >= 2e5);
    out.fewest = tiled ? 1 : (M == 16 && P > 1e5 ? 3 : 2);
    return out;
}

// With every state written a tiled launch saves only reads and launches, and writes each line in
// the pieces of its member groups: beyond 12 members and 4e5 node-members single steps (pairs
// for 16 FP32 members) take over.  Reverse sweep of 3 x 10 steps, time single / tiled: 8 members
// 1.17, 1.11, 1.06 at P = 5e4, 4e5, 4e6; 24 members 1.08, 1.00, 0.84; 40 members 1.10, 0.97, 0.80;
// FP32 16 members 1.15, 1.06, 0.92; 33 members 1.06, 1.02, 0.95.
bool tiles_keep_states(LbmDims d) {
    return d.members <= 12 || (double)d.nx * d.ny * d.members <= 4e5;
}

int plan_launches(const StepPlans& plans, int steps, bool even) {
    int best = 0;
    double least = 1e30;
    const int first = (steps + plans.most - 1) / plans.most;
    for (int launches = first; launches <= first + 3 + first / 2; ++launches) {
        if (even && (launches & 1)) continue;
        if (launches > steps && best) break;
        const int n = steps / launches, longer = steps - n * launches;  // of n + 1 steps
        double t = 0.0;
        if (longer) t += longer * plans.us[n + 1];
        if (n) t += (launches - longer) * plans.us[n];
        if (t < least) {
            least = t;
            best = launches;
        }
    }
    return best;
}

namespace {
template <typename T, int V, int I>
hipError_t launch_tile_t(const void* fin, void* fout, const double* force, LbmDims d, double tau0,
                         double smag, double mu, hipStream_t s, const StepPlan& pl, int steps,
                         void* fmid, size_t mid_bytes) {
    const int tx = pl.rx - 2 * (steps - 1), ty = pl.ry - 2 * (steps - 1);
    if (tx < 1 || ty < 1) return hipErrorInvalidValue;
    const int blocks = ((d.nx + tx - 1) / tx) * ((d.ny + ty - 1) / ty) *
                       ((d.members + pl.members - 1) / pl.members);
    const int items = pl.rx * pl.ry * (pl.members / V);
    const int threads = ((items + I - 1) / I + kWave - 1) / kWave * kWave;
    const size_t lds = (size_t)9 * pl.rx * pl.ry * pl.members * sizeof(T);
    constexpr size_t kMostLds = kMostTileLds;
    if (threads > 1024 || lds > kMostLds || pl.members % V) return hipErrorInvalidValue;
    static std::atomic<uint64_t> lds_ok{0};
    const hipError_t e = allow_lds(stream_collide_tile_kernel<T, V, I>, kMostLds, &lds_ok);
    if (e != hipSuccess) return e;
    stream_collide_tile_kernel<T, V, I><<<blocks, threads, lds, s>>>(
        (const T*)fin, (T*)fout, force, d.nx, d.ny, d.members, tau0, smag, mu, pl.rx, pl.ry,
        pl.members, steps, (T*)fmid, mid_bytes / sizeof(T));
    return hipGetLastError();
}
}  // namespace

hipError_t launch_stream_collide_tile(const void* fin, void* fout, const double* force, LbmDims d,
                                      double tau0, double cs, double mu, int storage, hipStream_t s,
                                      const StepPlan& pl, int steps, void* fmid,
                                      size_t mid_bytes) {
    if (pl.steps < 1 || steps < 1 || steps > pl.steps) return hipErrorInvalidValue;
    const double smag = 18.0 * sqrt(2.0) * cs * cs;
    if (storage != kStoreF32Dev)
        return pl.items == 1 ? launch_tile_t<double, 1, 1>(fin, fout, force, d, tau0, smag, mu, s,
                                                           pl, steps, fmid, mid_bytes)
                             : launch_tile_t<double, 1, 2>(fin, fout, force, d, tau0, smag, mu, s,
                                                           pl, steps, fmid, mid_bytes);
    if (members_per_thread(4, d.members) == 2)
        return pl.items == 1 ? launch_tile_t<float, 2, 1>(fin, fout, force, d, tau0, smag, mu, s,
                                                          pl, steps, fmid, mid_bytes)
                             : launch_tile_t<float, 2, 2>(fin, fout, force, d, tau0, smag, mu, s,
                                                          pl, steps, fmid, mid_bytes);
    return pl.items == 1 ? launch_tile_t<float, 1, 1>(fin, fout, force, d, tau0, smag, mu, s, pl,
                                                      steps, fmid, mid_bytes)
                         : launch_tile_t<float, 1, 2>(fin, fout, force, d, tau0, smag, mu, s, pl,
                                                      steps, fmid, mid_bytes);
}

hipError_t launch_stream_collide2(const void* fin, void* fout, const double* force, LbmDims d,
                                  double tau0, double cs, double mu, int storage, hipStream_t s,
                                  void* fmid) {
    if (!two_step_supported(d, storage)) return hipErrorInvalidValue;
    const int tiles = ((d.nx + kTwoT - 1) / kTwoT) * ((d.ny + kTwoT - 1) / kTwoT);
    const double smag = 18.0 * sqrt(2.0) * cs * cs;
    hipError_t e = hipSuccess;
    if (storage == kStoreF32Dev) {
        static std::atomic<uint64_t> ok32{0}, ok16{0};
        if (d.members % 32 == 0) {
            const size_t bytes = (size_t)kTwoR * kTwoR * 9 * 32 * sizeof(float);
            e = allow_lds(stream_collide2_dev_kernel<32>, bytes, &ok32);
            if (e != hipSuccess) return e;
            stream_collide2_dev_kernel<32><<<tiles * (d.members / 32), dim3(16, kTwoR * kTwoR),
                                             bytes, s>>>((const float*)fin, (float*)fout, force,
                                                         d.nx, d.ny, d.members, (float)tau0,
                                                         (float)smag, (float)mu, (float*)fmid);
        } else {
            const size_t bytes = (size_t)kTwoR * kTwoR * 9 * 16 * sizeof(float);
            e = allow_lds(stream_collide2_dev_kernel<16>, bytes, &ok16);
            if (e != hipSuccess) return e;
            stream_collide2_dev_kernel<16><<<tiles * (d.members / 16), dim3(8, kTwoR * kTwoR),
                                             bytes, s>>>((const float*)fin, (float*)fout, force,
                                                         d.nx, d.ny, d.members, (float)tau0,
                                                         (float)smag, (float)mu, (float*)fmid);
        }
        return hipGetLastError();
    }
    const dim3 grid(tiles * (d.members / kTwoMG)), block(kTwoMG, kTwoR * kTwoR);
    const size_t bytes = (size_t)two_step_lds_doubles() * sizeof(double);
    static std::atomic<uint64_t> lds_ok{0};
    e = allow_lds(stream_collide2_kernel, bytes, &lds_ok);
    if (e != hipSuccess) return e;
    stream_collide2_kernel<<<grid, block, bytes, s>>>(
        (const double*)fin, (double*)fout, force, d.nx, d.ny, d.members, tau0, smag, mu,
        (double*)fmid);
    return hipGetLastError();
}

hipError_t launch_stream_collide_batch(const LbmTask* d_tasks, int ntasks, int ntiles, int blocks,
                                       int storage, hipStream_t s) {
    if (storage == kStoreF32Dev)
        stream_collide_batch_kernel<float><<<blocks, kBlock, 0, s>>>(d_tasks, ntasks, ntiles);
    else
        stream_collide_batch_kernel<double><<<blocks, kBlock, 0, s>>>(d_tasks, ntasks, ntiles);
    return hipGetLastError();
}

int two_step_blocks(LbmDims d, int storage) {
    const int g = (storage == kStoreF32Dev && d.members % kTwoMG32 == 0) ? kTwoMG32 : kTwoMG;
    const int per = storage == kStoreF32Dev ? kTwoMG32 / g : 1;  // units per block
    const int units = ((d.nx + kTwoT - 1) / kTwoT) * ((d.ny + kTwoT - 1) / kTwoT) * (d.members / g);
    return (units + per - 1) / per;
}

hipError_t launch_stream_collide2_batch(const LbmTask* d_tasks, int ntasks, int nblocks,
                                        int storage, hipStream_t s) {
    static std::atomic<uint64_t> ok64{0}, ok32{0};
    hipError_t e = hipSuccess;
    if (storage == kStoreF32Dev) {
        const size_t bytes = (size_t)kTwoR * kTwoR * 9 * kTwoMG32 * sizeof(float);
        e = allow_lds(stream_collide2_batch_kernel<float>, bytes, &ok32);
        if (e != hipSuccess) return e;
        stream_collide2_batch_kernel<float><<<nblocks, dim3(kTwoMG32 / 2, kTwoR * kTwoR), bytes,
                                              s>>>(d_tasks, ntasks);
    } else {
        const size_t bytes = (size_t)two_step_lds_doubles() * sizeof(double);
        e = allow_lds(stream_collide2_batch_kernel<double>, bytes, &ok64);
        if (e != hipSuccess) return e;
        stream_collide2_batch_kernel<double><<<nblocks, dim3(kTwoMG, kTwoR * kTwoR), bytes, s>>>(
            d_tasks, ntasks);
    }
    return hipGetLastError();
}

hipError_t launch_import(const double* canon, void* f, LbmDims d, int storage, hipStream_t s) {
    const int eb = (int)state_elem_bytes(storage);
    const ConvTile c = conv_tile(d, eb);
    const int blocks = c.tiles * c.groups;
    const size_t lds = (size_t)9 * c.mg * ((1 << c.log_tile) + 1) * eb;
    if (storage == kStoreF32Dev) import_kernel<float><<<blocks, kBlock, lds, s>>>(canon, (float*)f, c);
    else import_kernel<double><<<blocks, kBlock, lds, s>>>(canon, (double*)f, c);
    return hipGetLastError();
}

hipError_t launch_export(const void* f, double* canon, LbmDims d, int storage, hipStream_t s) {
    const int eb = (int)state_elem_bytes(storage);
    const ConvTile c = conv_tile(d, eb);
    const int blocks = c.tiles * c.groups;
    const size_t lds = (size_t)9 * c.mg * ((1 << c.log_tile) + 1) * eb;
    if (storage == kStoreF32Dev)
        export_kernel<float><<<blocks, kBlock, lds, s>>>((const float*)f, canon, c);
    else
        export_kernel<double><<<blocks, kBlock, lds, s>>>((const double*)f, canon, c);
    return hipGetLastError();
}

hipError_t launch_init_equilibrium(const double* rho, const double* uv, void* f, LbmDims d,
                                   int storage, hipStream_t s) {
    const ConvTile c = conv_tile(d, (int)state_elem_bytes(storage));
    const int blocks = c.tiles * c.groups;
    const size_t lds = (size_t)3 * c.mg * ((1 << c.log_tile) + 1) * sizeof(double);
    if (storage == kStoreF32Dev)
        init_equilibrium_kernel<float><<<blocks, kBlock, lds, s>>>(rho, uv, (float*)f, c);
    else
        init_equilibrium_kernel<double><<<blocks, kBlock, lds, s>>>(rho, uv, (double*)f, c);
    return hipGetLastError();
}

hipError_t launch_moments(const void* f, double* out, LbmDims d, int storage, hipStream_t s) {
    const ConvTile c = conv_tile(d, (int)state_elem_bytes(storage));
    const int blocks = c.tiles * c.groups;
    const size_t lds = (size_t)3 * c.mg * ((1 << c.log_tile) + 1) * sizeof(double);
    if (storage == kStoreF32Dev)
        moments_kernel<float><<<blocks, kBlock, lds, s>>>((const float*)f, out, c);
    else
        moments_kernel<double><<<blocks, kBlock, lds, s>>>((const double*)f, out, c);
    return hipGetLastError();
}

}  // namespace lbmletkf
