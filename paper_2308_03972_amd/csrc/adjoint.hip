// Differentiation form: reverse-mode adjoint of the forecast (Sec. 2 LBE with
// BGK relaxation, Smagorinsky eddy viscosity, force and friction) and of the
// observation misfit J = sum_c sum_m sum_q (H_q(f_m(t_c)) - y^o_{c,q})^2.
//
// One forward step maps the canonical state f^n to f^{n+1} by
//     f^{n+1}_a(x) = C_a(f^n(x - c_a)),
// C the per-node collision.  Its adjoint is
//     lam^n_b(y) = sum_a lam^{n+1}_a(y + c_a) dC_a/df_b (f^n(y)),
// i.e. a push-direction gather of the adjoint and the transposed Jacobian of
// the collision at the forward state, written aligned.  The vector-Jacobian
// product below is the hand-derived reverse of the forward kernel's
// operations in reverse order (moments -> equilibrium -> non-equilibrium flux
// -> |Pi| -> tau -> omega, force with friction); it also returns the
// sensitivity to K = 18 sqrt(2) C_s^2, from which dJ/dC_s = (36 sqrt(2) C_s)
// * sum over steps, nodes and members.  At |Pi| = 0 the subgradient 0 is used.
#include <algorithm>

#include "common.h"
#include "device_util.h"

namespace lbmletkf {
namespace {
using namespace dev;

constexpr int kBlock = 256;

// Reverse of one collision.  f: pre-collision populations; L: adjoint of the
// post-collision outputs.  Returns the adjoint of f in Lf and d(out.L)/dK.
// The outputs' adjoint enters only through L.f and the moments of q_a = w_a L_a up to second
// order (feq and the force are polynomials of that order in c_a), and the reverse of the
// moments is one polynomial in c_a again: about 250 FP64 instructions, where the sums written
// out per population took 500.
__device__ __forceinline__ double collide_vjp(const double (&f)[9], const double (&L)[9],
                                              double tau0, double K, double fx_ext,
                                              double fy_ext, double mu, double (&Lf)[9]) {
    // ---- forward recomputation (same operations as the forward kernel)
    const double rho = ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7])) + f[8];
    const double jx = (f[1] - f[2]) + (f[5] - f[6]) + (f[7] - f[8]);
    const double jy = (f[3] - f[4]) + (f[5] - f[6]) + (f[8] - f[7]);
    const double ir = 1.0 / rho;
    const double u = jx * ir, v = jy * ir;
    const double uu = u * u, vv = v * v, uv = u * v;
    const double pxx = (f[1] + f[2] + f[5] + f[6] + f[7] + f[8]) - rho * (1.0 / 3.0 + uu);
    const double pyy = (f[3] + f[4] + f[5] + f[6] + f[7] + f[8]) - rho * (1.0 / 3.0 + vv);
    const double pxy = (f[5] + f[6] - f[7] - f[8]) - rho * uv;
    const double P = sqrt(pxx * pxx + pyy * pyy + 2.0 * pxy * pxy);
    const double R = sqrt(tau0 * tau0 + K * P * ir);
    const double tau = 0.5 * (tau0 + R);
    const double itr = 1.0 / (tau * R);  // 1 / tau = R itr, 1 / R = tau itr
    const double om = R * itr;
    const double gx = fx_ext - mu * u, gy = fy_ext - mu * v;
    // ---- moments of the outputs' adjoint: L.f and sum_a w_a L_a c_a^k
    double Lfs = L[0] * f[0];
#pragma unroll
    for (int a = 1; a < 9; ++a) Lfs = fma(L[a], f[a], Lfs);
    const double dg = L[5] + L[6], dh = L[7] + L[8];  // the two diagonals
    const double ex = L[5] - L[6], ey = L[7] - L[8];
    const double md = w_of(5) * (dg + dh);
    const double sx = w_of(1) * (L[1] + L[2]), sy = w_of(1) * (L[3] + L[4]);
    const double m0 = w_of(0) * L[0] + (sx + sy) + md;
    const double mx = w_of(1) * (L[1] - L[2]) + w_of(5) * (ex + ey);
    const double my = w_of(1) * (L[3] - L[4]) + w_of(5) * (ex - ey);
    const double mxx = sx + md, myy = sy + md, mxy = w_of(5) * (dg - dh);
    // ---- reverse: out_a = (1 - om) f_a + om feq_a + F_a,
    // feq_a = rho w_a (1 + 3 cu + 4.5 cu^2 - 1.5 u.u), F_a = 3 w_a rho (c_a.g)
    const double tx = mxx * u + mxy * v, ty = mxy * u + myy * v;
    const double E = m0 * (1.0 - 1.5 * (uu + vv)) + 3.0 * (mx * u + my * v) +
                     4.5 * (tx * u + ty * v);  // L.feq / rho
    const double Lom = rho * E - Lfs;
    double Lrho = om * E + 3.0 * (mx * gx + my * gy);
    const double r3 = 3.0 * rho;
    // (with the force's share: g = F_ext - mu u)
    double Lu = r3 * (om * (mx + 3.0 * tx - u * m0) - mu * mx);
    double Lv = r3 * (om * (my + 3.0 * ty - v * m0) - mu * my);
    // om = 1 / tau, tau = (tau0 + R) / 2, R = sqrt(tau0^2 + K P ir)
    const double Larg = -0.25 * Lom * om * om * (tau * itr);
    double Lir = Larg * K * P;
    const double LK = Larg * P * ir;
    // P = sqrt(pxx^2 + pyy^2 + 2 pxy^2)
    double Lpxx = 0.0, Lpyy = 0.0, Lpxy = 0.0;
    if (P > 0.0) {
        const double LPP = Larg * K * ir / P;
        Lpxx = LPP * pxx;
        Lpyy = LPP * pyy;
        Lpxy = 2.0 * LPP * pxy;
    }
    // pxx = sum cx^2 f - rho (1/3 + u^2), pyy likewise, pxy = sum cx cy f - rho u v
    Lrho -= Lpxx * (1.0 / 3.0 + uu) + Lpyy * (1.0 / 3.0 + vv) + Lpxy * uv;
    Lu -= rho * (2.0 * Lpxx * u + Lpxy * v);
    Lv -= rho * (2.0 * Lpyy * v + Lpxy * u);
    // u = jx ir, v = jy ir, ir = 1 / rho
    const double Ljx = Lu * ir, Ljy = Lv * ir;
    Lir += Lu * jx + Lv * jy;
    Lrho -= Lir * ir * ir;
    // Lf_a = (1 - om) L_a + Lrho + Lj.c_a + Lp:c_a c_a
    const double keep = 1.0 - om;
    const double cxx = Lrho + Lpxx, cyy = Lrho + Lpyy, cd = cxx + Lpyy;
    const double c5 = cd + Lpxy, c7 = cd - Lpxy, jp = Ljx + Ljy, jm = Ljx - Ljy;
    Lf[0] = keep * L[0] + Lrho;
    Lf[1] = keep * L[1] + (cxx + Ljx);
    Lf[2] = keep * L[2] + (cxx - Ljx);
    Lf[3] = keep * L[3] + (cyy + Ljy);
    Lf[4] = keep * L[4] + (cyy - Ljy);
    Lf[5] = keep * L[5] + (c5 + jp);
    Lf[6] = keep * L[6] + (c5 - jp);
    Lf[7] = keep * L[7] + (c7 + jm);
    Lf[8] = keep * L[8] + (c7 - jm);
    return LK;
}

// One reverse step, one thread per (node, member) as in the forward kernel.
// fstate: storage layout; lam_in, lam_out: adjoint states in the canonical
// node-major layout [node][a][member] (lam(y)_a of member m at slot(y, a, m)).
template <typename T>
__global__ __launch_bounds__(kBlock) void adjoint_step_kernel(
    const T* __restrict__ fstate, const double* __restrict__ lam_in, double* __restrict__ lam_out,
    const double* __restrict__ force, int nx, int ny, int members, double tau0, double K,
    double mu, double* __restrict__ k_partial) {
    const int plane = nx * ny;
    const int m = threadIdx.x;  // blockDim.x == members
    const int node = blockIdx.x * blockDim.y + threadIdx.y;
    double lk = 0.0;
    if (node < plane) {
        const int y = node / nx, x = node - y * nx;
        const int xm = wrap(x - 1, nx), xp = wrap(x + 1, nx);
        const int ym = wrap(y - 1, ny), yp = wrap(y + 1, ny);
        // forward state: canonical f_a(y) is held by the slot of node y - c_a
        const PullSlots<const T> fsrc(fstate, x, xm, xp, y, ym, yp, nx, members, m);
        // adjoint of f^{n+1}_a at the node this population streams to, y + c_a
        // (the same addressing with the neighbours swapped)
        const PullSlots<const double> lsrc(lam_in, x, xp, xm, y, yp, ym, nx, members, m);
        double f[9], L[9], Lf[9];
#pragma unroll
        for (int a = 0; a < 9; ++a) {
            f[a] = PopIO<T>::load(fsrc.at(a), a);
            L[a] = *lsrc.at(a);
        }
        const double fx = force ? force[node] : 0.0, fy = force ? force[plane + node] : 0.0;
        lk = collide_vjp(f, L, tau0, K, fx, fy, mu, Lf);
        double* const out = lam_out + (size_t)node * 9 * members + m;
#pragma unroll
        for (int a = 0; a < 9; ++a) out[(uint32_t)a * members] = Lf[a];
    }
    // per-block sum of dJ/dK, accumulated in this block's own slot (launches
    // on one stream are ordered, so the accumulation is deterministic)
    const int tid = threadIdx.y * blockDim.x + threadIdx.x;
    const int nthreads = blockDim.x * blockDim.y;
    __shared__ double red[kBlock];
    if (nthreads % kWave == 0) {
        // whole wavefronts (M a power of two): a DPP sum per wavefront, then
        // the wavefront sums in order, one barrier
        const double ws = wave_sum(lk);
        if (tid % kWave == 0) red[tid / kWave] = ws;
        __syncthreads();
        if (tid == 0) {
            double t = 0.0;
            for (int w = 0; w < nthreads / kWave; ++w) t += red[w];
            k_partial[blockIdx.x] += t;
        }
        return;
    }
    red[tid] = lk;
    __syncthreads();
    for (int s = kBlock / 2; s > 0; s >>= 1) {
        if (tid < s && tid + s < nthreads) red[tid] += red[tid + s];
        __syncthreads();
    }
    if (tid == 0) k_partial[blockIdx.x] += red[0];
}

// Several reverse steps per launch.  A block takes MG members of a region of R x R nodes, one
// thread per (node, member); the first step gathers from HBM, the later ones from LDS, each on
// one ring of nodes less, and after `steps` steps the inner T x T nodes (T = R - 2 (steps - 1))
// are written.  The gather y + c_a has one reader per value, so a step writes its results
// over the values it has read, and step s finds population a of node y + c_a at y + s c_a: one
// barrier per step, no second buffer.  fhi: the state of the first reversed step, the next
// ones `stride` elements below; flast: that of the last one.
// Bound by FP64 issue (about 240 FP64 instructions per node, member and step) and, on small
// problems, by the latency of a step.  Same arithmetic as single steps; only the order of the partial
// sums of dJ/dK differs.  Shapes: adjoint_plan.
template <typename T>
__global__ __launch_bounds__(1024) void adjoint_tile_kernel(
    const T* __restrict__ fhi, const T* __restrict__ flast, size_t stride,
    const double* __restrict__ lam_in, double* __restrict__ lam_out,
    const double* __restrict__ force, int nx, int ny, int members, double tau0, double K,
    double mu, int R, int MG, int steps, double* __restrict__ k_partial) {
    extern __shared__ double lds[];  // [9][R * R][MG]
    __shared__ double red[1024 / kWave];
    const int halo = steps - 1, tile = R - 2 * halo;
    const int groups = (members + MG - 1) / MG;
    const int tiles_x = (nx + tile - 1) / tile;
    const int b = xcd_remap(blockIdx.x, gridDim.x);  // the groups of a tile share lines
    const int t = b / groups, m0 = (b - t * groups) * MG;
    const int x0 = (t % tiles_x) * tile, y0 = (t / tiles_x) * tile;
    const int plane = nx * ny, rr = R * R;
    const int node_r = threadIdx.x / MG, m = threadIdx.x - node_r * MG;
    const int ry = node_r / R, rx = node_r - ry * R;
    bool on = node_r < rr && m0 + m < members;
    const bool inner = on && rx >= halo && rx < halo + tile && ry >= halo && ry < halo + tile &&
                       x0 + rx - halo < nx && y0 + ry - halo < ny;
    int x = (x0 - halo + rx) % nx, y = (y0 - halo + ry) % ny;
    x = x < 0 ? x + nx : x;
    y = y < 0 ? y + ny : y;
    const int node = y * nx + x;
    const int at = (ry * R + rx) * MG + m;
    double f[9], L[9];
    double fx = 0.0, fy = 0.0, lk = 0.0;
    // forward state: canonical f_a(y) is held by the slot of node y - c_a
    auto load_state = [&](const T* fs) {
        int xs = x, ys = y;  // (addresses anew: kept over the steps they hold 20 registers)
        asm volatile("" : "+v"(xs), "+v"(ys));
        const PullSlots<const T> src(fs, xs, wrap(xs - 1, nx), wrap(xs + 1, nx), ys,
                                     wrap(ys - 1, ny), wrap(ys + 1, ny), nx, members, m0 + m);
#pragma unroll
        for (int a = 0; a < 9; ++a) f[a] = PopIO<T>::load(src.at(a), a);
    };
    const T* fs = steps == 1 ? flast : fhi;
    if (on) {
        if (force) {
            fx = force[node];
            fy = force[plane + node];
        }
        // adjoint of f^{n+1}_a: at y + c_a (the same addressing with the neighbours swapped)
        const PullSlots<const double> src(lam_in, x, wrap(x + 1, nx), wrap(x - 1, nx), y,
                                          wrap(y + 1, ny), wrap(y - 1, ny), nx, members, m0 + m);
#pragma unroll
        for (int a = 0; a < 9; ++a) L[a] = *src.at(a);
        load_state(fs);
    }
    for (int s = 1;; ++s) {
        double* const l0 = lds + at;
        if (on) {
            double Lf[9];
            const double k = collide_vjp(f, L, tau0, K, fx, fy, mu, Lf);
            if (inner) lk += k;
            if (s == steps) {
                if (inner) {
                    double* const out = lam_out + (size_t)node * 9 * members + m0 + m;
#pragma unroll
                    for (int a = 0; a < 9; ++a) out[(uint32_t)a * members] = Lf[a];
                }
            } else {
#pragma unroll
                for (int a = 0; a < 9; ++a)
                    l0[(a * rr + (s - 1) * (cy_of(a) * R + cx_of(a))) * MG] = Lf[a];
            }
        }
        if (s == steps) break;
        on = on && rx >= s && rx < R - s && ry >= s && ry < R - s;
        fs = s + 1 == steps ? flast : fs - stride;
        if (on) load_state(fs);
        __syncthreads();
        if (on) {
#pragma unroll
            for (int a = 0; a < 9; ++a) L[a] = l0[(a * rr + s * (cy_of(a) * R + cx_of(a))) * MG];
        }
    }
    // this block's sum of dJ/dK goes to its own slot (launches on one stream are ordered,
    // so the accumulation is deterministic)
    const double ws = wave_sum(lk);
    if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = ws;
    __syncthreads();
    if (threadIdx.x == 0) {
        double total = 0.0;
        for (int w = 0; w < (int)blockDim.x / kWave; ++w) total += red[w];
        k_partial[blockIdx.x] += total;
    }
}

// Misfit at one observation time.  One thread per (point, member), members
// fastest: adds (H - y^o)^2 to jbuf[m * npts + k] (if jbuf) and, if lam is
// given, dJ/df at the observation node to the adjoint state.
template <typename T>
__global__ void misfit_kernel(const T* __restrict__ f, const int* __restrict__ pts, int npts,
                              int nvar, const double* __restrict__ yo, double* __restrict__ lam,
                              double* __restrict__ jbuf, int first, int nx, int ny, int members) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= npts * members) return;
    const int k = t / members, m = t - k * members;
    const int x = pts[2 * k], y = pts[2 * k + 1];
    double fa[9];
    double rho = 0.0, jx = 0.0, jy = 0.0;
#pragma unroll
    for (int a = 0; a < 9; ++a) {
        fa[a] = PopIO<T>::load(f + slot(src_node(x, y, a, nx, ny), a, m, members), a);
        rho += fa[a];
        jx += cx_of(a) * fa[a];
        jy += cy_of(a) * fa[a];
    }
    const double u = jx / rho, v = jy / rho;
    const double* y0 = yo + (size_t)k * nvar;
    double rr = 0.0, ru = 0.0, rv = 0.0;
    if (nvar == 3) {
        rr = rho - y0[0];
        ru = u - y0[1];
        rv = v - y0[2];
    } else {
        ru = u - y0[0];
        rv = v - y0[1];
    }
    if (jbuf) {
        double& j = jbuf[(size_t)m * npts + k];
        j = (first ? 0.0 : j) + (rr * rr + ru * ru + rv * rv);
    }
    if (lam) {
        // dJ/df_a = 2 rr + 2 ru (c_ax - u)/rho + 2 rv (c_ay - v)/rho
        const size_t node = (size_t)y * nx + x;
#pragma unroll
        for (int a = 0; a < 9; ++a) {
            const double g = 2.0 * rr + 2.0 * (ru * (cx_of(a) - u) + rv * (cy_of(a) - v)) / rho;
            lam[slot(node, a, m, members)] += g;
        }
    }
}

// Adjoint state [node][a][member] -> canonical public layout [member][a][y][x].
__global__ void lam_to_canonical_kernel(const double* __restrict__ lam, double* __restrict__ out,
                                        int plane, int members) {
    const size_t total = (size_t)plane * 9 * members;
    for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < total;
         t += (size_t)gridDim.x * blockDim.x) {
        const size_t i = t % plane;
        const int a = (int)((t / plane) % 9);
        const int m = (int)(t / ((size_t)plane * 9));
        out[t] = lam[slot(i, a, m, members)];
    }
}

// Deterministic single-block sum of n doubles into out[0] (times scale).
__global__ __launch_bounds__(256) void sum_kernel(const double* __restrict__ v, size_t n,
                                                  double scale, double* __restrict__ out) {
    __shared__ double red[256];
    double s = 0.0;
    for (size_t i = threadIdx.x; i < n; i += 256) s += v[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = scale * red[0];
}

__global__ void zero2_kernel(double* __restrict__ v0, size_t n0, double* __restrict__ v1,
                             size_t n1) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n0 + n1;
         i += (size_t)gridDim.x * blockDim.x)
        *(i < n0 ? v0 + i : v1 + (i - n0)) = 0.0;
}

}  // namespace

int adjoint_partials(LbmDims d) {
    const int npb = nodes_per_block(d.members);
    return (d.nx * d.ny + npb - 1) / npb;
}

hipError_t launch_adjoint_step(const void* fstate, const double* lam_in, double* lam_out,
                               const double* force, LbmDims d, double tau0, double cs, double mu,
                               int storage, double* k_partial, hipStream_t s) {
    const int npb = nodes_per_block(d.members);
    const dim3 block(d.members, npb);
    const dim3 grid(adjoint_partials(d));
    const double K = 18.0 * sqrt(2.0) * cs * cs;
    if (storage == kStoreF32Dev)
        adjoint_step_kernel<float><<<grid, block, 0, s>>>((const float*)fstate, lam_in, lam_out,
                                                          force, d.nx, d.ny, d.members, tau0, K,
                                                          mu, k_partial);
    else
        adjoint_step_kernel<double><<<grid, block, 0, s>>>((const double*)fstate, lam_in,
                                                           lam_out, force, d.nx, d.ny, d.members,
                                                           tau0, K, mu, k_partial);
    return hipGetLastError();
}

// Small problems only, where a step's launch and latency cost more than its work: up to
// P = 7e4 node-members for at most five members and 2e4 for more, whose blocks take one or two
// members and with them an eighth of each line they touch.  us of a reverse sweep of ten steps
// (about 40 of them its other launches), single / this: 1 member 84 / 51 at P = 3e3, 154 / 81 at
// 7e4; 5 members 82 / 53, 134 / 110; 8 members 82 / 56, 82 / 72 at 1.5e4; 24 members 82 / 53,
// 83 / 69 at 1.5e4, but 90 / 125 at 6e4 (40 members 86 / 115 at 5e4).  Of the
// shapes with one block per CU at most, the best by a fit of a sweep: a launch 2.5 us, a
// step 1.5 us and 2.5 us more per 1024 threads of the block.
StepPlan adjoint_plan(LbmDims d, int interval, int capacity) {
    StepPlan best{};
    if (interval < 2 || (double)d.nx * d.ny * d.members > (d.members <= 5 ? 7e4 : 2e4)) return best;
    double least = 1e30;
    for (int mg = 1; mg <= 4 && mg <= d.members; mg *= 2)
        for (int k = 2; k <= 6 && k <= interval; ++k)
            for (int tile = 4; tile <= 24; tile += 2) {
                const StepPlan pl{k, tile + 2 * (k - 1), tile + 2 * (k - 1), mg, 1};
                const int threads = pl.rx * pl.ry * mg;
                if (threads > 1024 || tile_blocks(d, pl) > std::min(256, capacity)) continue;
                const double t = 2.5 / k + 1.5 + 2.5 * threads / 1024;
                if (t < least) {
                    least = t;
                    best = pl;
                }
            }
    return best;
}

namespace {
template <typename T>
hipError_t launch_adjoint_tile_t(const void* fhi, const void* flast, size_t stride_bytes,
                                 const double* lam_in, double* lam_out, const double* force,
                                 LbmDims d, double tau0, double K, double mu, double* k_partial,
                                 int capacity, const StepPlan& pl, int steps, hipStream_t s) {
    const int R = pl.rx - 2 * (pl.steps - steps);
    const int tile = R - 2 * (steps - 1);
    const int blocks = tile_blocks(d, pl);
    const int threads = (R * R * pl.members + kWave - 1) / kWave * kWave;
    const size_t lds = (size_t)9 * R * R * pl.members * sizeof(double);
    constexpr size_t kMostLds = 80 * 1024;  // every plan's region: two blocks per CU
    if (tile < 1 || threads > 1024 || lds > kMostLds || blocks > capacity)
        return hipErrorInvalidValue;
    static std::atomic<uint64_t> lds_ok{0};
    const hipError_t e = allow_lds(adjoint_tile_kernel<T>, kMostLds, &lds_ok);
    if (e != hipSuccess) return e;
    adjoint_tile_kernel<T><<<blocks, threads, lds, s>>>(
        (const T*)fhi, (const T*)flast, stride_bytes / sizeof(T), lam_in, lam_out, force, d.nx, d.ny,
        d.members, tau0, K, mu, R, pl.members, steps, k_partial);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_adjoint_tile(const void* fhi, const void* flast, size_t stride_bytes,
                               const double* lam_in, double* lam_out, const double* force, LbmDims d,
                               double tau0, double cs, double mu, int storage, double* k_partial,
                               int capacity, const StepPlan& pl, int steps, hipStream_t s) {
    if (steps < 1 || steps > pl.steps) return hipErrorInvalidValue;
    const double K = 18.0 * sqrt(2.0) * cs * cs;
    return storage == kStoreF32Dev
               ? launch_adjoint_tile_t<float>(fhi, flast, stride_bytes, lam_in, lam_out, force, d,
                                              tau0, K, mu, k_partial, capacity, pl, steps, s)
               : launch_adjoint_tile_t<double>(fhi, flast, stride_bytes, lam_in, lam_out, force, d,
                                               tau0, K, mu, k_partial, capacity, pl, steps, s);
}

hipError_t launch_lam_to_canonical(const double* lam, double* out, LbmDims d, hipStream_t s) {
    const size_t total = (size_t)d.nx * d.ny * 9 * d.members;
    size_t g = (total + 255) / 256;
    lam_to_canonical_kernel<<<(int)(g > 65536 ? 65536 : g), 256, 0, s>>>(lam, out, d.nx * d.ny,
                                                                         d.members);
    return hipGetLastError();
}

hipError_t launch_misfit(const void* f, const int* pts, int npts, int nvar, const double* yo,
                         double* lam, double* jbuf, bool first, LbmDims d, int storage,
                         hipStream_t s) {
    const int total = npts * d.members;
    if (storage == kStoreF32Dev)
        misfit_kernel<float><<<(total + 127) / 128, 128, 0, s>>>((const float*)f, pts, npts, nvar,
                                                                 yo, lam, jbuf, first, d.nx,
                                                                 d.ny, d.members);
    else
        misfit_kernel<double><<<(total + 127) / 128, 128, 0, s>>>((const double*)f, pts, npts,
                                                                  nvar, yo, lam, jbuf, first, d.nx,
                                                                  d.ny, d.members);
    return hipGetLastError();
}

hipError_t launch_sum(const double* v, size_t n, double scale, double* out, hipStream_t s) {
    sum_kernel<<<1, 256, 0, s>>>(v, n, scale, out);
    return hipGetLastError();
}

hipError_t launch_zero2(double* v0, size_t n0, double* v1, size_t n1, hipStream_t s) {
    const size_t g = (n0 + n1 + 255) / 256;
    zero2_kernel<<<(int)(g > 65536 ? 65536 : (g == 0 ? 1 : g)), 256, 0, s>>>(v0, n0, v1, n1);
    return hipGetLastError();
}

}  // namespace lbmletkf
