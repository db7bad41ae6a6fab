// HIP kernels (gfx950) of the Cole-Hopf fourth-order MRT-LB solver.
//
// Data layout: a state buffer holds the q populations of every node in the
// chunked structure-of-arrays order of `slot` (lbm_kernels.h).  It is kept
// "stream-shifted": the slot of population i at node k holds f_i(k + e_i),
// the population that node k sent along e_i after its last collision, so one
// time step is a pull:
//     f_i(x) = src_i(x - e_i)          (pre-collision distribution at x)
//     dst_i(x) = (C f(x))_i            (collision, Sec. III.A)
// Every store is aligned and coalesced; the loads of a wavefront are 64
// consecutive doubles shifted by at most one element.  The update is
// HBM-bound (q*8 bytes read + q*8 written per node and step, a few flops per
// byte), so no matrix cores are used.
//
// Every thread owns one node; a block is 256 consecutive nodes of one row;
// y and (3-D) z run over grid.y and grid.z.
#include <algorithm>
#include <cmath>

#include "lbm_device.h"

namespace lbm {
namespace {

// ---------------------------------------------------------------------------
// time step
// ---------------------------------------------------------------------------
// RIN: src was written by a collision, so a twin population is read from
// the plane of the population it equals (twin<D>); WOUT: the twins are not
// stored (dst then holds a state that only a RIN read may use).  Both leave
// the arithmetic, and so the result, bitwise unchanged.
template <int D, bool RIN = false, bool WOUT = false, bool NT = true>
__global__ void __launch_bounds__(256) k_step(const double* __restrict__ src,
                                              double* __restrict__ dst, Geo g, Rates r) {
    constexpr int Q = Lat<D>::Q;
    int c[4];
    if (!thread_node<D>(g, c)) return;
    const Nbr nb = make_nbr<D>(c, g);
    double f[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) f[i] = src[slot<Q>(RIN ? twin<D>(i) : i, pull_index<D>(nb, i))];
    collide<D>(f, r);
    const int k = node_index(g, c);
#pragma unroll
    for (int i = 0; i < Q; ++i)
        if (!WOUT || twin<D>(i) == i) {
            if constexpr (NT)
                __builtin_nontemporal_store(f[i], dst + slot<Q>(i, k));
            else
                dst[slot<Q>(i, k)] = f[i];
        }
}

// ---------------------------------------------------------------------------
// initialisation
// ---------------------------------------------------------------------------
// Fourth-order central difference of theta along axis a at node c.
template <int D>
__device__ double fd4(const double* __restrict__ th, const Geo& g, const int (&c)[4], int a,
                      double inv12dx) {
    const int n[4] = {g.nx, g.ny, g.nz, g.nw};
    double v[4];
    const int off[4] = {2, 1, -1, -2};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        int cc[4] = {c[0], c[1], c[2], c[3]};
        cc[a] = wrapi(c[a] + off[t], n[a]);
        v[t] = th[node_index(g, cc)];
    }
    return ((v[3] - v[0]) + 8.0 * (v[1] - v[2])) * inv12dx;
}

// dst_i(y) = f0_i(y + e_i) with the closed-form initial distribution
// f0_i = w_i theta0 - dx w_i (e_i . g) - (1/s1 - 1)(dx/6) sum_a (d_{i,+a} - d_{i,-a}) g_a.
// GRAD: g is given; its values and theta0 are gathered at the push targets, whose
// lines the neighbouring threads read too (wrapping by a modulo per population and
// axis: 128^3 128 us; now 74, 2048^2 140 and 65; 512^3, 25 GB, 9.3 and 8.4 ms, held by
// the rate of its 19 write streams).
// Otherwise g is the fourth-order difference of theta0.
template <int D, bool GRAD, bool NT>
__global__ void __launch_bounds__(256) k_init(const double* __restrict__ th0,
                                              const double* __restrict__ grad,
                                              double* __restrict__ dst, Geo g, Rates r) {
    constexpr int Q = Lat<D>::Q;
    int c[4];
    if (!thread_node<D>(g, c)) return;
    const int k = node_index(g, c);
    const double corr = r.inv_s1_m1 * r.dx * (1.0 / 6.0);
    const int n[4] = {g.nx, g.ny, g.nz, g.nw};
    const Nbr nb = make_nbr<D>(c, g);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const int src = push_index<D>(nb, i);
        const double t = th0[src];
        double eg = 0.0, ax = 0.0;
        int cs[4] = {};
        if constexpr (!GRAD) {
#pragma unroll
            for (int b = 0; b < 4; ++b) cs[b] = wrapi(c[b] + Lat<D>::E[i][b], n[b]);
        }
#pragma unroll
        for (int a = 0; a < D; ++a) {
            const int e = Lat<D>::E[i][a];
            if (e == 0) continue;
            double ga;
            if constexpr (GRAD)
                ga = grad[(int64_t)a * g.V + src];
            else
                ga = fd4<D>(th0, g, cs, a, r.inv12dx);
            eg = e == 1 ? eg + ga : eg - ga;
            if (nnz<D>(i) == 1) ax = e == 1 ? ga : -ga;
        }
        const double w = weight<D>(i, r);
        const double f0 = w * t - r.dx * w * eg - corr * ax;
        if constexpr (NT)
            __builtin_nontemporal_store(f0, dst + slot<Q>(i, k));
        else
            dst[slot<Q>(i, k)] = f0;
    }
}

// ---------------------------------------------------------------------------
// macroscopic output, state conversions
// ---------------------------------------------------------------------------
// theta = sum f, u_a = (2 - s1) c j_a / theta and grad_a theta = -(3 s1/dx) j_a
// with j_a = sum_i e_{ia} f_i (Sec. III.C; sum_i e_i w_i = 0, so j needs no
// equilibrium subtracted).  Any of the three outputs may be NULL.
template <int D>
__global__ void __launch_bounds__(256) k_macro(const double* __restrict__ src,
                                               double* __restrict__ theta, double* __restrict__ u,
                                               double* __restrict__ grad, Geo g, Rates r) {
    constexpr int Q = Lat<D>::Q;
    int c[4];
    if (!thread_node<D>(g, c)) return;
    const Nbr nb = make_nbr<D>(c, g);
    double f[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) f[i] = src[slot<Q>(i, pull_index<D>(nb, i))];
    double th = 0.0;
#pragma unroll
    for (int i = 0; i < Q; ++i) th += f[i];
    const int k = node_index(g, c);
    if (theta) theta[k] = th;
    if (u || grad) {
        const double inv = r.ucoef / th;
#pragma unroll
        for (int a = 0; a < D; ++a) {
            double j = 0.0;
#pragma unroll
            for (int i = 0; i < Q; ++i) j = LBM_SADD(j, Lat<D>::E[i][a], f[i]);
            if (u) u[(int64_t)a * g.V + k] = j * inv;
            if (grad) grad[(int64_t)a * g.V + k] = r.gcoef * j;
        }
    }
}

template <int D>
__global__ void __launch_bounds__(256) k_get_state(const double* __restrict__ src,
                                                   double* __restrict__ dense, Geo g) {
    constexpr int Q = Lat<D>::Q;
    int c[4];
    if (!thread_node<D>(g, c)) return;
    const Nbr nb = make_nbr<D>(c, g);
    const int k = node_index(g, c);
#pragma unroll
    for (int i = 0; i < Q; ++i) dense[(int64_t)i * g.V + k] = src[slot<Q>(i, pull_index<D>(nb, i))];
}

template <int D>
__global__ void __launch_bounds__(256) k_set_state(const double* __restrict__ dense,
                                                   double* __restrict__ dst, Geo g) {
    constexpr int Q = Lat<D>::Q;
    int c[4];
    if (!thread_node<D>(g, c)) return;
    const Nbr nb = make_nbr<D>(c, g);
    const int k = node_index(g, c);
#pragma unroll
    for (int i = 0; i < Q; ++i) dst[slot<Q>(i, k)] = dense[(int64_t)i * g.V + push_index<D>(nb, i)];
}

// Canonical (no stream shift) conversions between a dense q x V array and
// the chunked layout, for distribution-shaped adjoint buffers.
template <int D>
__global__ void __launch_bounds__(256) k_layout_from_dense(const double* __restrict__ dense,
                                                           double* __restrict__ buf, Geo g) {
    constexpr int Q = Lat<D>::Q;
    int c[4];
    if (!thread_node<D>(g, c)) return;
    const int k = node_index(g, c);
#pragma unroll
    for (int i = 0; i < Q; ++i) buf[slot<Q>(i, k)] = dense[(int64_t)i * g.V + k];
}

template <int D>
__global__ void __launch_bounds__(256) k_layout_to_dense(const double* __restrict__ buf,
                                                         double* __restrict__ dense, Geo g) {
    constexpr int Q = Lat<D>::Q;
    int c[4];
    if (!thread_node<D>(g, c)) return;
    const int k = node_index(g, c);
#pragma unroll
    for (int i = 0; i < Q; ++i) dense[(int64_t)i * g.V + k] = buf[slot<Q>(i, k)];
}

// Sets *flag (pinned host memory: a plain store of 1 from whichever waves find one)
// when theta = sum_i f_i of some node of the state is not finite and positive (a
// diverged or corrupted run: u = -2 nu grad theta / theta needs theta > 0).
template <int D>
__global__ void __launch_bounds__(256) k_check_state(const double* __restrict__ src, int* flag,
                                                     Geo g) {
    constexpr int Q = Lat<D>::Q;
    int c[4];
    if (!thread_node<D>(g, c)) return;
    const Nbr nb = make_nbr<D>(c, g);
    double th = 0.0;
#pragma unroll
    for (int i = 0; i < Q; ++i) th += src[slot<Q>(i, pull_index<D>(nb, i))];
    if (!(th > 0.0) || !isfinite(th)) *(volatile int*)flag = 1;
}

__global__ void __launch_bounds__(256) k_check_theta(const double* __restrict__ th, int64_t n,
                                                     int* flag) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const double v = th[i];
    if (!(v > 0.0) || !isfinite(v)) atomicOr(flag, 1);
}

// ---------------------------------------------------------------------------
// adjoint
// ---------------------------------------------------------------------------
template <int D>
__global__ void __launch_bounds__(256) k_macro_adjoint(const double* __restrict__ src,
                                                       const double* __restrict__ gth,
                                                       const double* __restrict__ gu,
                                                       double* __restrict__ lam,
                                                       double* __restrict__ partials, Geo g,
                                                       Rates r) {
    constexpr int Q = Lat<D>::Q;
    int c[4];
    double ge = 0.0;
    if (thread_node<D>(g, c)) {
        const Nbr nb = make_nbr<D>(c, g);
        const int k = node_index(g, c);
        double f[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) f[i] = src[slot<Q>(i, pull_index<D>(nb, i))];
        double th = 0.0;
#pragma unroll
        for (int i = 0; i < Q; ++i) th += f[i];
        const double inv = 1.0 / th;
        const double gt = gth ? gth[k] : 0.0;
        double base = gt, coef[D];
#pragma unroll
        for (int a = 0; a < D; ++a) {
            double j = 0.0;
#pragma unroll
            for (int i = 0; i < Q; ++i) j = LBM_SADD(j, Lat<D>::E[i][a], f[i]);
            const double ga = gu ? gu[(int64_t)a * g.V + k] : 0.0;
            const double ua = r.ucoef * j * inv;
            // d u_a / d f_i = (2 - s1) c e_ia / theta - u_a / theta
            base -= ga * ua * inv;
            coef[a] = ga * r.ucoef * inv;
            // d u_a / d eps = -s1' c j_a / theta
            ge += ga * (-r.ds1) * r.c * j * inv;
        }
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            double v = base;
#pragma unroll
            for (int a = 0; a < D; ++a) v = LBM_SADD(v, Lat<D>::E[i][a], coef[a]);
            lam[slot<Q>(i, k)] = v;
        }
    }
    const double s = block_sum(ge);
    if (threadIdx.x == 0 && threadIdx.y == 0) partials[block_linear()] = s;
}

// lam_out(x) = C^T mu(x), mu_i(x) = lam_in_i(x + e_i); eps part <mu, C' f^n(x)>.
// One partial per block; blocks past the grid up to ntab - 1 are written zero.
// RIN: the state was written by a collision (twins read as in k_step).
template <int D, bool RIN = false>
__global__ void __launch_bounds__(256) k_adjoint_step(const double* __restrict__ state,
                                                      const double* __restrict__ lin,
                                                      double* __restrict__ lout,
                                                      double* __restrict__ partials,
                                                      int64_t ntab, Geo g, Rates r) {
    constexpr int Q = Lat<D>::Q;
    int c[4];
    double ge = 0.0;
    if (thread_node<D>(g, c)) {
        const Nbr nb = make_nbr<D>(c, g);
        const int k = node_index(g, c);
        double f[Q], mu[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            f[i] = state[slot<Q>(RIN ? twin<D>(i) : i, pull_index<D>(nb, i))];
            mu[i] = lin[slot<Q>(i, push_index<D>(nb, i))];
        }
        double df[Q];
        collide_deps<D>(f, r, df);
#pragma unroll
        for (int i = 0; i < Q; ++i) ge += mu[i] * df[i];
        double lam[Q];
        collide_adjoint<D>(mu, r, lam);
#pragma unroll
        for (int i = 0; i < Q; ++i) lout[slot<Q>(i, k)] = lam[i];
    }
    const double s = block_sum(ge);
    if (threadIdx.x == 0 && threadIdx.y == 0) {
        const int64_t b = block_linear();
        const int64_t nb = (int64_t)gridDim.x * gridDim.y * gridDim.z;
        partials[b] = s;
        for (int64_t t = nb + b; t < ntab; t += nb) partials[t] = 0.0;
    }
}

// h_a(x) = d L / d g_a(x) for the gradient input of the initialisation:
//   h_a = -dx [ sum_i w_i e_ia lam_i + (1/s1 - 1)(1/6)(lam_{+a} - lam_{-a}) ].
template <int D>
__device__ __forceinline__ double init_h(const double* __restrict__ lam, const Geo& g, int k,
                                         int a, const Rates& r) {
    constexpr int Q = Lat<D>::Q;
    double s = 0.0, ax = 0.0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const int e = Lat<D>::E[i][a];
        if (e == 0) continue;
        const double l = lam[slot<Q>(i, k)];
        const double wl = weight<D>(i, r) * l;
        s = e == 1 ? s + wl : s - wl;
        if (nnz<D>(i) == 1) ax = e == 1 ? ax + l : ax - l;
    }
    return -r.dx * (s + r.inv_s1_m1 * (1.0 / 6.0) * ax);
}

template <int D>
__global__ void __launch_bounds__(256) k_init_adjoint(const double* __restrict__ th0,
                                                      const double* __restrict__ grad,
                                                      const double* __restrict__ lam,
                                                      double* __restrict__ gth,
                                                      double* __restrict__ ggrad,
                                                      double* __restrict__ partials, Geo g,
                                                      Rates r) {
    constexpr int Q = Lat<D>::Q;
    int c[4];
    double ge = 0.0;
    if (thread_node<D>(g, c)) {
        const int k = node_index(g, c);
        double l[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) l[i] = lam[slot<Q>(i, k)];
        double gt = 0.0;
#pragma unroll
        for (int i = 0; i < Q; ++i) gt += weight<D>(i, r) * l[i];
        double gv[D];
#pragma unroll
        for (int a = 0; a < D; ++a)
            gv[a] = grad ? grad[(int64_t)a * g.V + k] : fd4<D>(th0, g, c, a, r.inv12dx);
        if (grad) {
            if (ggrad) {
#pragma unroll
                for (int a = 0; a < D; ++a) ggrad[(int64_t)a * g.V + k] = init_h<D>(lam, g, k, a, r);
            }
        } else {
            // g_theta0 += sum_a D_a^T h_a, D_a^T h(x) = (-h(x-2) + 8h(x-1) - 8h(x+1) + h(x+2)) / (12 dx)
            const int n[4] = {g.nx, g.ny, g.nz, g.nw};
#pragma unroll
            for (int a = 0; a < D; ++a) {
                const int off[4] = {-2, -1, 1, 2};
                const double cf[4] = {-1.0, 8.0, -8.0, 1.0};
                double acc = 0.0;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    int cc[4] = {c[0], c[1], c[2], c[3]};
                    cc[a] = wrapi(c[a] + off[t], n[a]);
                    acc += cf[t] * init_h<D>(lam, g, node_index(g, cc), a, r);
                }
                gt += acc * r.inv12dx;
            }
        }
        gth[k] = gt;
        // d f0_i / d eps = w_i' theta0 - dx w_i' (e_i . g) - (d(1/s1)/deps)(dx/6) (+-g_a on axis i)
        const double t0 = th0[k];
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            double eg = 0.0, ax = 0.0;
#pragma unroll
            for (int a = 0; a < D; ++a) {
                const int e = Lat<D>::E[i][a];
                if (e == 0) continue;
                eg = e == 1 ? eg + gv[a] : eg - gv[a];
                if (nnz<D>(i) == 1) ax = e == 1 ? gv[a] : -gv[a];
            }
            const double dw = dweight<D>(i, r);
            const double df = dw * t0 - r.dx * dw * eg - r.dinv_s1 * r.dx * (1.0 / 6.0) * ax;
            ge += l[i] * df;
        }
    }
    const double s = block_sum(ge);
    if (threadIdx.x == 0 && threadIdx.y == 0) partials[block_linear()] = s;
}

// *g_eps += sum of the partials; then, if g_nu != NULL, *g_nu = nu_scale * *g_eps
// (dL/dnu = (dt/dx^2) dL/deps, since eps = nu dt/dx^2).
__global__ void __launch_bounds__(256) k_finalize(const double* __restrict__ partials, int64_t n,
                                                  double* g_eps, double* g_nu, double nu_scale) {
    double v = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) v += partials[i];
    const double s = block_sum(v);
    if (threadIdx.x == 0) {
        const double ge = *g_eps + s;
        *g_eps = ge;
        if (g_nu) *g_nu = nu_scale * ge;
    }
}

// The reductions of k_finalize for m tables: block j sums table j with the
// same tree into sums[j]; k_accumulate then adds sums[m-1], ..., sums[0] to
// *g_eps one at a time, the order of m k_finalize launches.
__global__ void __launch_bounds__(256) k_table_sums(const double* __restrict__ partials, int64_t n,
                                                    double* __restrict__ sums) {
    const double* p = partials + (int64_t)blockIdx.x * n;
    double v = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) v += p[i];
    const double s = block_sum(v);
    if (threadIdx.x == 0) sums[blockIdx.x] = s;
}

__global__ void __launch_bounds__(64) k_accumulate(const double* __restrict__ sums, int64_t m,
                                                   double* g_eps) {
    if (threadIdx.x != 0) return;
    double acc = *g_eps;
    for (int64_t j = m - 1; j >= 0; --j) acc += sums[j];
    *g_eps = acc;
}

// ---------------------------------------------------------------------------
// Burgers front end: theta0 from the initial velocity u0 (inverse Cole-Hopf
// transformation, Sec. II: u = -2 nu grad(theta)/theta, so theta0 =
// exp(-phi/(2 nu)) with grad(phi) = u0).  phi is integrated along the path
// that runs along x_0 at x_1 = .. = 0, then along x_1 at x_2 = .. = 0, and so
// on; each cell integral uses the cubic through four nodes,
//     int_{x_j}^{x_j+1} u = dx (-u_{j-1} + 13 u_j + 13 u_{j+1} - u_{j+2}) / 24,
// (periodic indices).  phi = 0 at the origin.
// ---------------------------------------------------------------------------

// A line of axis a is (c_0..c_{a-1}, *, 0..0); its node j stands at line + lead j of
// the field (lead = n_0 .. n_{a-1}, also the number of lines), and at the same place
// of the axis' part of the workspace.  The lines are cut into segments of L nodes:
// k_potential_cells gives every node the integral from its segment's first node and
// every segment its total, k_potential_offsets turns the totals into the integrals up
// to the segments, and k_theta_from_potential adds the two.  (One thread per line
// walked the whole line: 0.6 ms for axis 0 and 1.0 ms for axis 1 at 2048^2; now
// 18 and 10 us for both axes.)
struct PotentialAxes {
    int64_t lines[4], part[4], total[4];  // lines; first element of the parts / totals
    int64_t first[5];                     // first thread of k_potential_cells, all axes
    int n[4], L[4], nseg[4];
    int d;
};

__global__ void __launch_bounds__(256) k_potential_cells(const double* __restrict__ u0, int64_t V,
                                                         double* __restrict__ work,
                                                         PotentialAxes ax, double dx) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= ax.first[ax.d]) return;
    int a = 0;
    while (t >= ax.first[a + 1]) ++a;
    const int64_t lead = ax.lines[a], seg = (t - ax.first[a]) / lead;
    const int64_t line = (t - ax.first[a]) - seg * lead;
    const int n = ax.n[a], j0 = (int)seg * ax.L[a], j1 = min(j0 + ax.L[a], n);
    const double* u = u0 + (int64_t)a * V + line;
    double* part = work + ax.part[a] + line;
    double um = u[lead * (j0 == 0 ? n - 1 : j0 - 1)], uc = u[lead * j0];
    double up = u[lead * (j0 + 1 < n ? j0 + 1 : j0 + 1 - n)];
    int jn = j0 + 2 < n ? j0 + 2 : wrapi(j0 + 2, n);  // node j + 2
    double phi = 0.0;
#pragma unroll 8
    for (int j = j0; j < j1; ++j) {
        part[lead * j] = phi;
        const double un = u[lead * jn];
        jn = jn + 1 == n ? 0 : jn + 1;
        phi += dx * ((13.0 * (uc + up) - (um + un)) / 24.0);
        um = uc;
        uc = up;
        up = un;
    }
    work[ax.total[a] + seg * lead + line] = phi;
}

// totals of a line, segment by segment -> integral up to each segment
__global__ void __launch_bounds__(256) k_potential_offsets(double* __restrict__ work,
                                                           PotentialAxes ax) {
    int64_t line = (int64_t)blockIdx.x * 256 + threadIdx.x;
    int a = 0;
    while (a < ax.d && line >= ax.lines[a]) line -= ax.lines[a++];
    if (a == ax.d) return;
    double* tot = work + ax.total[a] + line;
    double phi = 0.0;
#pragma unroll 8
    for (int s = 0; s < ax.nseg[a]; ++s) {
        const double v = tot[ax.lines[a] * s];
        tot[ax.lines[a] * s] = phi;
        phi += v;
    }
}

// theta0 = exp(-(sum_a phi_a)/(2 nu)); grad theta0 = -u0 theta0/(2 nu).
template <int D>
__global__ void __launch_bounds__(256) k_theta_from_potential(const double* __restrict__ u0,
                                                              const double* __restrict__ work,
                                                              double* __restrict__ theta,
                                                              double* __restrict__ grad, Geo g,
                                                              double inv2nu, PotentialAxes ax) {
    int c[4];
    if (!thread_node<D>(g, c)) return;
    double phi = 0.0;
    int64_t line = 0, stride = 1;
#pragma unroll
    for (int a = 0; a < D; ++a) {
        const int seg = c[a] / ax.L[a];
        phi += work[ax.part[a] + line + stride * c[a]] + work[ax.total[a] + stride * seg + line];
        line += stride * c[a];
        stride *= ax.n[a];
    }
    const int k = node_index(g, c);
    const double th = exp(-phi * inv2nu);
    theta[k] = th;
    if (grad) {
#pragma unroll
        for (int a = 0; a < D; ++a) grad[(int64_t)a * g.V + k] = -u0[(int64_t)a * g.V + k] * th * inv2nu;
    }
}

}  // namespace

Launch launch_shape(int d, const Geo& g) {
    Launch L;
    if (d == 1) {
        L.block = dim3(B1, 1, 1);
        L.grid = dim3((unsigned)((g.nx + B1 - 1) / B1), 1, 1);
    } else {
        // 256 threads: a whole row segment of 256 nodes, or for rows of at
        // most 128 (64) nodes 2 (4) rows of 128 (64), so that short rows do
        // not leave most of a block idle (64^4: one row of 64 per block left
        // three of its four waves without a node)
        const int bx = g.nx > 128 ? BX : (g.nx > 64 ? 128 : 64);
        const int by = BX * BY / bx;
        L.block = dim3(bx, by, 1);
        L.grid = dim3((unsigned)((g.nx + bx - 1) / bx), (unsigned)((g.ny + by - 1) / by),
                      (unsigned)(d >= 3 ? g.nz * g.nw : 1));
    }
    L.nblocks = (int64_t)L.grid.x * L.grid.y * L.grid.z;
    return L;
}

#define LBM_LAUNCH(kern, ...)                                                     \
    dispatch(d, [&](auto dc) {                                                    \
        constexpr int DD = decltype(dc)::value;                                   \
        const Launch L = launch_shape(DD, g);                                     \
        hipLaunchKernelGGL(kern<DD>, L.grid, L.block, 0, st, __VA_ARGS__);        \
        return hipGetLastError();                                                 \
    })

hipError_t launch_step(int d, const Geo& g, const Rates& r, const double* src, double* dst,
                       hipStream_t st, bool rin, bool wout, int states) {
    return dispatch(d, [&](auto dc) {
        constexpr int DD = decltype(dc)::value;
        const Launch L = launch_shape(DD, g);
        // two 1-D states that fit in the L2s are not stored through them: a step is short
        // enough there for the write-back at its end to count (us for 40 steps, cached and
        // not: 600,000 nodes 194 and 163, 1,000,000 331 and 368)
        constexpr uint64_t kL2Bytes = 32ull << 20;
        const bool nt = !states_fit_cache(DD, g, states) ||
                        (DD == 1 && 2ull * 3 * (uint64_t)g.V * sizeof(double) <= kL2Bytes);
        if constexpr (DD == 1) {  // D1Q3 has no twins
            return dispatch_io(nt, false, [&](auto n, auto) {
                hipLaunchKernelGGL((k_step<1, false, false, decltype(n)::value>), L.grid, L.block,
                                   0, st, src, dst, g, r);
                return hipGetLastError();
            });
        } else {
            return dispatch_io(rin, wout, [&](auto ri, auto wo) {
                return dispatch_io(nt, false, [&](auto n, auto) {
                    hipLaunchKernelGGL((k_step<DD, decltype(ri)::value, decltype(wo)::value,
                                               decltype(n)::value>),
                                       L.grid, L.block, 0, st, src, dst, g, r);
                    return hipGetLastError();
                });
            });
        }
    });
}

hipError_t launch_init(int d, const Geo& g, const Rates& r, const double* theta0,
                       const double* grad, double* dst, hipStream_t st) {
    return dispatch(d, [&](auto dc) {
        constexpr int DD = decltype(dc)::value;
        const Launch L = launch_shape(DD, g);
        // one state: the next call reads it, also where two do not fit (us, init to fields
        // around eight steps, non-temporal and cached: 1400 x 1350 157 and 145, 118^3, 250 MB,
        // 522 and 499; 2048^2, 302 MB, 323 and 322, without steps 192 and 200)
        return dispatch_io(grad != nullptr, !states_fit_cache(DD, g, 1), [&](auto gr, auto nt) {
            hipLaunchKernelGGL((k_init<DD, decltype(gr)::value, decltype(nt)::value>), L.grid,
                               L.block, 0, st, theta0, grad, dst, g, r);
            return hipGetLastError();
        });
    });
}

hipError_t launch_macro(int d, const Geo& g, const Rates& r, const double* state, double* theta,
                        double* u, double* grad, hipStream_t st) {
    return LBM_LAUNCH(k_macro, state, theta, u, grad, g, r);
}

hipError_t launch_check_state(int d, const Geo& g, const double* state, int* flag,
                              hipStream_t st) {
    return LBM_LAUNCH(k_check_state, state, flag, g);
}

hipError_t launch_get_state(int d, const Geo& g, const double* state, double* dense,
                            hipStream_t st) {
    return LBM_LAUNCH(k_get_state, state, dense, g);
}

hipError_t launch_set_state(int d, const Geo& g, const double* dense, double* state,
                            hipStream_t st) {
    return LBM_LAUNCH(k_set_state, dense, state, g);
}

hipError_t launch_layout_from_dense(int d, const Geo& g, const double* dense, double* buf,
                                   hipStream_t st) {
    return LBM_LAUNCH(k_layout_from_dense, dense, buf, g);
}

hipError_t launch_layout_to_dense(int d, const Geo& g, const double* buf, double* dense,
                                 hipStream_t st) {
    return LBM_LAUNCH(k_layout_to_dense, buf, dense, g);
}

// Segments of about sqrt(n) nodes, 16 to 64: a line is then one walk over a segment
// and one over its segments.
static PotentialAxes potential_axes(int d, const Geo& g, int64_t* doubles) {
    PotentialAxes ax = {};
    const int n[4] = {g.nx, g.ny, g.nz, g.nw};
    ax.d = d;
    int64_t lead = 1, parts = 0, at = 0;
    for (int a = 0; a < d; ++a) {
        ax.n[a] = n[a];
        ax.L[a] = std::min(64, std::max(16, (int)std::sqrt((double)n[a])));
        ax.nseg[a] = (n[a] + ax.L[a] - 1) / ax.L[a];
        ax.lines[a] = lead;
        ax.first[a] = at;
        at += lead * ax.nseg[a];
        ax.part[a] = parts;
        lead *= n[a];
        parts += lead;
    }
    ax.first[d] = at;
    for (int a = 0; a < d; ++a) {
        ax.total[a] = parts;
        parts += ax.lines[a] * ax.nseg[a];
    }
    if (doubles) *doubles = parts;
    return ax;
}

int64_t potential_workspace(int d, const Geo& g) {
    int64_t n = 0;
    (void)potential_axes(d, g, &n);
    return n;
}

hipError_t launch_theta_from_velocity(int d, const Geo& g, double dx, double nu, const double* u0,
                                      double* work, double* theta, double* grad,
                                      hipStream_t st) {
    const PotentialAxes ax = potential_axes(d, g, nullptr);
    int64_t lines = 0;
    for (int a = 0; a < d; ++a) lines += ax.lines[a];
    hipLaunchKernelGGL(k_potential_cells, dim3((unsigned)((ax.first[d] + 255) / 256)), dim3(256), 0,
                       st, u0, g.V, work, ax, dx);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_potential_offsets, dim3((unsigned)((lines + 255) / 256)), dim3(256), 0, st,
                       work, ax);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const double inv2nu = 1.0 / (2.0 * nu);
    return LBM_LAUNCH(k_theta_from_potential, u0, work, theta, grad, g, inv2nu, ax);
}

hipError_t launch_check_theta(const double* theta, int64_t n, int* flag, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_check_theta, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, theta,
                       n, flag);
    return hipGetLastError();
}

hipError_t launch_macro_adjoint(int d, const Geo& g, const Rates& r, const double* state,
                                const double* g_theta, const double* g_u, double* lambda,
                                double* partials, hipStream_t st) {
    return LBM_LAUNCH(k_macro_adjoint, state, g_theta, g_u, lambda, partials, g, r);
}

hipError_t launch_adjoint_step(int d, const Geo& g, const Rates& r, const double* state,
                               const double* lam_in, double* lam_out, double* partials,
                               int64_t ntab, hipStream_t st, bool rin) {
    if (ntab < launch_shape(d, g).nblocks) return hipErrorInvalidValue;
    return dispatch(d, [&](auto dc) {
        constexpr int DD = decltype(dc)::value;
        const Launch L = launch_shape(DD, g);
        constexpr bool HAS_TWINS = DD > 1;  // D1Q3 has none
        if (HAS_TWINS && rin)
            hipLaunchKernelGGL((k_adjoint_step<DD, HAS_TWINS>), L.grid, L.block, 0, st, state,
                               lam_in, lam_out, partials, ntab, g, r);
        else
            hipLaunchKernelGGL((k_adjoint_step<DD, false>), L.grid, L.block, 0, st, state, lam_in,
                               lam_out, partials, ntab, g, r);
        return hipGetLastError();
    });
}

hipError_t launch_init_adjoint(int d, const Geo& g, const Rates& r, const double* theta0,
                               const double* grad, const double* lambda0, double* g_theta0,
                               double* g_grad, double* partials, hipStream_t st) {
    return LBM_LAUNCH(k_init_adjoint, theta0, grad, lambda0, g_theta0, g_grad, partials, g, r);
}

hipError_t launch_finalize(const double* partials, int64_t n, double* g_eps, hipStream_t st,
                           double* g_nu, double nu_scale) {
    hipLaunchKernelGGL(k_finalize, dim3(1), dim3(256), 0, st, partials, n, g_eps, g_nu, nu_scale);
    return hipGetLastError();
}

hipError_t launch_finalize_tables(const double* partials, int64_t n, int64_t m, double* sums,
                                  double* g_eps, hipStream_t st) {
    if (m < 1 || m > (int64_t)INT32_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_table_sums, dim3((unsigned)m), dim3(256), 0, st, partials, n, sums);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_accumulate, dim3(1), dim3(64), 0, st, sums, m, g_eps);
    return hipGetLastError();
}

}  // namespace lbm
