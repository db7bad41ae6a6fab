// 1-D kernels: whole runs of small grids in one launch, and the bounded interval.
#include "lbm_device.h"

namespace lbm {
namespace {

// Small 1-D grids (n <= RESIDENT_MAX_1D): the whole state lives in LDS and
// one workgroup of T threads (PER nodes each, T * PER >= n) advances all
// nsteps in a single launch, so the run is not bound by one kernel launch per
// step; the smallest fitting shape keeps the per-step work and barrier cost
// proportional to n.  Same collision as k_step<1>.
//
// With walls != NULL the interval is bounded (wall_pull1): step s forms the
// distribution of the time whose boundary theta is wall_now (s = 0) or
// walls[2(s-1) .. 2(s-1)+1]; at the end wall_now takes the last pair.
// src and dst may be the same buffer (an even step count ends where it
// started): every load of src happens before the first store to dst, so the
// pointers carry no __restrict__.
template <int T, int PER>
__global__ void __launch_bounds__(T) k_step_resident1(const double* src, double* dst, int n,
                                                      int64_t nsteps, Rates r,
                                                      const double* __restrict__ walls,
                                                      double* __restrict__ wall_now) {
    constexpr int RES_THREADS = T;
    __shared__ double lds[3 * RESIDENT_MAX_1D];
    for (int x = threadIdx.x; x < n; x += RES_THREADS)
#pragma unroll
        for (int i = 0; i < 3; ++i) lds[i * RESIDENT_MAX_1D + x] = src[slot<3>(i, x)];
    __syncthreads();
    for (int64_t s = 0; s < nsteps; ++s) {
        const double* wall = walls ? (s == 0 ? wall_now : walls + 2 * (s - 1)) : nullptr;
        double f[PER][3];
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            const int x = threadIdx.x + p * RES_THREADS;
            if (x < n) {
                const int xm = x == 0 ? n - 1 : x - 1;
                const int xp = x == n - 1 ? 0 : x + 1;
                double g[3] = {lds[x], lds[RESIDENT_MAX_1D + xm], lds[2 * RESIDENT_MAX_1D + xp]};
                if (wall) {
                    if (x == 0) g[1] = wall[0] - (g[0] + g[2]);
                    if (x == n - 1) g[2] = wall[1] - (g[0] + g[1]);
                }
                collide<1>(g, r);
                f[p][0] = g[0];
                f[p][1] = g[1];
                f[p][2] = g[2];
            }
        }
        __syncthreads();
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            const int x = threadIdx.x + p * RES_THREADS;
            if (x < n) {
                lds[x] = f[p][0];
                lds[RESIDENT_MAX_1D + x] = f[p][1];
                lds[2 * RESIDENT_MAX_1D + x] = f[p][2];
            }
        }
        __syncthreads();
    }
    for (int x = threadIdx.x; x < n; x += RES_THREADS)
#pragma unroll
        for (int i = 0; i < 3; ++i) dst[slot<3>(i, x)] = lds[i * RESIDENT_MAX_1D + x];
    if (walls && nsteps > 0 && threadIdx.x < 2) wall_now[threadIdx.x] = walls[2 * (nsteps - 1) + threadIdx.x];
}

// ---------------------------------------------------------------------------
// 1-D interval with theta given at the end nodes (Example 1 of Sec. IV)
//
// Nodes x = 0..n-1 (n >= 2), the two ends on the boundary.  The distribution
// at x is pulled as usual, except for the one population that would come
// from outside the interval: it takes the value that makes sum_i f_i equal
// the boundary theta of the current time, wall[0] at x = 0 and wall[1] at
// x = n-1.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void wall_pull1(const double* __restrict__ src, int x, int n,
                                           const double* __restrict__ wall, double (&f)[3]) {
    f[0] = src[slot<3>(0, x)];
    f[1] = x > 0 ? src[slot<3>(1, x - 1)] : 0.0;
    f[2] = x < n - 1 ? src[slot<3>(2, x + 1)] : 0.0;
    if (x == 0) f[1] = wall[0] - (f[0] + f[2]);
    if (x == n - 1) f[2] = wall[1] - (f[0] + f[1]);
}

__global__ void __launch_bounds__(256) k_step_wall1(const double* __restrict__ src,
                                                    double* __restrict__ dst, int n, Rates r,
                                                    const double* __restrict__ wall) {
    const int x = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (x >= n) return;
    double f[3];
    wall_pull1(src, x, n, wall, f);
    collide<1>(f, r);
#pragma unroll
    for (int i = 0; i < 3; ++i) __builtin_nontemporal_store(f[i], dst + slot<3>(i, x));
}

// theta, u and grad theta as k_macro<1>, from the bounded-interval distribution.
__global__ void __launch_bounds__(256) k_macro_wall1(const double* __restrict__ src,
                                                     double* __restrict__ theta,
                                                     double* __restrict__ u,
                                                     double* __restrict__ grad, int n, Rates r,
                                                     const double* __restrict__ wall) {
    const int x = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (x >= n) return;
    double f[3];
    wall_pull1(src, x, n, wall, f);
    double th = 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i) th += f[i];
    if (theta) theta[x] = th;
    if (u || grad) {
        double j = 0.0;
#pragma unroll
        for (int i = 0; i < 3; ++i) j = LBM_SADD(j, Lat<1>::E[i][0], f[i]);
        if (u) u[x] = j * (r.ucoef / th);
        if (grad) grad[x] = r.gcoef * j;
    }
}

__global__ void __launch_bounds__(256) k_get_state_wall1(const double* __restrict__ src,
                                                         double* __restrict__ dense, int n,
                                                         const double* __restrict__ wall) {
    const int x = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (x >= n) return;
    double f[3];
    wall_pull1(src, x, n, wall, f);
#pragma unroll
    for (int i = 0; i < 3; ++i) dense[(int64_t)i * n + x] = f[i];
}

// Boundary theta of a dense 3 x n distribution: sum_i f_i at the end nodes.
__global__ void k_wall_from_dense1(const double* __restrict__ dense, int n, double* __restrict__ wall) {
    const int e = (int)threadIdx.x;
    if (e >= 2) return;
    const int x = e == 0 ? 0 : n - 1;
    wall[e] = (dense[x] + dense[(int64_t)n + x]) + dense[2 * (int64_t)n + x];
}

// ---------------------------------------------------------------------------
// Small 1-D grids in one wave: lane l holds nodes l*PER .. l*PER+PER-1 in
// registers for the whole run; each step pulls f_{+1} from the node on the
// left and f_{-1} from the node on the right, inside the lane by register
// moves and across lanes by one DPP move each (a rotation for a periodic grid
// of exactly 64*PER nodes, a plain shift on a bounded interval, where the end
// nodes then take the wall rule of wall_pull1).  No LDS and no barrier; the
// arithmetic is that of k_step<1> / k_step_resident1.
// ---------------------------------------------------------------------------
// src and dst may be the same buffer, as for k_step_resident1.
template <int PER, bool PERIODIC>
__global__ void __launch_bounds__(64) k_step_wave1(const double* src, double* dst, int n,
                                                   int64_t nsteps,
                                                   Rates r, const double* __restrict__ walls,
                                                   double* __restrict__ wall_now) {
    const int lane = threadIdx.x;
    double s0[PER], sp[PER], sm[PER];
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int x = lane * PER + p;
        s0[p] = x < n ? src[slot<3>(0, x)] : 0.0;
        sp[p] = x < n ? src[slot<3>(1, x)] : 0.0;
        sm[p] = x < n ? src[slot<3>(2, x)] : 0.0;
    }
    for (int64_t s = 0; s < nsteps; ++s) {
        const double left = PERIODIC ? lane_rotate<1>(sp[PER - 1]) : lane_shift<1>(sp[PER - 1]);
        const double right = PERIODIC ? lane_rotate<-1>(sm[0]) : lane_shift<-1>(sm[0]);
        double w0 = 0.0, w1 = 0.0;
        if (!PERIODIC) {
            const double* wall = s == 0 ? wall_now : walls + 2 * (s - 1);
            w0 = wall[0];
            w1 = wall[1];
        }
        double t0[PER], tp[PER], tm[PER];
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            const int x = lane * PER + p;
            double g[3] = {s0[p], p > 0 ? sp[p - 1] : left, p < PER - 1 ? sm[p + 1] : right};
            if (!PERIODIC) {
                if (x == 0) g[1] = w0 - (g[0] + g[2]);
                if (x == n - 1) g[2] = w1 - (g[0] + g[1]);
            }
            collide<1>(g, r);
            t0[p] = g[0];
            tp[p] = g[1];
            tm[p] = g[2];
        }
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            s0[p] = t0[p];
            sp[p] = tp[p];
            sm[p] = tm[p];
        }
    }
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int x = lane * PER + p;
        if (x < n) {
            dst[slot<3>(0, x)] = s0[p];
            dst[slot<3>(1, x)] = sp[p];
            dst[slot<3>(2, x)] = sm[p];
        }
    }
    if (!PERIODIC && nsteps > 0 && lane < 2) wall_now[lane] = walls[2 * (nsteps - 1) + lane];
}
}  // namespace

hipError_t launch_step_resident1(const Geo& g, const Rates& r, const double* src, double* dst,
                                int64_t nsteps, const double* walls, double* wall_now,
                                hipStream_t st) {
    if (g.nx > RESIDENT_MAX_1D || g.ny != 1 || g.nz != 1 || g.nw != 1) return hipErrorInvalidValue;
    if (walls && (!wall_now || g.nx < 2)) return hipErrorInvalidValue;
    const int n = g.nx;
#define LBM_WAVE1(PER, PERIODIC)                                                                  \
    hipLaunchKernelGGL((k_step_wave1<PER, PERIODIC>), dim3(1), dim3(64), 0, st, src, dst, n, nsteps, \
                       r, walls, wall_now)
    if (!walls) {
        // periodic grids of exactly 64, 128 or 256 nodes: one wave, lane rotations
        if (n == 64) { LBM_WAVE1(1, true); return hipGetLastError(); }
        if (n == 128) { LBM_WAVE1(2, true); return hipGetLastError(); }
        if (n == 256) { LBM_WAVE1(4, true); return hipGetLastError(); }
    } else {
        if (n <= 64) { LBM_WAVE1(1, false); return hipGetLastError(); }
        if (n <= 128) { LBM_WAVE1(2, false); return hipGetLastError(); }
        if (n <= 256) { LBM_WAVE1(4, false); return hipGetLastError(); }
    }
#undef LBM_WAVE1
#define LBM_RES1(T, PER)                                                                          \
    hipLaunchKernelGGL((k_step_resident1<T, PER>), dim3(1), dim3(T), 0, st, src, dst, n, nsteps, r, \
                       walls, wall_now)
    if (n <= 64) LBM_RES1(64, 1);
    else if (n <= 128) LBM_RES1(64, 2);
    else if (n <= 256) LBM_RES1(128, 2);
    else if (n <= 512) LBM_RES1(256, 2);
    else if (n <= 1024) LBM_RES1(256, 4);
    else LBM_RES1(256, 8);
#undef LBM_RES1
    static_assert(256 * 8 >= RESIDENT_MAX_1D, "resident shapes cover RESIDENT_MAX_1D");
    return hipGetLastError();
}

static dim3 grid_1d(int n) { return dim3((unsigned)((n + 255) / 256)); }

hipError_t launch_step_wall1(const Geo& g, const Rates& r, const double* src, double* dst,
                             const double* wall, hipStream_t st) {
    if (g.nx < 2 || g.ny != 1 || g.nz != 1 || g.nw != 1 || !wall) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_step_wall1, grid_1d(g.nx), dim3(256), 0, st, src, dst, g.nx, r, wall);
    return hipGetLastError();
}

hipError_t launch_macro_wall1(const Geo& g, const Rates& r, const double* state, double* theta,
                              double* u, double* grad, const double* wall, hipStream_t st) {
    if (g.nx < 2 || g.ny != 1 || g.nz != 1 || g.nw != 1 || !wall) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_macro_wall1, grid_1d(g.nx), dim3(256), 0, st, state, theta, u, grad, g.nx,
                       r, wall);
    return hipGetLastError();
}

hipError_t launch_get_state_wall1(const Geo& g, const double* state, double* dense,
                                  const double* wall, hipStream_t st) {
    if (g.nx < 2 || g.ny != 1 || g.nz != 1 || g.nw != 1 || !wall) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_get_state_wall1, grid_1d(g.nx), dim3(256), 0, st, state, dense, g.nx, wall);
    return hipGetLastError();
}

hipError_t launch_wall_from_dense1(const Geo& g, const double* dense, double* wall,
                                   hipStream_t st) {
    if (g.nx < 2 || !wall) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_wall_from_dense1, dim3(1), dim3(64), 0, st, dense, g.nx, wall);
    return hipGetLastError();
}

}  // namespace lbm
