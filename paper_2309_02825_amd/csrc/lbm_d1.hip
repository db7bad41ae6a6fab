// 1-D kernels: whole runs of small grids in one launch, and the bounded interval.
#include <algorithm>

#include "lbm_device.h"

namespace lbm {
namespace {

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
                                           const double* wall, double (&f)[3]) {
    f[0] = src[slot<3>(0, x)];
    f[1] = x > 0 ? src[slot<3>(1, x - 1)] : 0.0;
    f[2] = x < n - 1 ? src[slot<3>(2, x + 1)] : 0.0;
    if (x == 0) f[1] = wall[0] - (f[0] + f[2]);
    if (x == n - 1) f[2] = wall[1] - (f[0] + f[1]);
}

// next != NULL: the boundary theta after the step, which wall (the solver's, only read
// by the end nodes' threads) takes.
__global__ void __launch_bounds__(256) k_step_wall1(const double* __restrict__ src,
                                                    double* __restrict__ dst, int n, Rates r,
                                                    const double* wall, double* wall_now,
                                                    const double* next) {
    const int x = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (x >= n) return;
    double f[3];
    wall_pull1(src, x, n, wall, f);
    if (next && x == 0) wall_now[0] = next[0];
    if (next && x == n - 1) wall_now[1] = next[1];
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
// Small 1-D grids (n <= RESIDENT_MAX_1D): all steps in one launch, the state in
// registers.
//
// A run is a serial chain of steps of a few dependent operations each, so what
// counts is the time of one step.  One workgroup of W waves, each on a window of
// 64 PER consecutive nodes: lane l holds nodes l PER .. l PER + PER - 1 of its
// wave's window and pulls f_{+1} and f_{-1} inside the lane by register names and
// across lanes by DPP moves, so a step needs no LDS and no barrier.  A wave owns
// `own` nodes with a halo of `halo` nodes on each side; the halo's outermost
// valid node moves in by one per step, and every `halo` steps (a multiple of PER,
// at most 64) the waves write their nodes to LDS and read their halos back.
// The shape comes from run1_shape.
//
// ROT (periodic grids of exactly 64 PER nodes): one wave, the lanes rotate, no
// halo.  BOUNDED: the interval's end nodes take the wall rule of wall_pull1; step
// s forms the distribution of the time whose boundary theta is wall_now (s = 0)
// or walls[2(s-1) .. 2(s-1)+1], and at the end wall_now takes the last pair.  A
// lane loads the wall values of one step of the round each, a round ahead, and
// every wave with an end node in its window, owned or halo, reads them by lane.
//
// Measured: n = 64, 256 steps 15.8 -> 7.0 us (one wave, generic collision
// before); bounded n = 321, 12,800 steps 4,181 -> 934 us (before: state in LDS,
// two barriers and a wall load from memory per step, 330 ns).
// src and dst may be the same buffer (an even step count ends where it
// started): every load of src happens before the first store to dst, so the
// pointers carry no __restrict__.
// ---------------------------------------------------------------------------
constexpr int RUN1_MAX_WAVES = 4;  // one per SIMD (run1_shape): more never came out faster

__device__ __forceinline__ double lane_value(double x, int lane) {
    const long long b = __double_as_longlong(x);
    const unsigned lo = __builtin_amdgcn_readlane((unsigned)(b & 0xffffffff), lane);
    const unsigned hi = __builtin_amdgcn_readlane((unsigned)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | lo);
}

template <int PER>
struct Run1State {
    double s0[PER], sp[PER], sm[PER];  // post-collision f_0, f_{+1}, f_{-1}
};

// One step of a window.  LEFT / RIGHT: register 0 of lane llane / register
// PER - 1 of lane rlane is the interval's end node, with the boundary theta in
// lane t of w0 / w1.
template <int PER, bool ROT, bool LEFT, bool RIGHT>
__device__ __forceinline__ void run1_step(Run1State<PER>& s, const FoldedRates1& fr, int t,
                                          bool at_left, bool at_right, double w0, double w1) {
    double left = ROT ? lane_rotate<1>(s.sp[PER - 1]) : lane_shift<1>(s.sp[PER - 1]);
    double right = ROT ? lane_rotate<-1>(s.sm[0]) : lane_shift<-1>(s.sm[0]);
    if constexpr (LEFT) {
        const double v = lane_value(w0, t) - (s.s0[0] + (PER > 1 ? s.sm[PER > 1 ? 1 : 0] : right));
        left = at_left ? v : left;
    }
    if constexpr (RIGHT) {
        const double v =
            lane_value(w1, t) - (s.s0[PER - 1] + (PER > 1 ? s.sp[PER > 1 ? PER - 2 : 0] : left));
        right = at_right ? v : right;
    }
    double g[PER][3];
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        g[p][0] = s.s0[p];
        g[p][1] = p > 0 ? s.sp[p > 0 ? p - 1 : 0] : left;
        g[p][2] = p < PER - 1 ? s.sm[p < PER - 1 ? p + 1 : 0] : right;
        collide_d1q3(g[p], fr);
    }
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        s.s0[p] = g[p][0];
        s.sp[p] = g[p][1];
        s.sm[p] = g[p][2];
    }
}

// `round` steps without an exchange (a few per trip of the loop, so that the
// registers rotate by name and not by copies).
template <int PER, bool ROT, bool LEFT, bool RIGHT>
__device__ __forceinline__ void run1_round(Run1State<PER>& s, const FoldedRates1& fr, int round,
                                           bool at_left, bool at_right, double w0, double w1) {
    constexpr int UNROLL = PER <= 2 ? 4 : 2;
    int t = 0;
    for (; t + UNROLL <= round; t += UNROLL)
#pragma unroll
        for (int v = 0; v < UNROLL; ++v)
            run1_step<PER, ROT, LEFT, RIGHT>(s, fr, t + v, at_left, at_right, w0, w1);
    for (; t < round; ++t)
        run1_step<PER, ROT, LEFT, RIGHT>(s, fr, t, at_left, at_right, w0, w1);
}

template <int PER, bool ROT, bool BOUNDED>
__global__ void __launch_bounds__(ROT ? 64 : 64 * RUN1_MAX_WAVES)
k_run1(const double* src, double* dst, int n, int own, int halo, int64_t nsteps, Rates r,
       const double* __restrict__ walls, double* __restrict__ wall_now) {
    __shared__ double lds[ROT ? 1 : 3 * RESIDENT_MAX_1D];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int first = ROT ? 0 : wave * own;  // first owned node
    const int last = ROT ? n : min(first + own, n);
    int base = first - (ROT ? 0 : halo);  // first node of the window
    // Bounded: where this window, halo included, holds the interval's end nodes.
    // x = 0 falls on register 0 (own and halo are multiples of PER); a window
    // that holds x = n - 1 moves left by less than PER nodes, so that it falls on
    // register PER - 1 (with PER > 1 no window holds both: run1_shape).
    int llane = -1, rlane = -1;
    if constexpr (BOUNDED) {
        if (n - 1 - base < 64 * PER) base -= (PER - 1 - (n - 1 - base) % PER);
        if (base <= 0 && -base < 64 * PER) llane = -base / PER;
        if (n - 1 - base < 64 * PER) rlane = (n - 1 - base) / PER;
    }
    const FoldedRates1 fr = folded1(r);
    // node of every register, wrapped periodically (a bounded window may reach
    // outside the interval: those registers hold values that never get in)
    int node[PER];
    bool mine[PER];
    Run1State<PER> s;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int x = base + lane * PER + p;
        mine[p] = x >= first && x < last;
        node[p] = ROT ? x : wrapi(x, n);
        s.s0[p] = src[slot<3>(0, node[p])];
        s.sp[p] = src[slot<3>(1, node[p])];
        s.sm[p] = src[slot<3>(2, node[p])];
    }
    const bool at_left = lane == llane, at_right = lane == rlane;
    // boundary theta (left, right) of step t0 + lane
    double w0 = 0.0, w1 = 0.0, nw0 = 0.0, nw1 = 0.0;
    auto wall_load = [&](int64_t t0) {
        const int64_t t = t0 + lane;
        if (t < nsteps) {
            const double* w = t == 0 ? wall_now : walls + 2 * (t - 1);
            nw0 = w[0];
            nw1 = w[1];
        }
    };
    if (BOUNDED && (llane >= 0 || rlane >= 0)) wall_load(0);
    for (int64_t done = 0; done < nsteps;) {
        const int round = (int)min(ROT ? (int64_t)(1 << 30) : (int64_t)halo, nsteps - done);
        if (BOUNDED && (llane >= 0 || rlane >= 0)) {
            w0 = nw0;
            w1 = nw1;
            wall_load(done + round);
            if (rlane < 0)
                run1_round<PER, ROT, true, false>(s, fr, round, at_left, at_right, w0, w1);
            else if (llane < 0)
                run1_round<PER, ROT, false, true>(s, fr, round, at_left, at_right, w0, w1);
            else if (PER == 1)
                run1_round<PER, ROT, true, true>(s, fr, round, at_left, at_right, w0, w1);
        } else {
            run1_round<PER, ROT, false, false>(s, fr, round, false, false, 0.0, 0.0);
        }
        done += round;
        if (!ROT && done < nsteps) {
            __syncthreads();  // every wave has read its halo of the round before
#pragma unroll
            for (int p = 0; p < PER; ++p)
                if (mine[p]) {
                    lds[node[p]] = s.s0[p];
                    lds[RESIDENT_MAX_1D + node[p]] = s.sp[p];
                    lds[2 * RESIDENT_MAX_1D + node[p]] = s.sm[p];
                }
            __syncthreads();
#pragma unroll
            for (int p = 0; p < PER; ++p)
                if (!mine[p]) {
                    s.s0[p] = lds[node[p]];
                    s.sp[p] = lds[RESIDENT_MAX_1D + node[p]];
                    s.sm[p] = lds[2 * RESIDENT_MAX_1D + node[p]];
                }
        }
    }
    // every load of src by this workgroup is done before its first store
    if (!ROT) __syncthreads();
#pragma unroll
    for (int p = 0; p < PER; ++p)
        if (mine[p]) {
            dst[slot<3>(0, node[p])] = s.s0[p];
            dst[slot<3>(1, node[p])] = s.sp[p];
            dst[slot<3>(2, node[p])] = s.sm[p];
        }
    if (BOUNDED && nsteps > 0 && threadIdx.x < 2)
        wall_now[threadIdx.x] = walls[2 * (nsteps - 1) + threadIdx.x];
}

}  // namespace

// Shape of k_run1 for n nodes: nodes per lane, waves, nodes owned by a wave and
// halo.  The cost of a step is modelled in cycles as the issue of a SIMD's one wave
// (32 per node of a lane and 16 for the lane moves, at least kLatency, the
// length of one step's dependent chain) plus a share of the exchange; the
// constants only order the shapes (n = 321: 4 waves of 2 nodes a lane).
Run1Shape run1_shape(int n, bool bounded) {
    constexpr int kPer[] = {1, 2, 3, 4, 6, 8, 10};
    constexpr int kLatency = 60, kExchange = 350, kExchangePer = 24;
    Run1Shape best{0, 0, 0, 0};
    int64_t best_cost = INT64_MAX;
    for (int per : kPer) {
        // a bounded window of several nodes per lane holds one end at most, and
        // may move left by up to per - 1 nodes
        if (bounded && per > 1 && n < 64 * per + per) continue;
        const int window = 64 * per - (bounded ? per - 1 : 0);
        for (int waves = 1; waves <= RUN1_MAX_WAVES; ++waves) {
            int own = (n + waves - 1) / waves;
            own = (own + per - 1) / per * per;
            if (own >= window) continue;
            int halo = (window - own) / 2 / per * per;
            if (halo > 64) halo = 64 / per * per;
            if (halo < per) continue;
            if ((int64_t)(waves - 1) * own >= n && waves > 1) continue;  // an idle wave
            const int issue = std::max(kLatency, 32 * per + 16);
            const int64_t cost = (int64_t)issue * 1024 +
                                 (int64_t)(kExchange + kExchangePer * per) * 1024 / halo;
            if (cost < best_cost) {
                best_cost = cost;
                best = Run1Shape{per, waves, own, halo};
            }
        }
    }
    return best;
}

hipError_t launch_step_resident1(const Geo& g, const Rates& r, const double* src, double* dst,
                                int64_t nsteps, const Run1Shape& s, const double* walls,
                                double* wall_now, hipStream_t st) {
    if (g.nx > RESIDENT_MAX_1D || g.ny != 1 || g.nz != 1 || g.nw != 1) return hipErrorInvalidValue;
    if (walls && (!wall_now || g.nx < 2)) return hipErrorInvalidValue;
    const int n = g.nx;
    if (!walls && (n == 64 || n == 128)) {
        if (n == 64)
            hipLaunchKernelGGL((k_run1<1, true, false>), dim3(1), dim3(64), 0, st, src, dst, n, n, 0,
                               nsteps, r, walls, wall_now);
        else
            hipLaunchKernelGGL((k_run1<2, true, false>), dim3(1), dim3(64), 0, st, src, dst, n, n, 0,
                               nsteps, r, walls, wall_now);
        return hipGetLastError();
    }
    const dim3 block(64 * s.waves);
    switch (s.per) {
#define LBM_RUN1(PER)                                                                             \
    case PER:                                                                                     \
        if (walls)                                                                                \
            hipLaunchKernelGGL((k_run1<PER, false, true>), dim3(1), block, 0, st, src, dst, n,    \
                               s.own, s.halo, nsteps, r, walls, wall_now);                        \
        else                                                                                      \
            hipLaunchKernelGGL((k_run1<PER, false, false>), dim3(1), block, 0, st, src, dst, n,   \
                               s.own, s.halo, nsteps, r, walls, wall_now);                        \
        break;
        LBM_RUN1(1)
        LBM_RUN1(2)
        LBM_RUN1(3)
        LBM_RUN1(4)
        LBM_RUN1(6)
        LBM_RUN1(8)
        LBM_RUN1(10)
#undef LBM_RUN1
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

static dim3 grid_1d(int n) { return dim3((unsigned)((n + 255) / 256)); }

hipError_t launch_step_wall1(const Geo& g, const Rates& r, const double* src, double* dst,
                             const double* wall, double* wall_now, const double* next,
                             hipStream_t st) {
    if (g.nx < 2 || g.ny != 1 || g.nz != 1 || g.nw != 1 || !wall) return hipErrorInvalidValue;
    if (next && wall_now != wall) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_step_wall1, grid_1d(g.nx), dim3(256), 0, st, src, dst, g.nx, r, wall,
                       wall_now, next);
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
