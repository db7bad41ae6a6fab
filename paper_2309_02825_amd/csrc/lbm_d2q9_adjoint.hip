// D2Q9 passes of an adjoint checkpoint segment: the recomputation that keeps every
// state, and the reverse sweep.
#include <algorithm>

#include "lbm_march.h"

namespace lbm {
namespace {

// The same pass writing the state after every one of its S steps: step j to
// out + (j - 1) stride (the adjoint's recomputation of a checkpoint segment).
// RIN / WOUT as for k_step (WOUT applies to every state written).
template <int S, bool OFF32, bool RIN, bool WOUT>
__global__ void __launch_bounds__(MS_THREADS) __attribute__((amdgpu_waves_per_eu(2)))
k_steps_d2q9_all(const double* __restrict__ src, double* __restrict__ out, int64_t stride, Geo g,
                 Rates r, int ly, int nstrips) {
    const unsigned t = xcd_remap(blockIdx.x, gridDim.x);
    const int strip = (int)(t % (unsigned)nstrips);
    const int seg = (int)(t / (unsigned)nstrips);
    const int ys = seg * ly;
    ms_tile<S, true, OFF32, true, RIN ? FORM_TWIN : FORM_FULL, WOUT ? FORM_TWIN : FORM_FULL>(
        src, out + (int64_t)(S - 1) * stride, g.nx, g.ny,
                                             folded(r), strip * strip_width(S), ys,
                                             min(ys + ly, g.ny), stride);
}

// ---------------------------------------------------------------------------
// S adjoint D2Q9 steps per pass (the reverse sweep of a checkpoint segment).
//
// An adjoint step maps lambda^{n+1} to lambda^n = C^T mu with
// mu_i(x) = lambda^{n+1}_i(x + e_i): the forward step with every velocity
// reversed and C^T in place of C.  The one-wave march of k_steps_d2q9 applies
// with e -> -e (a population with e_y = +1 is used in the iteration its row
// arrives, e_y = -1 two iterations later; e_x = +1 comes from the lane on the
// right).  Stage j produces lambda^{N-j} from lambda^{N-j+1}; at the nodes the
// wave owns it also adds the eps part <mu, (dC/deps) f^{N-j}> (through the
// dual moments of mu, eps_part_d2q9), with f^{N-j}
// pulled from its state buffer at ftop - (j - 1) stride (ftop = f^{N-1});
// RIN: those states were written by a collision and twin populations are
// read from their partners' planes (as in k_step).  The partner planes of the
// twins (those of the (+,+) and (-,+) edges) serve two rows of the pull each
// (row y - 1 for the edge itself, row y + 1 for its twin), so each of their
// rows is loaded once at the lane's own column, kept two rows in a per-wave
// LDS delay and pulled along x by a DPP lane shift (as_load_f_tw, as_edges):
// every plane row of the recomputed states is read once per pass.
// Each lane sums the eps parts of its nodes over all stages and rows in a
// fixed order; the wave's sum goes to partials[block], and the blocks from
// nblocks to ntab - 1 write zeros, so the table always holds ntab entries.
// lambda is bitwise that of S launches of k_adjoint_step<2>.
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int as_ex(int i) { return -Lat<2>::E[i][0]; }
__host__ __device__ constexpr int as_ey(int i) { return -Lat<2>::E[i][1]; }

template <int S>
struct AsState : MsState<S> {
    double fp[S][9];  // f^{N-j} at the node of the next iteration's row, per stage
};

// f^{N-j} pulled at node (x, y): population i from (x - e_i, y - e_i).
template <bool RIN>
__device__ __forceinline__ void as_load_f(double (&fn)[9], const double* __restrict__ fs, int x,
                                          int y, int nx, int ny) {
    const int rows[3] = {wrapi(y + 1, ny) * nx, y * nx, wrapi(y - 1, ny) * nx};
    const int cols[3] = {x == nx - 1 ? 0 : x + 1, x, x == 0 ? nx - 1 : x - 1};
#pragma unroll
    for (int i = 0; i < 9; ++i)
        fn[i] = fs[slot<9>(RIN ? twin<2>(i) : i, rows[ms_ey(i) + 1] + cols[ms_ex(i) + 1])];
}

// RIN: the per-wave LDS delay of the two partner planes for stage j holds,
// per row parity, the raw rows (own column of each lane) of planes 5 and 6:
// tw[((j - 1) * 2 + parity) * 128 + plane * 64 + lane].  Each lane reads
// and writes only its own entries.
constexpr int AS_TW = 128;  // doubles per stage and parity
// f^{N-j} for row y (RIN): populations 0-4 pulled as in as_load_f (own
// lanes); fn[7], fn[8] the raw rows y + 1 of planes 5 and 6 (every lane).
// as_edges completes the pull when the row is used.
__device__ __forceinline__ void as_load_f_tw(double (&fn)[9], const double* __restrict__ fs,
                                             int x, int gx, int y, int nx, int ny, bool own) {
    if (own) {
        const int rows[3] = {wrapi(y + 1, ny) * nx, y * nx, wrapi(y - 1, ny) * nx};
        const int cols[3] = {x == nx - 1 ? 0 : x + 1, x, x == 0 ? nx - 1 : x - 1};
#pragma unroll
        for (int i = 0; i < 5; ++i) fn[i] = fs[slot<9>(i, rows[ms_ey(i) + 1] + cols[ms_ex(i) + 1])];
    }
    const int yp = wrapi(y + 1, ny) * nx + gx;
    fn[7] = fs[slot<9>(5, yp)];
    fn[8] = fs[slot<9>(6, yp)];
}
// Row y of stage j: take the raw rows y - 1 of planes 5 and 6 from the LDS
// delay (stored two rows earlier, or at the start of the segment), store the
// raw rows y + 1 in their place for row y + 2, and pull the four edge
// populations along x: population i of plane 5 or 6 from the lane at
// x - e_x (e = (1,1), (-1,1) from row y - 1; (-1,-1), (1,-1) from row y + 1).
__device__ __forceinline__ void as_edges(double (&fn)[9], double* tw) {
    const double m5 = tw[threadIdx.x], m6 = tw[64 + threadIdx.x];
    tw[threadIdx.x] = fn[7];
    tw[64 + threadIdx.x] = fn[8];
    fn[5] = lane_shift<1>(m5);
    fn[6] = lane_shift<-1>(m6);
    fn[7] = lane_shift<-1>(fn[7]);
    fn[8] = lane_shift<1>(fn[8]);
}
static_assert(ms_ex(5) == 1 && ms_ey(5) == 1 && ms_ex(6) == -1 && ms_ey(6) == 1 &&
                  twin<2>(7) == 5 && twin<2>(8) == 6,
              "the edge planes 5 and 6 carry the (+,+) and (-,+) edges and their twins");

template <int S, int P, int ACTIVE, bool RIN>
__device__ __forceinline__ void as_row(AsState<S>& st, double& ge, int k,
                                       const double* __restrict__ src, double* __restrict__ dst,
                                       const double* __restrict__ ftop, int64_t stride, int nx,
                                       int ny, int gx, int ys, int x0, int nrows, const Rates& r,
                                       double* tw) {
    constexpr int W = MS_THREADS - 2 * S;
    const int lane = threadIdx.x;
    const int x = x0 - S + lane;
    const bool own = lane >= S && lane < S + W && x < nx;
    double f[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) f[i] = st.pre[0][i];
    {
        // next lambda row (unused in the last iteration, as in ms_row)
        const int base = wrapi(ys - S + k + 1, ny) * nx + gx;
#pragma unroll
        for (int i = 0; i < 9; ++i) st.pre[0][i] = src[slot<9>(i, base)];
    }
#pragma unroll
    for (int j = 1; j <= S; ++j) {
        double in[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const double v = as_ex(i) == 0 ? f[i]
                                           : (as_ex(i) == 1 ? lane_shift<1>(f[i]) : lane_shift<-1>(f[i]));
            if (as_ey(i) == -1) {
                in[i] = v;
            } else if (as_ey(i) == 0) {
                in[i] = st.z[j - 1][ms_yslot(i)];
                st.z[j - 1][ms_yslot(i)] = v;
            } else {
                in[i] = st.u[P][j - 1][ms_yslot(i)];
                st.u[P][j - 1][ms_yslot(i)] = v;
            }
        }
        if (j <= ACTIVE) {
            const int rr = k - S - j;  // owned row ys + rr of this stage
            // the dual moments of mu serve the eps part and C^T mu
            const Dual2 du = dual_d2q9(in);
            if (rr >= 0 && rr < nrows) {
                if constexpr (RIN) as_edges(st.fp[j - 1], tw + ((j - 1) * 2 + (rr & 1)) * AS_TW);
                if (own) ge += eps_part_d2q9(du, st.fp[j - 1], r);
            }
            double lam[9];
            collide_adjoint_d2q9(du, r, lam);  // as collide_adjoint<2>
#pragma unroll
            for (int i = 0; i < 9; ++i) f[i] = lam[i];
            if (j == S && ACTIVE == S && own) {
                const int row = (ys + k - 2 * S) * nx + x;
#pragma unroll
                for (int i = 0; i < 9; ++i) dst[slot<9>(i, row)] = lam[i];
            }
        }
    }
    // f^{N-j} for the rows the stages own in the next iteration
#pragma unroll
    for (int j = 1; j <= S; ++j) {
        const int rr = k + 1 - S - j;
        if constexpr (RIN) {
            if (rr >= 0 && rr < nrows)
                as_load_f_tw(st.fp[j - 1], ftop - (int64_t)(j - 1) * stride, x, gx, ys + rr, nx,
                             ny, own);
        } else {
            if (own && rr >= 0 && rr < nrows)
                as_load_f<RIN>(st.fp[j - 1], ftop - (int64_t)(j - 1) * stride, x, ys + rr, nx, ny);
        }
    }
}

template <int S, int K, bool RIN>
__device__ __forceinline__ void as_fill(AsState<S>& st, double& ge,
                                        const double* __restrict__ src, double* __restrict__ dst,
                                        const double* __restrict__ ftop, int64_t stride, int nx,
                                        int ny, int gx, int ys, int x0, int nrows, const Rates& r,
                                        double* tw) {
    if constexpr (K < 2 * S) {
        as_row<S, K & 1, K / 2, RIN>(st, ge, K, src, dst, ftop, stride, nx, ny, gx, ys, x0, nrows,
                                     r, tw);
        as_fill<S, K + 1, RIN>(st, ge, src, dst, ftop, stride, nx, ny, gx, ys, x0, nrows, r, tw);
    }
}

template <int S, bool RIN>
__global__ void __launch_bounds__(MS_THREADS) __attribute__((amdgpu_waves_per_eu(2)))
k_adjoint_steps_d2q9(const double* __restrict__ src, double* __restrict__ dst,
                     const double* __restrict__ ftop, int64_t stride,
                     double* __restrict__ partials, int ntab, Geo g, Rates r, int ly,
                     int nstrips) {
    const int nx = g.nx, ny = g.ny;
    const unsigned t = xcd_remap(blockIdx.x, gridDim.x);
    const int strip = (int)(t % (unsigned)nstrips);
    const int seg = (int)(t / (unsigned)nstrips);
    const int x0 = strip * strip_width(S);
    const int ys = seg * ly;
    const int ye = min(ys + ly, ny);
    const int gx = wrapi(x0 - S + (int)threadIdx.x, nx);
    const int kend = ye - ys + 2 * S - 1;
    const int nrows = ye - ys;
    AsState<S> st;
    {
        const int base = wrapi(ys - S, ny) * nx + gx;
#pragma unroll
        for (int i = 0; i < 9; ++i) st.pre[0][i] = src[slot<9>(i, base)];
    }
#pragma unroll
    for (int j = 0; j < S; ++j) {
#pragma unroll
        for (int a = 0; a < 3; ++a) st.z[j][a] = st.u[0][j][a] = st.u[1][j][a] = 0.0;
#pragma unroll
        for (int i = 0; i < 9; ++i) st.fp[j][i] = 0.0;
    }
    // RIN: the LDS delay of the partner planes starts with the raw rows
    // ys - 1 (parity 0) and ys (parity 1) of every stage's state; each lane
    // reads back only what it wrote, so no barrier is needed
    __shared__ double tw[RIN ? S * 2 * AS_TW : 1];
    if constexpr (RIN) {
#pragma unroll
        for (int j = 0; j < S; ++j) {
            const double* fs = ftop - (int64_t)j * stride;
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int row = wrapi(ys - 1 + p, ny) * nx + gx;
                tw[(j * 2 + p) * AS_TW + threadIdx.x] = fs[slot<9>(5, row)];
                tw[(j * 2 + p) * AS_TW + 64 + threadIdx.x] = fs[slot<9>(6, row)];
            }
        }
    }
    double ge = 0.0;
    as_fill<S, 0, RIN>(st, ge, src, dst, ftop, stride, nx, ny, gx, ys, x0, nrows, r, tw);
    // row pairs in the loop, a last odd row after it (as in ms_tile)
    int k = 2 * S;
    for (; k + 1 <= kend; k += 2) {
        as_row<S, 0, S, RIN>(st, ge, k, src, dst, ftop, stride, nx, ny, gx, ys, x0, nrows, r, tw);
        as_row<S, 1, S, RIN>(st, ge, k + 1, src, dst, ftop, stride, nx, ny, gx, ys, x0, nrows, r,
                             tw);
    }
    if (k <= kend)
        as_row<S, 0, S, RIN>(st, ge, k, src, dst, ftop, stride, nx, ny, gx, ys, x0, nrows, r, tw);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) ge += __shfl_xor(ge, o, 64);
    if (threadIdx.x == 0) {
        partials[blockIdx.x] = ge;
        for (int i = (int)gridDim.x + (int)blockIdx.x; i < ntab; i += (int)gridDim.x)
            partials[i] = 0.0;
    }
}

}  // namespace

template <int S>
static hipError_t launch_steps_all_t(const Geo& g, const Rates& r, const double* src, double* out,
                                     int64_t stride, hipStream_t st, bool rin, bool wout) {
    const int w = strip_width(S);
    const int nstrips = (g.nx + w - 1) / w;
    const int ly = steps_rows(g, nstrips, kMinRowsSegment);
    const dim3 grid((unsigned)((int64_t)nstrips * ((g.ny + ly - 1) / ly)));
    const bool off32 = ms_off32(g);
    return dispatch_io(rin, wout, [&](auto ri, auto wo) {
        constexpr bool RI = decltype(ri)::value, WO = decltype(wo)::value;
        if (off32)
            hipLaunchKernelGGL((k_steps_d2q9_all<S, true, RI, WO>), grid, dim3(MS_THREADS), 0, st,
                               src, out, stride, g, r, ly, nstrips);
        else
            hipLaunchKernelGGL((k_steps_d2q9_all<S, false, RI, WO>), grid, dim3(MS_THREADS), 0, st,
                               src, out, stride, g, r, ly, nstrips);
        return hipGetLastError();
    });
}

hipError_t launch_steps_all(int nsteps, const Geo& g, const Rates& r, const double* src,
                            double* out, int64_t stride, hipStream_t st, bool rin, bool wout) {
    switch (nsteps) {
        case 2: return launch_steps_all_t<2>(g, r, src, out, stride, st, rin, wout);
        case 4: return launch_steps_all_t<4>(g, r, src, out, stride, st, rin, wout);
        case 8: return launch_steps_all_t<8>(g, r, src, out, stride, st, rin, wout);
        default: return hipErrorInvalidValue;
    }
}

template <int S>
static int64_t adjoint_steps_blocks_t(const Geo& g) {
    const int w = strip_width(S);
    const int64_t nstrips = (g.nx + w - 1) / w;
    const int ly = steps_rows(g, (int)nstrips, kMinRowsSegment);
    return nstrips * ((g.ny + ly - 1) / ly);
}

int64_t adjoint_steps_table(const Geo& g) {
    return std::max(adjoint_steps_blocks_t<2>(g), adjoint_steps_blocks_t<4>(g));
}

template <int S>
static hipError_t launch_adjoint_steps_t(const Geo& g, const Rates& r, const double* lam_in,
                                         double* lam_out, const double* ftop, int64_t stride,
                                         double* partials, int64_t ntab, hipStream_t st,
                                         bool rin) {
    const int w = strip_width(S);
    const int nstrips = (g.nx + w - 1) / w;
    const int ly = steps_rows(g, nstrips, kMinRowsSegment);
    const int64_t nb = (int64_t)nstrips * ((g.ny + ly - 1) / ly);
    if (nb > ntab || ntab > (int64_t)INT32_MAX) return hipErrorInvalidValue;
    if (rin)
        hipLaunchKernelGGL((k_adjoint_steps_d2q9<S, true>), dim3((unsigned)nb), dim3(MS_THREADS),
                           0, st, lam_in, lam_out, ftop, stride, partials, (int)ntab, g, r, ly,
                           nstrips);
    else
        hipLaunchKernelGGL((k_adjoint_steps_d2q9<S, false>), dim3((unsigned)nb), dim3(MS_THREADS),
                           0, st, lam_in, lam_out, ftop, stride, partials, (int)ntab, g, r, ly,
                           nstrips);
    return hipGetLastError();
}

hipError_t launch_adjoint_steps(int nsteps, const Geo& g, const Rates& r, const double* lam_in,
                                double* lam_out, const double* ftop, int64_t stride,
                                double* partials, int64_t ntab, hipStream_t st, bool rin) {
    switch (nsteps) {
        case 2:
            return launch_adjoint_steps_t<2>(g, r, lam_in, lam_out, ftop, stride, partials, ntab,
                                             st, rin);
        case 4:
            return launch_adjoint_steps_t<4>(g, r, lam_in, lam_out, ftop, stride, partials, ntab,
                                             st, rin);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace lbm
