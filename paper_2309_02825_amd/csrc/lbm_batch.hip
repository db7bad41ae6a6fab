// The batched form: 2-D steps over a tile table.
#include "lbm_march.h"

namespace lbm {
namespace {

// ---------------------------------------------------------------------------
// batched 2-D step over a tile table
// ---------------------------------------------------------------------------
// One block per tile.  tx > 0: a tx x (256/tx) rectangle of one instance at
// (x0, y0); tx == 0: 256 consecutive node indices of one instance starting at
// x0, crossing row ends, so no lane idles except at the instance's last tile.
template <bool RIN, bool WOUT>
__global__ void __launch_bounds__(256) k_batch_step(const BatchInst* __restrict__ insts,
                                                    const BatchTile* __restrict__ tiles, int tx,
                                                    int log2tx, const double* __restrict__ src,
                                                    double* __restrict__ dst) {
    constexpr int Q = 9;
    const BatchTile t = tiles[xcd_remap(blockIdx.x, gridDim.x)];
    const BatchInst& in = insts[t.inst];
    const int tid = threadIdx.x;
    int x, y;
    if (tx == 0) {
        const int k = t.x0 + tid;
        if (k >= in.nx * in.ny) return;
        y = k / in.nx;
        x = k - y * in.nx;
    } else {
        x = t.x0 + (tid & (tx - 1));
        y = t.y0 + (tid >> log2tx);
        if (x >= in.nx || y >= in.ny) return;
    }
    Geo g;
    g.nx = in.nx;
    g.ny = in.ny;
    g.nz = 1;
    g.nw = 1;
    g.V = (int64_t)in.nx * in.ny;
    const int c[4] = {x, y, 0, 0};
    const Nbr nb = make_nbr<2>(c, g);
    const double* s = src + in.offset;
    double* d = dst + in.offset;
    double f[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) f[i] = s[slot<Q>(RIN ? twin<2>(i) : i, pull_index<2>(nb, i))];
    const Rates r = in.r;
    collide<2>(f, r);
    const int k = y * g.nx + x;
#pragma unroll
    for (int i = 0; i < Q; ++i)
        if (!WOUT || twin<2>(i) == i) __builtin_nontemporal_store(f[i], d + slot<Q>(i, k));
}

// ---------------------------------------------------------------------------
// S D2Q9 time steps per pass, two-wave variant for the batched form.
//
// A block of LW_THREADS = 128 threads owns a strip of 128 - 2S columns (112
// at S = 8 against 48 for one wave), which wastes fewer columns on the
// halo and on the ragged last strip of instances 64..1024 nodes wide.  Thread
// t owns column x0 - S + t in every stage; the populations with e_x != 0
// cross between the two waves through LDS, written already shifted by e_x
// (producer column t -> slot t + e_x) so that every consumer reads its own
// column, with a barrier per stage; stages alternate between two LDS buffers
// of 6 x 128 doubles.  Rows are delayed in registers as in the one-wave
// routine.  Same arithmetic, so also bitwise S single steps.
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int lw_ex(int i) { return Lat<2>::E[i][0]; }
__host__ __device__ constexpr int lw_ey(int i) { return Lat<2>::E[i][1]; }
// index of population i among those with e_x != 0
__host__ __device__ constexpr int lw_xslot(int i) {
    int s = 0;
    for (int j = 0; j < i; ++j) s += lw_ex(j) != 0;
    return s;
}
// index of population i among those with the same e_y
__host__ __device__ constexpr int lw_yslot(int i) {
    int s = 0;
    for (int j = 0; j < i; ++j) s += lw_ey(j) == lw_ey(i);
    return s;
}

template <int S>
struct LwState {
    double pre[9];      // next input row (prefetched)
    double z[S][3];     // e_y = 0 populations of the previous row, per stage input
    double u[2][S][3];  // e_y = +1 populations of the rows of each parity
};

// One iteration k of the march; P = k & 1.
template <int S, int P, bool OFF32, bool RIN, bool WOUT>
__device__ __forceinline__ void lw_row(LwState<S>& st, double (&lds)[2][6][LW_THREADS], int k,
                                       int kend, const double* __restrict__ src,
                                       double* __restrict__ dst, int nx, int ny, int gx, int ys,
                                       int x0, const FoldedRates& r) {
    constexpr int W = LW_THREADS - 2 * S;
    const int tid = threadIdx.x;
    double f[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) f[i] = st.pre[RIN ? twin<2>(i) : i];
    // (an unconditional prefetch as in ms_row raised this kernel to 260
    // VGPRs, one wave per SIMD, and cost 20 % on the batch)
    if (k < kend) {
        const MsAddr<OFF32> a(wrapi(ys - S + k + 1, ny) * nx + gx);
#pragma unroll
        for (int i = 0; i < 9; ++i)
            if (!RIN || twin<2>(i) == i) st.pre[i] = a.load(src, i);
    }
#pragma unroll
    for (int i = 0; i < 9; ++i)
        if (lw_ex(i) != 0) {
            const int c = tid + lw_ex(i);
            if (c >= 0 && c < LW_THREADS) lds[0][lw_xslot(i)][c] = f[i];
        }
    __syncthreads();
#pragma unroll
    for (int j = 1; j <= S; ++j) {
        // inputs of stage j: stage j-1 rows of iterations k (e_y = -1), k-1
        // (e_y = 0) and k-2 (e_y = +1)
        double in[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const double v = lw_ex(i) != 0 ? lds[(j - 1) & 1][lw_xslot(i)][tid] : f[i];
            if (lw_ey(i) == -1) {
                in[i] = v;
            } else if (lw_ey(i) == 0) {
                in[i] = st.z[j - 1][lw_yslot(i)];
                st.z[j - 1][lw_yslot(i)] = v;
            } else {
                in[i] = st.u[P][j - 1][lw_yslot(i)];
                st.u[P][j - 1][lw_yslot(i)] = v;
            }
        }
        // stage j holds valid rows from iteration 2j on, in columns j .. T-1-j
        if (k >= 2 * j && tid >= j && tid < LW_THREADS - j) {
            collide_d2q9(in, r);
            if (j < S) {
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    f[i] = in[i];
                    if (lw_ex(i) != 0) {
                        const int c = tid + lw_ex(i);
                        if (c >= 0 && c < LW_THREADS) lds[j & 1][lw_xslot(i)][c] = in[i];
                    }
                }
            } else if (tid >= S && tid < S + W && x0 - S + tid < nx) {
                const MsAddr<OFF32> a(wrapi(ys - 2 * S + k, ny) * nx + x0 - S + tid);
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    if (!WOUT || twin<2>(i) == i) a.store(dst, i, in[i]);
            }
        }
        if (j < S) __syncthreads();
    }
    // with S odd the last stage reads buffer 0, which the next load rewrites
    if (S & 1) __syncthreads();
}

// Advance rows [ys, ye) of the columns [x0, x0 + LW_THREADS - 2S) of one
// D2Q9 grid by S steps (reads rows ys-S .. ye-1+S and columns x0-S ..
// x0+LW_THREADS-S-1, wrapped periodically).
template <int S, bool OFF32, bool RIN, bool WOUT>
__device__ __forceinline__ void lw_tile(const double* __restrict__ src, double* __restrict__ dst,
                                        int nx, int ny, const FoldedRates& r, int x0, int ys, int ye,
                                        double (&lds)[2][6][LW_THREADS]) {
    const int gx = wrapi(x0 - S + (int)threadIdx.x, nx);
    const int kend = ye - ys + 2 * S - 1;
    LwState<S> st;
    {
        const MsAddr<OFF32> a(wrapi(ys - S, ny) * nx + gx);
#pragma unroll
        for (int i = 0; i < 9; ++i)
            if (!RIN || twin<2>(i) == i) st.pre[i] = a.load(src, i);
    }
#pragma unroll
    for (int j = 0; j < S; ++j)
#pragma unroll
        for (int a = 0; a < 3; ++a) st.z[j][a] = st.u[0][j][a] = st.u[1][j][a] = 0.0;
    // row pairs in the loop, a last odd row after it (as in ms_tile)
    int k = 0;
    for (; k + 1 <= kend; k += 2) {
        lw_row<S, 0, OFF32, RIN, WOUT>(st, lds, k, kend, src, dst, nx, ny, gx, ys, x0, r);
        lw_row<S, 1, OFF32, RIN, WOUT>(st, lds, k + 1, kend, src, dst, nx, ny, gx, ys, x0, r);
    }
    if (k <= kend) lw_row<S, 0, OFF32, RIN, WOUT>(st, lds, k, kend, src, dst, nx, ny, gx, ys, x0, r);
}


// Batched S-step pass: tile (inst, x0, y0, y1) = rows [y0, y1) of the strip
// at x0 (batch_strip_width(S) columns) of one instance.  OFF32: every
// instance's state is under 4 GiB (MsAddr<true> from the instance's start).
// RIN / WOUT as for k_step.
template <int S, bool OFF32, bool RIN, bool WOUT>
__global__ void __launch_bounds__(LW_THREADS) k_batch_steps(const BatchInst* __restrict__ insts,
                                                            const BatchTile* __restrict__ tiles,
                                                            const double* __restrict__ src,
                                                            double* __restrict__ dst) {
    __shared__ double lds[2][6][LW_THREADS];
    const BatchTile t = tiles[xcd_remap(blockIdx.x, gridDim.x)];
    const BatchInst& in = insts[t.inst];
    lw_tile<S, OFF32, RIN, WOUT>(src + in.offset, dst + in.offset, in.nx, in.ny, folded(in.r),
                                 t.x0, t.y0, t.pad, lds);
}

// The same pass with the one-wave march of k_steps_d2q9: tile (inst, x0, y0,
// y1) = rows [y0, y1) of the strip at x0 (strip_width(S) columns).  IN / OUT:
// what the pools hold (FORM_*).
template <int S, bool OFF32, int IN, int OUT>
__global__ void __launch_bounds__(MS_THREADS) __attribute__((amdgpu_waves_per_eu(2)))
k_batch_steps_w(const BatchInst* __restrict__ insts, const BatchTile* __restrict__ tiles,
                const double* __restrict__ src, double* __restrict__ dst) {
    const BatchTile t = tiles[xcd_remap(blockIdx.x, gridDim.x)];
    const BatchInst& in = insts[t.inst];
    ms_tile<S, false, OFF32, true, IN, OUT>(src + in.offset, dst + in.offset, in.nx, in.ny,
                                            folded(in.r), t.x0, t.y0, t.pad, 0);
}

}  // namespace

template <int S, bool OFF32>
static hipError_t launch_batch_steps_t(const BatchInst* insts, const BatchTile* tiles,
                                       int64_t ntiles, const double* src, double* dst,
                                       bool one_wave, hipStream_t st, int in, int out) {
    const dim3 grid((unsigned)ntiles), block(one_wave ? MS_THREADS : LW_THREADS);
    return dispatch_form(in, [&](auto fi) {
        return dispatch_form(out, [&](auto fo) {
            constexpr int IN = decltype(fi)::value, OUT = decltype(fo)::value;
            constexpr bool MOM = IN == FORM_MOM || OUT == FORM_MOM;
            if (one_wave) {
                if constexpr (OFF32 || !MOM) {
                    hipLaunchKernelGGL((k_batch_steps_w<S, OFF32, IN, OUT>), grid, block, 0, st,
                                       insts, tiles, src, dst);
                    return hipGetLastError();
                }
            } else if constexpr (!MOM) {
                hipLaunchKernelGGL((k_batch_steps<S, OFF32, IN == FORM_TWIN, OUT == FORM_TWIN>), grid,
                                   block, 0, st, insts, tiles, src, dst);
                return hipGetLastError();
            }
            return hipErrorInvalidValue;  // batch_form
        });
    });
}

template <int S>
static hipError_t launch_batch_steps_s(const BatchInst* insts, const BatchTile* tiles,
                                       int64_t ntiles, const double* src, double* dst, bool off32,
                                       bool one_wave, hipStream_t st, int in, int out) {
    return off32 ? launch_batch_steps_t<S, true>(insts, tiles, ntiles, src, dst, one_wave, st, in, out)
                 : launch_batch_steps_t<S, false>(insts, tiles, ntiles, src, dst, one_wave, st, in, out);
}

hipError_t launch_batch_steps(int nsteps, const BatchInst* insts, const BatchTile* tiles,
                              int64_t ntiles, const double* src, double* dst, bool off32,
                              bool one_wave, hipStream_t st, int in, int out) {
    if (ntiles <= 0) return hipSuccess;
    switch (nsteps) {
        case 2: return launch_batch_steps_s<2>(insts, tiles, ntiles, src, dst, off32, one_wave, st, in, out);
        case 4: return launch_batch_steps_s<4>(insts, tiles, ntiles, src, dst, off32, one_wave, st, in, out);
        case 8: return launch_batch_steps_s<8>(insts, tiles, ntiles, src, dst, off32, one_wave, st, in, out);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_batch_step(const BatchInst* insts, const BatchTile* tiles, int64_t ntiles,
                             int tx, int ty, const double* src, double* dst, hipStream_t st,
                             bool rin, bool wout) {
    (void)ty;
    int log2tx = 0;
    while (tx > 0 && (1 << log2tx) < tx) ++log2tx;
    if (ntiles <= 0) return hipSuccess;
    return dispatch_io(rin, wout, [&](auto ri, auto wo) {
        hipLaunchKernelGGL((k_batch_step<decltype(ri)::value, decltype(wo)::value>),
                           dim3((unsigned)ntiles), dim3(256), 0, st, insts, tiles, tx, log2tx, src,
                           dst);
        return hipGetLastError();
    });
}

}  // namespace lbm
