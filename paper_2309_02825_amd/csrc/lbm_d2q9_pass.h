// The D2Q9 pass of S steps, compiled for one S per source, or one S and input form.
#pragma once

#include "lbm_pair.h"

namespace lbm {
namespace {

// One strip of a pass.  Odd row segments march up: two neighbouring segments then
// read the halo rows they share at the same time (both at their ends, or both at
// their starts), so the second read finds them in the caches (512^2 +2.7 %,
// 1024^2 +1.3 %, 2048^2 +1.7 %, 4096^2 +0.7 %).
template <int S, bool OFF32, bool NT, int IN, int OUT, int DEPTH = 1>
__device__ __forceinline__ void ms_strip(const double* __restrict__ src, double* __restrict__ dst,
                                         const Geo& g, const Rates& r, int ly, int nstrips) {
    const unsigned t = xcd_remap(blockIdx.x, gridDim.x);
    const int strip = (int)(t % (unsigned)nstrips);
    const int seg = (int)(t / (unsigned)nstrips);
    const int ys = seg * ly, ye = min(ys + ly, g.ny), x0 = strip * strip_width(S);
    if (seg & 1)
        ms_tile<S, false, OFF32, NT, IN, OUT, true, DEPTH>(src, dst, g.nx, g.ny, folded(r), x0, ys, ye);
    else
        ms_tile<S, false, OFF32, NT, IN, OUT, false, DEPTH>(src, dst, g.nx, g.ny, folded(r), x0, ys, ye);
}

__device__ __forceinline__ void mp_strip(const double* __restrict__ src, double* __restrict__ dst,
                                         const Geo& g, const Rates& r, int ly, int nstrips,
                                         MpTwo (*row)[6][64], MpTwo (*pre)[6][64]) {
    const unsigned t = xcd_remap(blockIdx.x, gridDim.x);
    const int strip = (int)(t % (unsigned)nstrips);
    const int seg = (int)(t / (unsigned)nstrips);
    const int ys = seg * ly, ye = min(ys + ly, g.ny), x0 = strip * MP_WIDTH;
    if (seg & 1)
        mp_tile<true>(src, dst, g.nx, g.ny, folded(r), x0, ys, ye, row, pre);
    else
        mp_tile<false>(src, dst, g.nx, g.ny, folded(r), x0, ys, ye, row, pre);
}

// Two waves per SIMD: the register budget (256 per wave) holds S = 8.
// RIN / WOUT: the source / the result is in the reduced form that the passes of
// this grid hand to one another (pass_form).  The pass between two others goes by the
// two-wave march (pair_fits; other grids by k_steps_d2q9_seam).  4096^2, 8 steps:
// 379 us a launch with the 7 planes of FORM_TWIN, 349 us with the 6 of FORM_MOM
// (1.61 GB algorithmic), 321 us by the two-wave march.
// The two-wave march moves a lane's two columns as 16 bytes: even rows, so that a pair
// lies in one chunk and starts on 16 bytes, and buffers that do.  It is taken on grids
// beyond the Infinity Cache, us for 8 steps by one and two waves: 1600^2 65.8 and 65.5,
// 2048^2 97.7 and 97.5, 2500^2 150 and 136, 6000^2 728 and 660, 8000 x 7000 1128 and
// 1022; below, where a segment has few rows, its longer fill loses: 1000^2 28.6 and
// 40.1, 1448^2 53.7 and 57.7.  Oblong grids just beyond it have segments of 18
// to 22 rows (one wave and 7 planes, and two waves: 4096 x 512 60.8 and 58.5, 8192 x 256
// 62.1 and 57.5, 3278 x 609 59.2 and 56.1, 16384 x 128 61.5 and 58.0); half a round
// (pass_rows) is weighed against the one-wave march only.
inline bool pair_fits(const Geo& g, const double* src, const double* dst) {
    return g.nx % 2 == 0 && ((uintptr_t)src | (uintptr_t)dst) % 16 == 0;
}
constexpr bool pair_pass(int s, bool off32, bool rin, bool wout) {
    return s == MP_STEPS && off32 && rin && wout;
}
template <int S, bool OFF32, bool RIN, bool WOUT>
__global__ void __launch_bounds__(pair_pass(S, OFF32, RIN, WOUT) ? MP_THREADS : MS_THREADS)
    __attribute__((amdgpu_waves_per_eu(2)))
k_steps_d2q9(const double* __restrict__ src, double* __restrict__ dst, Geo g, Rates r, int ly,
             int nstrips) {
    constexpr int REDUCED = OFF32 ? FORM_MOM : FORM_TWIN;
    if constexpr (pair_pass(S, OFF32, RIN, WOUT)) {
        __shared__ MpTwo row[2][6][64], pre[2][6][64];
        return mp_strip(src, dst, g, r, ly, nstrips, row, pre);
    }
    ms_strip<S, OFF32, true, RIN ? REDUCED : FORM_FULL, WOUT ? REDUCED : FORM_FULL>(src, dst, g, r,
                                                                                    ly, nstrips);
}

// The same pass with cached stores, for grids whose two states fit in the
// Infinity Cache (the next pass then reads its input from there).
template <int S, bool OFF32, bool RIN, bool WOUT>
__global__ void __launch_bounds__(MS_THREADS) __attribute__((amdgpu_waves_per_eu(2)))
k_steps_d2q9_cached(const double* __restrict__ src, double* __restrict__ dst, Geo g, Rates r,
                    int ly, int nstrips) {
    ms_strip<S, OFF32, false, RIN ? FORM_MOM : FORM_FULL, WOUT ? FORM_MOM : FORM_FULL>(
        src, dst, g, r, ly, nstrips);
}

// Half a round (pass_rows): one wave per SIMD, which has to hide the latency of its
// loads alone and has the registers to load two rows ahead.
template <int S, bool NT, int IN, int OUT>
__global__ void __launch_bounds__(MS_THREADS) __attribute__((amdgpu_waves_per_eu(1, 1)))
k_steps_d2q9_half(const double* __restrict__ src, double* __restrict__ dst, Geo g, Rates r, int ly,
                  int nstrips) {
    ms_strip<S, true, NT, IN, OUT, 2>(src, dst, g, r, ly, nstrips);
}

// The one-wave passes that the kernels above leave, under 4 GiB: odd rows, the first
// of a call on a state that an earlier call left (its twins are equal, so 7 planes are
// read), the one before a single step, which reads populations, and short runs
// (tile_plan).
template <int S, bool NT, int IN, int OUT>
__global__ void __launch_bounds__(MS_THREADS) __attribute__((amdgpu_waves_per_eu(2)))
k_steps_d2q9_seam(const double* __restrict__ src, double* __restrict__ dst, Geo g, Rates r, int ly,
                  int nstrips) {
    ms_strip<S, true, NT, IN, OUT>(src, dst, g, r, ly, nstrips);
}

}  // namespace

// A pass from buffers in form IN (a source of its own for each at eight steps, whose
// kernels take minutes to compile).
template <int S, int IN>
hipError_t launch_steps_from(const Geo& g, const Rates& r, const double* src, double* dst,
                             hipStream_t st, int out) {
    const int w = strip_width(S);
    const int nstrips = (g.nx + w - 1) / w;
    bool half;
    const int ly = pass_rows(g, nstrips, kMinRows, S, &half);
    const int nseg = (g.ny + ly - 1) / ly;
    const dim3 grid((unsigned)((int64_t)nstrips * nseg)), block(MS_THREADS);
    const bool off32 = ms_off32(g), cached = d2q9_cached_stores(g);
    return dispatch_form(out, [&](auto fo) {
        constexpr int OUT = decltype(fo)::value;
        constexpr bool RI = IN != FORM_FULL, WO = OUT != FORM_FULL;
        constexpr bool MOM = IN == FORM_MOM || OUT == FORM_MOM;
        if (!off32) {
            if constexpr (MOM)
                return hipErrorInvalidValue;  // pass_form
            else
                hipLaunchKernelGGL((k_steps_d2q9<S, false, RI, WO>), grid, block, 0, st, src, dst,
                                   g, r, ly, nstrips);
            return hipGetLastError();
        }
        if (half && cached) {
            hipLaunchKernelGGL((k_steps_d2q9_half<S, false, IN, OUT>), grid, block, 0, st, src,
                               dst, g, r, ly, nstrips);
            return hipGetLastError();
        }
        if constexpr (S == MAX_STEPS_PER_PASS) {  // pass_rows: no shorter ones
            if (half) {
                hipLaunchKernelGGL((k_steps_d2q9_half<S, true, IN, OUT>), grid, block, 0, st, src,
                                   dst, g, r, ly, nstrips);
                return hipGetLastError();
            }
        }
        if constexpr (IN == FORM_TWIN || OUT == FORM_TWIN) {
            if (cached)
                hipLaunchKernelGGL((k_steps_d2q9_seam<S, false, IN, OUT>), grid, block, 0, st,
                                   src, dst, g, r, ly, nstrips);
            else
                hipLaunchKernelGGL((k_steps_d2q9_seam<S, true, IN, OUT>), grid, block, 0, st,
                                   src, dst, g, r, ly, nstrips);
        } else if (cached) {  // both states fit in 256 MB, so under 4 GiB
            hipLaunchKernelGGL((k_steps_d2q9_cached<S, true, RI, WO>), grid, block, 0, st, src,
                               dst, g, r, ly, nstrips);
        } else if constexpr (pair_pass(S, true, RI, WO)) {  // FORM_MOM to FORM_MOM
            if (pair_fits(g, src, dst)) {
                const int np = (g.nx + MP_WIDTH - 1) / MP_WIDTH;
                const int lp = steps_rows(g, np, kMinRows, 4 * compute_units());
                const dim3 gp((unsigned)((int64_t)np * ((g.ny + lp - 1) / lp)));
                hipLaunchKernelGGL((k_steps_d2q9<S, true, RI, WO>), gp, dim3(MP_THREADS), 0, st,
                                   src, dst, g, r, lp, np);
            } else {
                hipLaunchKernelGGL((k_steps_d2q9_seam<S, true, IN, OUT>), grid, block, 0, st,
                                   src, dst, g, r, ly, nstrips);
            }
        } else {
            hipLaunchKernelGGL((k_steps_d2q9<S, true, RI, WO>), grid, block, 0, st, src, dst,
                               g, r, ly, nstrips);
        }
        return hipGetLastError();
    });
}

template <int S>
hipError_t launch_steps_t(const Geo& g, const Rates& r, const double* src, double* dst,
                          hipStream_t st, int in, int out) {
    return dispatch_form(in, [&](auto fi) {
        return launch_steps_from<S, decltype(fi)::value>(g, r, src, dst, st, out);
    });
}

}  // namespace lbm
