// D2Q9 passes of several steps.
#include <atomic>

#include "lbm_march.h"

namespace lbm {
namespace {

// Two waves per SIMD: the register budget (256 per wave) holds S = 8.
// RIN / WOUT: twin populations read from their twins' planes / not stored,
// as for k_step.  Odd row segments march up: two neighbouring segments then
// read the halo rows they share at the same time (both at their ends, or
// both at their starts), so the second read finds them in the caches
// (512^2 +2.7 %, 1024^2 +1.3 %, 2048^2 +1.7 %, 4096^2 +0.7 %).
template <int S, bool OFF32, bool RIN, bool WOUT>
__global__ void __launch_bounds__(MS_THREADS) __attribute__((amdgpu_waves_per_eu(2)))
k_steps_d2q9(const double* __restrict__ src,
                                                           double* __restrict__ dst, Geo g,
                                                           Rates r, int ly, int nstrips) {
    const unsigned t = xcd_remap(blockIdx.x, gridDim.x);
    const int strip = (int)(t % (unsigned)nstrips);
    const int seg = (int)(t / (unsigned)nstrips);
    const int ys = seg * ly;
    if (seg & 1)
        ms_tile<S, false, OFF32, true, RIN, WOUT, true>(src, dst, g.nx, g.ny, folded(r),
                                                        strip * strip_width(S), ys,
                                                        min(ys + ly, g.ny), 0);
    else
        ms_tile<S, false, OFF32, true, RIN, WOUT>(src, dst, g.nx, g.ny, folded(r),
                                                  strip * strip_width(S), ys, min(ys + ly, g.ny),
                                                  0);
}

// The same pass with cached stores, for grids whose two states fit in the
// Infinity Cache (the next pass then reads its input from there).
template <int S, bool OFF32, bool RIN, bool WOUT>
__global__ void __launch_bounds__(MS_THREADS) __attribute__((amdgpu_waves_per_eu(2)))
k_steps_d2q9_cached(const double* __restrict__ src, double* __restrict__ dst, Geo g, Rates r,
                    int ly, int nstrips) {
    const unsigned t = xcd_remap(blockIdx.x, gridDim.x);
    const int strip = (int)(t % (unsigned)nstrips);
    const int seg = (int)(t / (unsigned)nstrips);
    const int ys = seg * ly;
    if (seg & 1)
        ms_tile<S, false, OFF32, false, RIN, WOUT, true>(src, dst, g.nx, g.ny, folded(r),
                                                         strip * strip_width(S), ys,
                                                         min(ys + ly, g.ny), 0);
    else
        ms_tile<S, false, OFF32, false, RIN, WOUT>(src, dst, g.nx, g.ny, folded(r),
                                                   strip * strip_width(S), ys,
                                                   min(ys + ly, g.ny), 0);
}

}  // namespace

// Rows per segment of an S-step launch.  A one-wave block of k_steps_d2q9
// holds about 240 VGPRs, so a CU runs 8 of them at once: the segments are
// cut so that all blocks fit in one round of 8 x (number of CUs) (fewer,
// longer segments amortise the 2S-row pipeline fill; a partial second round
// costs far more), at least 8 rows, and in more rounds when a segment would
// exceed 512 rows.  Measured minimum (MLUPS at 8 steps per pass): 512^2
// 47,500 at 24 rows, 70,200 at 8; 1024^2 132,000 and 148,300; 2048^2 and
// 4096^2 unchanged (their segments are longer).
// Blocks of k_steps_d2q9 one round holds on the current device (8 per CU),
// looked up once per device.
static int round_slots() {
    constexpr int kMaxDevices = 64;
    static std::atomic<int> cached[kMaxDevices] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) dev = 0;
    const int d = dev < kMaxDevices ? dev : kMaxDevices - 1;
    int slots = cached[d].load(std::memory_order_relaxed);
    if (slots == 0) {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            cus <= 0)
            cus = 256;
        slots = 8 * cus;
        cached[d].store(slots, std::memory_order_relaxed);
    }
    return slots;
}

int steps_rows(const Geo& g, int nstrips, int min_rows) {
    const int slots = round_slots();
    int64_t per_round = slots / nstrips;
    if (per_round < 1) per_round = 1;
    int64_t nseg = per_round;
    int64_t ly = (g.ny + nseg - 1) / nseg;
    while (ly > 512) {
        nseg += per_round;
        ly = (g.ny + nseg - 1) / nseg;
    }
    if (ly < min_rows) ly = min_rows;
    if (ly > g.ny) ly = g.ny;
    return (int)ly;
}

template <int S>
static hipError_t launch_steps_t(const Geo& g, const Rates& r, const double* src, double* dst,
                                 hipStream_t st, bool rin, bool wout) {
    const int w = strip_width(S);
    const int nstrips = (g.nx + w - 1) / w;
    const int ly = steps_rows(g, nstrips, kMinRows);
    const int nseg = (g.ny + ly - 1) / ly;
    const dim3 grid((unsigned)((int64_t)nstrips * nseg));
    return dispatch_io(rin, wout, [&](auto ri, auto wo) {
        constexpr bool RI = decltype(ri)::value, WO = decltype(wo)::value;
        if (d2q9_cached_stores(g))  // both states fit in 256 MB, so under 4 GiB
            hipLaunchKernelGGL((k_steps_d2q9_cached<S, true, RI, WO>), grid, dim3(MS_THREADS), 0,
                               st, src, dst, g, r, ly, nstrips);
        else if (ms_off32(g))
            hipLaunchKernelGGL((k_steps_d2q9<S, true, RI, WO>), grid, dim3(MS_THREADS), 0, st, src,
                               dst, g, r, ly, nstrips);
        else
            hipLaunchKernelGGL((k_steps_d2q9<S, false, RI, WO>), grid, dim3(MS_THREADS), 0, st,
                               src, dst, g, r, ly, nstrips);
        return hipGetLastError();
    });
}

hipError_t launch_steps(int nsteps, const Geo& g, const Rates& r, const double* src, double* dst,
                        hipStream_t st, bool rin, bool wout) {
    switch (nsteps) {
        case 2: return launch_steps_t<2>(g, r, src, dst, st, rin, wout);
        case 4: return launch_steps_t<4>(g, r, src, dst, st, rin, wout);
        case 8: return launch_steps_t<8>(g, r, src, dst, st, rin, wout);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace lbm
