// D2Q9 passes of several steps: the choice of a pass.
#include <algorithm>
#include <atomic>

#include "lbm_d2q9_pass.h"

namespace lbm {

// Compute units of the current device, looked up once per device.
int compute_units() {
    constexpr int kMaxDevices = 64;
    static std::atomic<int> cached[kMaxDevices] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) dev = 0;
    const int d = dev < kMaxDevices ? dev : kMaxDevices - 1;
    int cus = cached[d].load(std::memory_order_relaxed);
    if (cus == 0) {
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            cus <= 0)
            cus = 256;
        cached[d].store(cus, std::memory_order_relaxed);
    }
    return cus;
}
// Blocks of k_steps_d2q9 one round holds (8 per CU).
static int round_slots() { return 8 * compute_units(); }

// Rows per segment of an S-step launch.  A one-wave block of k_steps_d2q9
// holds about 250 VGPRs, so a CU runs 8 of them at once: the segments are
// cut so that all blocks fit in one round of 8 x (number of CUs) (fewer,
// longer segments amortise the 2S-row pipeline fill; a partial second round
// costs far more), at least min_rows, and in more rounds when a segment would
// exceed 512 rows.  Half a round, one wave per SIMD, is taken instead where it is
// faster: a row then takes 0.83 us (k_steps_d2q9_half) against 1.47 with two waves on
// the SIMD, and a segment of ly rows costs ly + S of them (its fill computes half of
// 2S rows), so that halving the fill wins below 27 rows at eight steps (us a step,
// 2,048 and 1,024 slots: 800^2 3.36 and 2.82, 1000 x 700 3.44 and 2.92, 1280^2 5.56
// and 5.40, 1448^2 7.08 and 6.92; 1800^2, 34 rows, 10.16 and 10.23).  Shorter passes
// only where the state stays in the Infinity Cache (4 steps: 1024^2 5.21 and 4.88,
// 1448^2 11.0 and 11.1).
int pass_rows(const Geo& g, int nstrips, int min_rows, int nsteps, bool* half) {
    const int two = steps_rows(g, nstrips, min_rows);
    const int64_t nseg = std::max(1, 4 * compute_units() / nstrips);
    const int one = (int)std::min<int64_t>(g.ny, (g.ny + nseg - 1) / nseg);
    *half = one > two && nseg * nstrips <= 4 * compute_units() &&
            0.83 * (one + nsteps) < 1.47 * (two + nsteps) &&
            (nsteps == MAX_STEPS_PER_PASS || states_fit_cache(2, g));
    return *half ? one : two;
}

int steps_rows(const Geo& g, int nstrips, int min_rows, int slots) {
    if (slots == 0) slots = round_slots();
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

int pass_form(int d, const Geo& g) {
    return (d == 2 && ms_off32(g)) || (d == 3 && march3_fits(g)) ? FORM_MOM : FORM_TWIN;
}

extern template hipError_t launch_steps_from<8, FORM_FULL>(const Geo&, const Rates&,
                                                           const double*, double*, hipStream_t,
                                                           int);
extern template hipError_t launch_steps_from<8, FORM_TWIN>(const Geo&, const Rates&,
                                                           const double*, double*, hipStream_t,
                                                           int);
extern template hipError_t launch_steps_from<8, FORM_MOM>(const Geo&, const Rates&,
                                                          const double*, double*, hipStream_t,
                                                          int);
extern template hipError_t launch_steps_t<2>(const Geo&, const Rates&, const double*, double*,
                                             hipStream_t, int, int);
extern template hipError_t launch_steps_t<4>(const Geo&, const Rates&, const double*, double*,
                                             hipStream_t, int, int);

hipError_t launch_steps(int nsteps, const Geo& g, const Rates& r, const double* src, double* dst,
                        hipStream_t st, int in, int out) {
    switch (nsteps) {
        case 2: return launch_steps_t<2>(g, r, src, dst, st, in, out);
        case 4: return launch_steps_t<4>(g, r, src, dst, st, in, out);
        case 8: return launch_steps_t<8>(g, r, src, dst, st, in, out);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace lbm
