// The two-wave march of eight D2Q9 steps with two columns a lane.
#pragma once

#include "lbm_march.h"

namespace lbm {
namespace {

// ---------------------------------------------------------------------------
// Eight steps as the one-wave march takes them, by two waves: the first does steps 1
// to 4 of a row, the second 5 to 8 of the row that the first left in LDS in the
// iteration before, with a barrier an iteration.  A lane has two neighbouring columns,
// so that 112 of 128 columns count (48 of 64 with one wave) and a shift by one column
// moves one of the two: 5.5 vector instructions a column and step against 7.4.  The
// rows of eight steps and one column fill a wave's registers just as those of four
// steps and two columns do.  The first wave's input goes from memory into LDS by itself
// (global_load_lds), a row ahead: prefetched in registers it spilled (4096^2, 8 steps:
// 545 us).  Same arithmetic a node, so bitwise single steps.
//
// Bounds: memory.  4096^2, 8 steps: 349 us by one wave, which issues vector
// instructions three quarters of the time at a clock of 1.9 GHz; 312-321 us here, about
// 5.6 TB/s with the halos.  Two rows ahead: no change.
// ---------------------------------------------------------------------------
constexpr int MP_THREADS = 128, MP_STEPS = 8, MP_STAGES = 4;
constexpr int MP_COLUMNS = 128, MP_WIDTH = MP_COLUMNS - 2 * MP_STEPS;

typedef double MpTwo __attribute__((ext_vector_type(2)));

// Rows a wave keeps of its four stages, per column of the lane (MsState).
struct MpState {
    double z[MP_STAGES][2][3];
    double u[2][MP_STAGES][2][3];
};

// Four stages on one row of quantities (FORM_MOM), in place.
template <int P, bool UP>
__device__ __forceinline__ void mp_stages(MpState& st, Mom2 (&mom)[2], const FoldedRates& r) {
#pragma unroll
    for (int j = 0; j < MP_STAGES; ++j) {
        double f[2][9], in[2][9];
#pragma unroll
        for (int c = 0; c < 2; ++c) expand_d2q9(mom[c], r, f[c]);
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            double v[2] = {f[0][i], f[1][i]};
            if (ms_ex(i) == 1) {
                v[0] = lane_shift<1>(f[1][i]);
                v[1] = f[0][i];
            } else if (ms_ex(i) == -1) {
                v[0] = f[1][i];
                v[1] = lane_shift<-1>(f[0][i]);
            }
            const int ey = UP ? -ms_ey(i) : ms_ey(i);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                if (ey == -1) {
                    in[c][i] = v[c];
                } else if (ey == 0) {
                    in[c][i] = st.z[j][c][ms_yslot(i)];
                    st.z[j][c][ms_yslot(i)] = v[c];
                } else {
                    in[c][i] = st.u[P][j][c][ms_yslot(i)];
                    st.u[P][j][c][ms_yslot(i)] = v[c];
                }
            }
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) moments_d2q9(in[c], r, mom[c]);
    }
}

// The lane, found anew: kept over the stages it costs a register that spills.
__device__ __forceinline__ int mp_lane() {
    int v;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(v));
    return v;
}
// A row of a wave: the quantities of the lane's two columns.
__device__ __forceinline__ void mp_get(MpTwo (&row)[6][64], int lane, Mom2 (&mom)[2]) {
    MpTwo m[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) m[i] = row[i][lane];
#pragma unroll
    for (int c = 0; c < 2; ++c) mom[c] = Mom2{m[0][c], m[1][c], m[2][c], m[3][c], m[4][c], m[5][c]};
}
__device__ __forceinline__ void mp_planes(const Mom2 (&mom)[2], MpTwo (&p)[6]) {
    p[0] = MpTwo{mom[0].th, mom[1].th};
    p[1] = MpTwo{mom[0].jx, mom[1].jx};
    p[2] = MpTwo{mom[0].jy, mom[1].jy};
    p[3] = MpTwo{mom[0].hPx, mom[1].hPx};
    p[4] = MpTwo{mom[0].hPy, mom[1].hPy};
    p[5] = MpTwo{mom[0].Pxy, mom[1].Pxy};
}
// The barrier of an iteration: LDS writes done, loads into LDS still in flight.
__device__ __forceinline__ void mp_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Rows [ys, ye) of the columns [x0, x0 + MP_WIDTH), from FORM_MOM to FORM_MOM.
template <bool UP>
__device__ __forceinline__ void mp_tile(const double* __restrict__ src, double* __restrict__ dst,
                                        int nx, int ny, const FoldedRates& r, int x0, int ys,
                                        int ye, MpTwo (*row)[6][64], MpTwo (*pre)[6][64]) {
    constexpr int S = MP_STEPS;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int nrows = ye - ys;
    const int last = nrows + 2 * S;  // iterations 0 .. last
    MpState st;
#pragma unroll
    for (int j = 0; j < MP_STAGES; ++j)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int a = 0; a < 3; ++a) st.z[j][c][a] = st.u[0][j][c][a] = st.u[1][j][c][a] = 0.0;
    if (wave == 0) {
        const int gx = wrapi(x0 - S + 2 * lane, nx);
        auto fetch = [&](int k, int buf) {
            const int y = wrapi(UP ? ye - 1 + S - k : ys - S + k, ny) * nx;
            const MsAddr<true, 6> a(y + gx);
#pragma unroll
            for (int i = 0; i < 6; ++i)
                __builtin_amdgcn_global_load_lds(
                    (__attribute__((address_space(1))) void*)(wave_base(src + (int64_t)i * CHUNK) +
                                                              a.off),
                    (__attribute__((address_space(3))) void*)&pre[buf][i][0], 16, 0, 0);
        };
        auto step = [&](auto par, int k) {
            constexpr int P = decltype(par)::value;
            // vmcnt(0): the row that the iteration before asked for
            __builtin_amdgcn_s_waitcnt(0x0f70);
            asm volatile("" ::: "memory");
            Mom2 mom[2];
            mp_get(pre[P], lane, mom);
            fetch(k + 1, 1 - P);
            __builtin_amdgcn_sched_barrier(0);
            mp_stages<P, UP>(st, mom, r);
            MpTwo p[6];
            mp_planes(mom, p);
#pragma unroll
            for (int i = 0; i < 6; ++i) row[P][i][lane] = p[i];
            mp_barrier();
        };
        fetch(0, 0);
        int k = 0;
        for (; k + 1 <= last; k += 2) {
            step(std::integral_constant<int, 0>{}, k);
            step(std::integral_constant<int, 1>{}, k + 1);
        }
        if (k <= last) step(std::integral_constant<int, 0>{}, k);
    } else {
        // row k of the upper stages is the row that the other wave left in
        // iteration k - 1
        const bool own = lane >= S / 2 && lane < 64 - S / 2 && x0 - S + 2 * lane < nx;
        auto step = [&](auto par, int k) {
            constexpr int P = decltype(par)::value;
            Mom2 mom[2];
            mp_get(row[1 - P], mp_lane(), mom);
            mp_stages<P, UP>(st, mom, r);
            if (k >= 2 * S + 1 && own) {
                const int y = (UP ? ye + 2 * S - k : ys - 2 * S - 1 + k) * nx;
                const MsAddr<true, 6> a(y + x0 - S + 2 * mp_lane());
                MpTwo p[6];
                mp_planes(mom, p);
#pragma unroll
                for (int i = 0; i < 6; ++i)
                    __builtin_nontemporal_store(
                        p[i], (__attribute__((address_space(1))) MpTwo*)(
                                  wave_base(dst + (int64_t)i * CHUNK) + a.off));
            }
            mp_barrier();
        };
        int k = 0;
        for (; k + 1 <= last; k += 2) {
            step(std::integral_constant<int, 0>{}, k);
            step(std::integral_constant<int, 1>{}, k + 1);
        }
        if (k <= last) step(std::integral_constant<int, 0>{}, k);
    }
}

}  // namespace
}  // namespace lbm
