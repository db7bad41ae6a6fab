// The one-wave march of several D2Q9 steps, shared by the plain, adjoint and
// batched passes.
#pragma once

#include "lbm_device.h"

namespace lbm {
namespace {

// ---------------------------------------------------------------------------
// S D2Q9 time steps per pass over HBM (temporal blocking).
//
// One wave (64 lanes) owns a strip of 64 - 2S output columns plus an
// S-column halo on each side; lane t owns column x0 - S + t in every stage.
// The wave marches down a segment of rows: in iteration k it loads input
// row ys - S + k and stage j = 1..S computes row ys - S + k - j of step j from
// rows (that row + {-1, 0, +1}) of step j - 1.  Only stage S stores, so each
// value crosses HBM once per S steps (plus the halo).
//
// Exchange between stages never leaves the wave: a population with e_x = +1
// (-1) is pulled from the lane on the left (right) with a DPP wave shift
// (wave_shr:1 / wave_shl:1, two 32-bit moves per double), e_x = 0 stays in
// its lane.  Rows are delayed in registers: e_y = -1 is used in the
// iteration it arrives, e_y = 0 one iteration later, e_y = +1 two iterations
// later (two registers that alternate with the row parity; the march is
// unrolled by two so that the parity is static).  No LDS and no barrier.
//
// Every lane computes every stage (halo lanes produce values that only halo
// lanes consume); only stage S stores, from its valid lanes.  The first 2S
// iterations fill the pipeline (stage j holds valid rows from iteration 2j
// on) and are unrolled at compile time with the stages that are already
// valid, so the steady-state loop has no per-stage branch.  The arithmetic is
// collide<2> S times, so the result is bitwise that of S single steps.
// ---------------------------------------------------------------------------

// Addressing of a D2Q9 chunked buffer by node index k (population i at
// slot<9>(i, k)).  MsAddr<true>: the byte offset of population 0 as a 32-bit
// value from the buffer start, population i then at a base that is the same
// for the whole wave (buffer + i chunks), held in scalar registers; every
// access is one load or store with a scalar base and a 32-bit lane offset, and
// no 64-bit address arithmetic per access (the buffer must be under 4 GiB).
// MsAddr<false>: 64-bit element indices, any size.  Both address the same
// element, so the arithmetic and the results do not depend on the choice.
typedef __attribute__((address_space(1))) char GChar;
typedef __attribute__((address_space(1))) double GDouble;
__device__ __forceinline__ GChar* wave_base(const double* p) {
    const unsigned long long v = (unsigned long long)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return (GChar*)(((unsigned long long)hi << 32) | lo);
}
template <bool OFF32, int Q = 9> struct MsAddr;  // Q: planes of the buffer
typedef unsigned int MsU2 __attribute__((__vector_size__(8)));  // a double as buffer data
template <int Q> struct MsAddr<true, Q> {
    unsigned off;
    __device__ __forceinline__ explicit MsAddr(int k)
        : off((unsigned)((((k >> 12) * Q) << 12) | (k & (CHUNK - 1))) * 8u) {}
    __device__ __forceinline__ double load(const double* p, int i) const {
        return *(GDouble*)(wave_base(p + (int64_t)i * CHUNK) + off);
    }
    __device__ __forceinline__ void store(double* p, int i, double v) const {
        __builtin_nontemporal_store(v, (GDouble*)(wave_base(p + (int64_t)i * CHUNK) + off));
    }
    __device__ __forceinline__ void store_cached(double* p, int i, double v) const {
        *(GDouble*)(wave_base(p + (int64_t)i * CHUNK) + off) = v;
    }
};
template <int Q> struct MsAddr<false, Q> {
    int k;
    __device__ __forceinline__ explicit MsAddr(int k_) : k(k_) {}
    __device__ __forceinline__ double load(const double* p, int i) const { return p[slot<Q>(i, k)]; }
    __device__ __forceinline__ void store(double* p, int i, double v) const {
        __builtin_nontemporal_store(v, p + slot<Q>(i, k));
    }
    __device__ __forceinline__ void store_cached(double* p, int i, double v) const {
        p[slot<Q>(i, k)] = v;
    }
};
// Whether a D2Q9 state buffer of g allows MsAddr<true>.
__host__ __device__ inline bool ms_off32(const Geo& g) {
    return (uint64_t)9 * (uint64_t)chunks_of(g.V) * CHUNK * sizeof(double) <= 0xffffffffull;
}

// Whether the plain D2Q9 passes write with cached stores (states_fit_cache).  GLUPS of
// passes that handed on 7 planes, non-temporal / cached: 1024^2 196 / 207, 1280^2
// 216 / 247, 1448^2 (288 MiB) 215 / 220, 1600^2 (352 MiB) 231 / 223, 4096^2 280 / 266.
// With 6 planes a pass moves two thirds of what the rule counts, and 1600^2 takes 65.5 us
// non-temporal and 61.7 cached, 2048^2 97.5 and 95.8.
inline bool d2q9_cached_stores(const Geo& g) { return states_fit_cache(2, g); }

template <int S, int DEPTH = 1>
struct MsState {
    double pre[DEPTH][9];  // next input rows (prefetched DEPTH rows ahead)
    double z[S][3];     // e_y = 0 populations of the previous row, per stage input
    double u[2][S][3];  // e_y = +1 populations of the rows of each parity
};

// The populations of a node from the planes of a buffer in form IN, and the
// planes of FORM_MOM.
template <int IN>
__device__ __forceinline__ void ms_populations(const double (&pre)[9], const FoldedRates& r,
                                               double (&f)[9]) {
    if constexpr (IN == FORM_MOM) {
        expand_d2q9(Mom2{pre[0], pre[1], pre[2], pre[3], pre[4], pre[5]}, r, f);
    } else {
#pragma unroll
        for (int i = 0; i < 9; ++i) f[i] = pre[IN == FORM_TWIN ? twin<2>(i) : i];
    }
}
__device__ __forceinline__ void ms_planes(const Mom2& m, double (&p)[9]) {
    p[0] = m.th;
    p[1] = m.jx;
    p[2] = m.jy;
    p[3] = m.hPx;
    p[4] = m.hPy;
    p[5] = m.Pxy;
}

// One iteration k of the march; P = k & 1; stages above ACTIVE are skipped
// (pipeline fill), stage S stores only when ACTIVE == S.  ALL: stage j < S
// also stores its rows of [ys, ye) to dst - (S - j) stride (the state after
// j steps, for a caller that keeps every intermediate state).  NT: stage S
// writes with non-temporal stores (otherwise through the caches).  UP: the
// march runs from row ye - 1 + S up to ys - S, so the roles of e_y = +1 and
// e_y = -1 in the row delays swap (same arithmetic per node).
template <int S, int P, int ACTIVE, bool ALL, bool OFF32, bool NT = true,
          int IN = FORM_FULL, int OUT = FORM_FULL, bool UP = false, int DEPTH = 1>
__device__ __forceinline__ void ms_row(MsState<S, DEPTH>& st, int k,
                                       const double* __restrict__ src, double* __restrict__ dst,
                                       int nx, int ny, int gx, int ys, int x0, const FoldedRates& r,
                                       int nrows, int64_t stride) {
    constexpr int W = MS_THREADS - 2 * S;
    const int lane = threadIdx.x;
    double f[9];
    ms_populations<IN>(st.pre[P % DEPTH], r, f);
    {
        // Prefetch the next input row.  In the last iteration the row is not
        // used (its address is wrapped, so in bounds); loading it anyway
        // keeps the memory counters equal on both sides of the branch a
        // conditional load would need, so the wait at the row start is not
        // widened by a missing load (512^2: 90 -> 106 GLUPS).  The masked
        // stores of stage S still make that wait cover the previous row's
        // stores; two waves per SIMD hide it.
        const int row = UP ? ys + nrows - 1 + S - (k + DEPTH) : ys - S + k + DEPTH;
        const MsAddr<OFF32, form_planes<2>(IN)> a(wrapi(row, ny) * nx + gx);
#pragma unroll
        for (int i = 0; i < 9; ++i)
            if (form_holds<2>(IN, i)) st.pre[P % DEPTH][i] = a.load(src, i);
    }
#pragma unroll
    for (int j = 1; j <= S; ++j) {
        // inputs of stage j: stage j-1 rows of iterations k (e_y = -1), k-1
        // (e_y = 0) and k-2 (e_y = +1), pulled from lane t - e_x (marching
        // up, e_y = +1 and -1 trade places)
        double in[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const double v = ms_ex(i) == 0 ? f[i]
                                           : (ms_ex(i) == 1 ? lane_shift<1>(f[i]) : lane_shift<-1>(f[i]));
            const int ey = UP ? -ms_ey(i) : ms_ey(i);
            if (ey == -1) {
                in[i] = v;
            } else if (ey == 0) {
                in[i] = st.z[j - 1][ms_yslot(i)];
                st.z[j - 1][ms_yslot(i)] = v;
            } else {
                in[i] = st.u[P][j - 1][ms_yslot(i)];
                st.u[P][j - 1][ms_yslot(i)] = v;
            }
        }
        if (j <= ACTIVE) {
            Mom2 mom;
            moments_d2q9(in, r, mom);
            if (j < S || OUT != FORM_MOM)
                expand_d2q9(mom, r, in);
            else
                ms_planes(mom, in);
#pragma unroll
            for (int i = 0; i < 9; ++i) f[i] = in[i];
            if (j == S && ACTIVE == S && lane >= S && lane < S + W && x0 - S + lane < nx) {
                const int row = UP ? ys + nrows - 1 + 2 * S - k : ys - 2 * S + k;
                const MsAddr<OFF32, form_planes<2>(OUT)> a(wrapi(row, ny) * nx + x0 - S + lane);
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    if (!form_holds<2>(OUT, i)) continue;
                    if constexpr (NT)
                        a.store(dst, i, in[i]);
                    else
                        a.store_cached(dst, i, in[i]);
                }
            }
            if (ALL && j < S) {
                // row ys + k - S - j of step j; lanes S .. S+W-1 hold valid
                // values from stage j on (the valid band shrinks one lane per
                // side per stage)
                const int rr = k - S - j;
                if (rr >= 0 && rr < nrows && lane >= S && lane < S + W && x0 - S + lane < nx) {
                    const MsAddr<OFF32> a((UP ? ys + nrows - 1 - rr : ys + rr) * nx + x0 - S + lane);
                    double* out = dst - (int64_t)(S - j) * stride;
                    if constexpr (OFF32) {
                        // a buffer descriptor per state and the plane as a
                        // scalar offset shared by all S states: a 64-bit
                        // base per plane and state would exceed the scalar
                        // registers (they spill into VGPR lanes).  Records:
                        // the bytes of one state (below 2^32 here); cache
                        // policy 2 is the non-temporal hint of the other
                        // stores.
                        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                            out, (short)0, (int)(unsigned)((uint64_t)9 * CHUNK * 8 *
                                                          (uint64_t)((nx * ny + CHUNK - 1) >> 12)),
                            0x00020000);
#pragma unroll
                        for (int i = 0; i < 9; ++i)
                            if (form_holds<2>(OUT, i))
                                __builtin_amdgcn_raw_buffer_store_b64(
                                    __builtin_bit_cast(MsU2, in[i]), rs, a.off, i * CHUNK * 8, 2);
                    } else {
#pragma unroll
                        for (int i = 0; i < 9; ++i)
                            if (form_holds<2>(OUT, i)) a.store(out, i, in[i]);
                    }
                }
            }
        }
    }
}

template <int S, int K, bool ALL, bool OFF32, bool NT = true, int IN = FORM_FULL,
          int OUT = FORM_FULL, bool UP = false, int DEPTH = 1>
__device__ __forceinline__ void ms_fill(MsState<S, DEPTH>& st, const double* __restrict__ src,
                                        double* __restrict__ dst, int nx, int ny, int gx, int ys,
                                        int x0, const FoldedRates& r, int nrows, int64_t stride) {
    if constexpr (K < 2 * S) {
        ms_row<S, K & 1, K / 2, ALL, OFF32, NT, IN, OUT, UP, DEPTH>(st, K, src, dst, nx, ny, gx, ys, x0,
                                                               r, nrows, stride);
        ms_fill<S, K + 1, ALL, OFF32, NT, IN, OUT, UP, DEPTH>(st, src, dst, nx, ny, gx, ys, x0, r, nrows,
                                                         stride);
    }
}

// DEPTH (1 or 2, the period of the row pairs): input rows loaded ahead.
// Advance rows [ys, ye) (ye > ys) of the columns [x0, x0 + 64 - 2S) of one
// D2Q9 grid by S steps (reads rows ys-S .. ye-1+S and columns x0-S ..
// x0+63-S, wrapped periodically), marching down the rows or, with UP, up.
// All 64 lanes of the wave must be active.
template <int S, bool ALL, bool OFF32, bool NT = true, int IN = FORM_FULL,
          int OUT = FORM_FULL, bool UP = false, int DEPTH = 1>
__device__ __forceinline__ void ms_tile(const double* __restrict__ src, double* __restrict__ dst,
                                        int nx, int ny, const FoldedRates& r, int x0, int ys,
                                        int ye, int64_t stride = 0) {
    const int gx = wrapi(x0 - S + (int)threadIdx.x, nx);
    const int kend = ye - ys + 2 * S - 1;  // >= 2S
    MsState<S, DEPTH> st;
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
        const MsAddr<OFF32, form_planes<2>(IN)> a(wrapi(UP ? ye - 1 + S - d : ys - S + d, ny) * nx + gx);
#pragma unroll
        for (int i = 0; i < 9; ++i)
            if (form_holds<2>(IN, i)) st.pre[d][i] = a.load(src, i);
    }
#pragma unroll
    for (int j = 0; j < S; ++j)
#pragma unroll
        for (int a = 0; a < 3; ++a) st.z[j][a] = st.u[0][j][a] = st.u[1][j][a] = 0.0;
    const int nrows = ye - ys;
    ms_fill<S, 0, ALL, OFF32, NT, IN, OUT, UP, DEPTH>(st, src, dst, nx, ny, gx, ys, x0, r, nrows,
                                                 stride);
    // whole row pairs in the loop and a last odd row after it: the loop then
    // has a single path back to its head, and the compiler keeps the row
    // delays in place instead of copying them at the join (bitwise the same;
    // 37 instead of 52 copies per row pair)
    int k = 2 * S;
    for (; k + 1 <= kend; k += 2) {
        ms_row<S, 0, S, ALL, OFF32, NT, IN, OUT, UP, DEPTH>(st, k, src, dst, nx, ny, gx, ys, x0, r,
                                                       nrows, stride);
        ms_row<S, 1, S, ALL, OFF32, NT, IN, OUT, UP, DEPTH>(st, k + 1, src, dst, nx, ny, gx, ys, x0, r,
                                                       nrows, stride);
    }
    if (k <= kend)
        ms_row<S, 0, S, ALL, OFF32, NT, IN, OUT, UP, DEPTH>(st, k, src, dst, nx, ny, gx, ys, x0, r,
                                                       nrows, stride);
}

}  // namespace

// Minimum rows per segment: plain passes 8; the passes of an adjoint
// checkpoint segment (recomputation and reverse sweep) 3, since at the sizes
// the adjoint runs (512^2) they are short of waves (measured per step of a
// 45-step segment at 512^2: 15.1 us at 8 rows, 12.9 us at 3).
constexpr int kMinRows = 8;
constexpr int kMinRowsSegment = 3;

// slots: blocks of one round, 0 for those of the one-wave march.
int steps_rows(const Geo& g, int nstrips, int min_rows, int slots = 0);
// The same for a plain pass of nsteps, which may leave half of the round empty.
int pass_rows(const Geo& g, int nstrips, int min_rows, int nsteps, bool* half);

}  // namespace lbm
