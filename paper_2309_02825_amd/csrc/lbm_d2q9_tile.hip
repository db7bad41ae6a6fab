// D2Q9 passes of up to eight steps for grids that do not fill the chip: a
// workgroup per tile, the tile in registers.
#include <algorithm>

#include "lbm_march.h"

namespace lbm {
namespace {

// ---------------------------------------------------------------------------
// S steps (1 <= S <= 8) of one tile.  The block's waves own R consecutive rows of
// 64 columns each, one above the other: rin = rows + 2S rows and 64 columns with
// a halo of S on every side, of which the inner `rows` x (64 - 2S) are stored.
// All rows advance together, one step at a time: x neighbours come from DPP lane
// shifts, y neighbours from the wave's own registers, and only the outermost rows
// of a wave (three populations each) go to the next wave through LDS, written at
// the lane's own column and read one column to the side; two buffers alternate,
// so a step has one barrier.
//
// The one-wave march of k_steps_d2q9 walks its rows one after the other, and a
// segment computes 2S rows of pipeline fill whatever its length: at 320^2 a wave
// marches 24 rows for 8 rows of output while most of the chip is idle.  Here the
// rows of a segment are computed side by side.  What bounds it: the issue of a
// SIMD's rows, 43 VALU instructions each (40^2: 0.45 us a step for 6 rows a SIMD),
// after 3.4 us of launch, loads and stores; at 700^2 the loads and stores, which do
// not overlap the steps.
// ---------------------------------------------------------------------------
constexpr int TILE_MAX_WAVES = 8;
constexpr int TILE_ROW = 66;  // a row of 64 doubles in LDS and one to each side

template <int R, bool TWINS>
struct TileRows {
    double f[R][TWINS ? 7 : 9];  // post-collision populations; TWINS: 7 = 5, 8 = 6
};
template <bool TWINS>
__device__ __forceinline__ constexpr int tile_plane(int i) {
    return TWINS ? twin<2>(i) : i;
}

// Hands the outer rows of a wave to its neighbours.
template <int R, bool TWINS>
__device__ __forceinline__ void tile_publish(const TileRows<R, TWINS>& a, double* xch, int wave) {
    double* own = xch + wave * 6 * TILE_ROW + 1 + (threadIdx.x & 63);
    own[0 * TILE_ROW] = a.f[R - 1][2];
    own[1 * TILE_ROW] = a.f[R - 1][5];
    own[2 * TILE_ROW] = a.f[R - 1][6];
    own[3 * TILE_ROW] = a.f[0][4];
    own[4 * TILE_ROW] = a.f[0][tile_plane<TWINS>(7)];
    own[5 * TILE_ROW] = a.f[0][tile_plane<TWINS>(8)];
}

// One step: from `a` (post-collision, TWINS as read) to `b` (post-collision; may
// be `a`: a row is replaced once the values that its neighbours pull are taken).
// The inner rows come first, while the neighbours' rows are on their way from LDS.
// MOM: `b` receives the planes of FORM_MOM instead.
template <int R, bool TWINS, bool MOM>
__device__ __forceinline__ void tile_step(TileRows<R, TWINS>& a, TileRows<R, true>& b,
                                          const double* xch, int wave, int waves,
                                          const FoldedRates& fr) {
    constexpr int P7 = tile_plane<TWINS>(7), P8 = tile_plane<TWINS>(8);
    // rows outside the tile: any value, it stays in the halo
    const double* up = xch + max(wave - 1, 0) * 6 * TILE_ROW + 1 + (threadIdx.x & 63);
    const double* dn = xch + min(wave + 1, waves - 1) * 6 * TILE_ROW + 1 + (threadIdx.x & 63);
    const double u2 = up[0], u5 = up[1 * TILE_ROW - 1], u6 = up[2 * TILE_ROW + 1];
    const double e4 = dn[3 * TILE_ROW], e7 = dn[4 * TILE_ROW + 1], e8 = dn[5 * TILE_ROW - 1];
    // what row 0 pulls from row 1, and the next row from the one above it
    const double m4 = R > 1 ? a.f[R > 1 ? 1 : 0][4] : e4;
    const double m7 = R > 1 ? lane_shift<-1>(a.f[R > 1 ? 1 : 0][P7]) : e7;
    const double m8 = R > 1 ? lane_shift<1>(a.f[R > 1 ? 1 : 0][P8]) : e8;
    double p2 = a.f[0][2], p5 = lane_shift<1>(a.f[0][5]), p6 = lane_shift<-1>(a.f[0][6]);
#pragma unroll
    for (int q = 1; q <= R; ++q) {
        const int r = q % R;  // rows 1 .. R - 1, then row 0
        double in[9];
        in[0] = a.f[r][0];
        in[1] = lane_shift<1>(a.f[r][1]);
        in[3] = lane_shift<-1>(a.f[r][3]);
        if (r == 0) {
            in[2] = u2;
            in[5] = u5;
            in[6] = u6;
            in[4] = m4;
            in[7] = m7;
            in[8] = m8;
        } else {
            in[2] = p2;
            in[5] = p5;
            in[6] = p6;
            in[4] = r < R - 1 ? a.f[r < R - 1 ? r + 1 : r][4] : e4;
            in[7] = r < R - 1 ? lane_shift<-1>(a.f[r < R - 1 ? r + 1 : r][P7]) : e7;
            in[8] = r < R - 1 ? lane_shift<1>(a.f[r < R - 1 ? r + 1 : r][P8]) : e8;
            p2 = a.f[r][2];
            p5 = lane_shift<1>(a.f[r][5]);
            p6 = lane_shift<-1>(a.f[r][6]);
        }
        Mom2 m;
        moments_d2q9(in, fr, m);
        if (MOM)
            ms_planes(m, in);
        else
            expand_d2q9(m, fr, in);
#pragma unroll
        for (int i = 0; i < (MOM ? 6 : 7); ++i) b.f[r][i] = in[i];
    }
}

template <int R, int IN, int OUT>
__global__ void __launch_bounds__(64 * TILE_MAX_WAVES)
k_tile_d2q9(const double* __restrict__ src, double* __restrict__ dst, Geo g, Rates r, int S,
            int rows, int nstrips) {
    extern __shared__ double xch[];  // [2][waves][6][TILE_ROW]
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int waves = (int)blockDim.x >> 6;
    const unsigned t = xcd_remap(blockIdx.x, gridDim.x);
    const int x0 = (int)(t % (unsigned)nstrips) * (64 - 2 * S);
    const int y0 = (int)(t / (unsigned)nstrips) * rows;
    const int gx = wrapi(x0 - S + lane, g.nx);
    const int top = wave * R;                        // first row of this wave in the tile
    const int rin = min(rows, g.ny - y0) + 2 * S;    // rows of the tile that are needed
    const FoldedRates fr = folded(r);
    constexpr bool TWINS = IN != FORM_FULL;
    TileRows<R, TWINS> a;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const MsAddr<true, form_planes<2>(IN)> at(wrapi(y0 - S + top + q, g.ny) * g.nx + gx);
#pragma unroll
        for (int i = 0; i < 9; ++i)
            if (form_holds<2>(IN, i)) a.f[q][i] = at.load(src, i);
    }
    if constexpr (IN == FORM_MOM) {
#pragma unroll
        for (int q = 0; q < R; ++q) {
            double f[9];
            expand_d2q9(Mom2{a.f[q][0], a.f[q][1], a.f[q][2], a.f[q][3], a.f[q][4], a.f[q][5]}, fr, f);
#pragma unroll
            for (int i = 0; i < 7; ++i) a.f[q][i] = f[i];
        }
    }
    TileRows<R, true> b;
    const int half = waves * 6 * TILE_ROW;
    // step s needs rows s .. rin - 1 - s of its result (one less at each end per
    // step): a wave computes while it holds one of them
    auto needed = [&](int s) { return top + R > s && top < rin - s; };
    tile_publish<R, TWINS>(a, xch, wave);
    __syncthreads();
    constexpr bool MOM = OUT == FORM_MOM;
    if (S == 1) {
        if (needed(1)) tile_step<R, TWINS, MOM>(a, b, xch, wave, waves, fr);
    } else {
        if (needed(1)) {
            tile_step<R, TWINS, false>(a, b, xch, wave, waves, fr);
            tile_publish<R, true>(b, xch + half, wave);
        }
        for (int s = 2; s < S; ++s) {
            __syncthreads();
            if (needed(s)) {
                tile_step<R, true, false>(b, b, xch + ((s & 1) ? 0 : half), wave, waves, fr);
                tile_publish<R, true>(b, xch + ((s & 1) ? half : 0), wave);
            }
        }
        __syncthreads();
        if (needed(S)) tile_step<R, true, MOM>(b, b, xch + ((S & 1) ? 0 : half), wave, waves, fr);
    }
    const int x = x0 - S + lane;
    if (lane >= S && lane < 64 - S && x < g.nx) {
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int row = top + q;
            if (row >= S && row < rin - S) {
                const MsAddr<true, form_planes<2>(OUT)> at((y0 - S + row) * g.nx + x);
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    if (form_holds<2>(OUT, i)) at.store_cached(dst, i, b.f[q][twin<2>(i)]);
            }
        }
    }
}

}  // namespace

// Rows of a tile where a run on this grid goes by tiles, 0 where it goes by the
// march.  Tiles win while one block per CU holds the grid in tiles of at most 48 rows
// (8 rows a wave; more spill): the smallest tiles that do, since every block of the
// round then computes the least (us a step, march and tiles: 40^2 1.86 and 0.83,
// 320^2 2.02 and 1.24, 512^2 2.13 and 1.72, 700^2 3.27 and 2.61).  In a second round
// the blocks' loads and stores no longer hide behind one another (1000 x 700 3.52 and
// 3.70), where the march's rows do.
int tile_rows(const Geo& g) {
    constexpr int kMinRows = 2, kMaxRows = 48;
    const int cus = compute_units(), w = 64 - 2 * MAX_STEPS_PER_PASS;
    const int nstrips = (g.nx + w - 1) / w;
    if (nstrips > cus || !ms_off32(g)) return 0;
    const int nseg = cus / nstrips;
    const int rows = std::max(kMinRows, (g.ny + nseg - 1) / nseg);
    return rows <= kMaxRows ? rows : 0;
}

hipError_t launch_tile(int nsteps, const Geo& g, const Rates& r, const double* src, double* dst,
                       hipStream_t st, int in, int out) {
    const int rows = tile_rows(g);
    if (nsteps < 1 || nsteps > MAX_STEPS_PER_PASS || rows == 0) return hipErrorInvalidValue;
    const int w = 64 - 2 * nsteps;
    const int nstrips = (g.nx + w - 1) / w, nseg = (g.ny + rows - 1) / rows;
    const int R = (rows + 2 * nsteps + TILE_MAX_WAVES - 1) / TILE_MAX_WAVES;
    const int waves = (rows + 2 * nsteps + R - 1) / R;
    const dim3 grid((unsigned)(nstrips * nseg)), block(64 * waves);
    const size_t lds = (size_t)2 * waves * 6 * TILE_ROW * sizeof(double);  // at most 51 KB
    return dispatch_form(in, [&](auto fi) {
        return dispatch_form(out, [&](auto fo) {
            constexpr int IN = decltype(fi)::value, OUT = decltype(fo)::value;
            switch (R) {
#define LBM_TILE(RR)                                                                         \
    case RR:                                                                                 \
        hipLaunchKernelGGL((k_tile_d2q9<RR, IN, OUT>), grid, block, lds, st, src, dst, g, r, \
                           nsteps, rows, nstrips);                                           \
        break;
                LBM_TILE(1)
                LBM_TILE(2)
                LBM_TILE(3)
                LBM_TILE(4)
                LBM_TILE(5)
                LBM_TILE(6)
                LBM_TILE(7)
                LBM_TILE(8)
#undef LBM_TILE
                default: return hipErrorInvalidValue;
            }
            return hipGetLastError();
        });
    });
}

}  // namespace lbm
