// D2Q9 passes of up to eight steps for grids that do not fill the chip: a
// workgroup per tile, the tile in registers.
#include <algorithm>

#include "lbm_march.h"

namespace lbm {
namespace {

// ---------------------------------------------------------------------------
// S steps (2 <= S <= 8) of one tile.  The block's waves own R consecutive rows of
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
constexpr int TILE_ADJOINT_ROWS = 6;  // rows a wave holds of lambda and f (242 VGPRs)
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

// One block runs on a CU (tile_rows), two waves on a SIMD: scheduled for more, with
// fewer registers in flight, 40^2 takes 163 us for 200 steps, 157 so, 700^2 523 and 510.
template <int R, int IN, int OUT>
__global__ void __launch_bounds__(64 * TILE_MAX_WAVES) __attribute__((amdgpu_waves_per_eu(2, 2)))
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

// The same tile keeping every state: step s to out + (s - 1) stride, without the
// twins (the adjoint's recomputation of a checkpoint segment).  Cached stores: the
// reverse sweep reads the states from the Infinity Cache (512^2, 8 steps: 23.3 us,
// 34 us with non-temporal ones, the march 31).
template <int R, int IN>
__global__ void __launch_bounds__(64 * TILE_MAX_WAVES)
k_tile_d2q9_all(const double* __restrict__ src, double* __restrict__ out, int64_t stride, Geo g,
                Rates r, int S, int rows, int nstrips) {
    extern __shared__ double xch[];  // [2][waves][6][TILE_ROW]
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int waves = (int)blockDim.x >> 6;
    const unsigned t = xcd_remap(blockIdx.x, gridDim.x);
    const int x0 = (int)(t % (unsigned)nstrips) * (64 - 2 * S);
    const int y0 = (int)(t / (unsigned)nstrips) * rows;
    const int gx = wrapi(x0 - S + lane, g.nx);
    const int top = wave * R;
    const int rin = min(rows, g.ny - y0) + 2 * S;
    const FoldedRates fr = folded(r);
    constexpr bool TWINS = IN != FORM_FULL;
    TileRows<R, TWINS> a;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const MsAddr<true> at(wrapi(y0 - S + top + q, g.ny) * g.nx + gx);
#pragma unroll
        for (int i = 0; i < 9; ++i)
            if (form_holds<2>(IN, i)) a.f[q][i] = at.load(src, i);
    }
    TileRows<R, true> b;
    const int half = waves * 6 * TILE_ROW;
    const int x = x0 - S + lane;
    const bool own = lane >= S && lane < 64 - S && x < g.nx;
    auto needed = [&](int s) { return top + R > s && top < rin - s; };
    auto keep = [&](int s) {
        double* dst = out + (int64_t)(s - 1) * stride;
#pragma unroll
        for (int q = 0; q < R; ++q)
            if (top + q >= S && top + q < rin - S && own) {
                const MsAddr<true> at((y0 - S + top + q) * g.nx + x);
#pragma unroll
                for (int i = 0; i < 7; ++i) at.store_cached(dst, i, b.f[q][i]);
            }
    };
    tile_publish<R, TWINS>(a, xch, wave);
    __syncthreads();
    if (needed(1)) {
        tile_step<R, TWINS, false>(a, b, xch, wave, waves, fr);
        tile_publish<R, true>(b, xch + half, wave);
        keep(1);
    }
    for (int s = 2; s <= S; ++s) {
        __syncthreads();
        if (needed(s)) {
            tile_step<R, true, false>(b, b, xch + ((s & 1) ? 0 : half), wave, waves, fr);
            tile_publish<R, true>(b, xch + ((s & 1) ? half : 0), wave);
            keep(s);
        }
    }
}

// ---------------------------------------------------------------------------
// S adjoint steps of one tile (the reverse sweep of a checkpoint segment on the
// grids of tile_rows): lambda^{N-S} from lambda^N, the forward tile with every
// velocity reversed and C^T in place of C, and the eps parts <mu, (dC/deps) f^{N-j}>
// of the nodes the block owns.
//
// f^{N-j} is read from its state buffer at each lane's own column, the rows of the
// next step while this one is computed, and pulled along x by lane shifts; f_7 and
// f_8 come from the planes p7 and p8 (5 and 6 in a state written by a collision, 7
// and 8 in the checkpoint, which may be any state).  Every lane sums the parts of its
// nodes over steps and rows, a block its lanes, in a fixed order.
//
// Bounds: FP64 issue at two waves a SIMD (about 190 vector instructions a row and
// step), then the first loads and the last stores, which no other block hides.  512^2:
// 41 us for 7.5 steps, the march 6.5 us a step; with the loads of f behind a branch,
// and so waited for in their own step, 44.
// ---------------------------------------------------------------------------
template <int R>
__global__ void __launch_bounds__(64 * TILE_MAX_WAVES)
k_tile_adjoint_d2q9(const double* __restrict__ src, double* __restrict__ dst,
                    const double* __restrict__ ftop, int64_t stride,
                    const double* __restrict__ ckpt, double* __restrict__ partials, int ntab,
                    Geo g, Rates r, int S, int rows, int nstrips) {
    extern __shared__ double xch[];  // [2][waves][6][TILE_ROW]
    __shared__ double sums[TILE_MAX_WAVES];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int waves = (int)blockDim.x >> 6;
    const unsigned t = xcd_remap(blockIdx.x, gridDim.x);
    const int x0 = (int)(t % (unsigned)nstrips) * (64 - 2 * S);
    const int y0 = (int)(t / (unsigned)nstrips) * rows;
    const int gx = wrapi(x0 - S + lane, g.nx);
    const int top = wave * R;
    const int rin = min(rows, g.ny - y0) + 2 * S;
    const int x = x0 - S + lane;
    const bool own = lane >= S && lane < 64 - S && x < g.nx;
    // byte offsets of the rows top - 1 .. top + R at the lane's column
    unsigned at[R + 2];
#pragma unroll
    for (int q = 0; q < R + 2; ++q)
        at[q] = MsAddr<true>(wrapi(y0 - S + top + q - 1, g.ny) * g.nx + gx).off;
    auto get = [&](const double* p, int plane, unsigned off) {
        return *(GDouble*)(wave_base(p + (int64_t)plane * CHUNK) + off);
    };
    double lam[R][9];
#pragma unroll
    for (int q = 0; q < R; ++q)
#pragma unroll
        for (int i = 0; i < 9; ++i) lam[q][i] = get(src, i, at[q + 1]);
    auto owned = [&](int q) { return top + q >= S && top + q < rin - S; };
    // f^{N-j} of row q, before the lane shifts.  A row that the block does not own, and
    // every row after the last step, reads nothing (tile_read): behind a branch the
    // loads of the next step would be waited for where the branch ends.
    double f[R][9];
    const unsigned bytes = (unsigned)(9 * CHUNK * 8 * ((g.nx * g.ny + CHUNK - 1) / CHUNK));
    auto load_f = [&](int j, int q) {
        const TileRead rd = tile_read(j, S, owned(q));
        const bool last = rd.step == S && ckpt != nullptr;
        const double* fs = last ? ckpt : ftop - (int64_t)(rd.step - 1) * stride;
        const int p7 = last ? 7 : 5, p8 = last ? 8 : 6;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<double*>(fs), (short)0, (int)bytes, 0x00020000);
        auto fetch = [&](int plane, unsigned off) {
            return __builtin_bit_cast(
                double, __builtin_amdgcn_raw_buffer_load_b64(rs, off | rd.skip, plane * (int)CHUNK * 8, 0));
        };
        f[q][0] = fetch(0, at[q + 1]);
        f[q][1] = fetch(1, at[q + 1]);
        f[q][3] = fetch(3, at[q + 1]);
        f[q][2] = fetch(2, at[q]);
        f[q][5] = fetch(5, at[q]);
        f[q][6] = fetch(6, at[q]);
        f[q][4] = fetch(4, at[q + 2]);
        f[q][7] = fetch(p7, at[q + 2]);
        f[q][8] = fetch(p8, at[q + 2]);
    };
#pragma unroll
    for (int q = 0; q < R; ++q) load_f(1, q);
    const int half = waves * 6 * TILE_ROW;
    double ge = 0.0;
    for (int j = 1; j <= S; ++j) {
        double* buf = xch + ((j & 1) ? 0 : half);
        {
            double* line = buf + wave * 6 * TILE_ROW + 1 + lane;
            line[0 * TILE_ROW] = lam[R - 1][4];
            line[1 * TILE_ROW] = lam[R - 1][7];
            line[2 * TILE_ROW] = lam[R - 1][8];
            line[3 * TILE_ROW] = lam[0][2];
            line[4 * TILE_ROW] = lam[0][5];
            line[5 * TILE_ROW] = lam[0][6];
        }
        __syncthreads();
        // step j needs rows j .. rin - 1 - j (as k_tile_d2q9)
        if (!(top + R > j && top < rin - j)) continue;
        const double* up = buf + max(wave - 1, 0) * 6 * TILE_ROW + 1 + lane;
        const double* dn = buf + min(wave + 1, waves - 1) * 6 * TILE_ROW + 1 + lane;
        double m4 = up[0], m7 = up[1 * TILE_ROW - 1], m8 = up[2 * TILE_ROW + 1];
        const double e2 = dn[3 * TILE_ROW], e5 = dn[4 * TILE_ROW + 1], e6 = dn[5 * TILE_ROW - 1];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int n = q < R - 1 ? q + 1 : q;
            double mu[9];
            mu[0] = lam[q][0];
            mu[1] = lane_shift<-1>(lam[q][1]);
            mu[3] = lane_shift<1>(lam[q][3]);
            mu[4] = m4;
            mu[7] = m7;
            mu[8] = m8;
            mu[2] = q < R - 1 ? lam[n][2] : e2;
            mu[5] = q < R - 1 ? lane_shift<-1>(lam[n][5]) : e5;
            mu[6] = q < R - 1 ? lane_shift<1>(lam[n][6]) : e6;
            m4 = lam[q][4];
            m7 = lane_shift<1>(lam[q][7]);
            m8 = lane_shift<-1>(lam[q][8]);
            const Dual2 du = dual_d2q9(mu);
            collide_adjoint_d2q9(du, r, lam[q]);  // as collide_adjoint<2>
            if (owned(q)) {
                double fn[9];
                fn[0] = f[q][0];
                fn[2] = f[q][2];
                fn[4] = f[q][4];
                fn[1] = lane_shift<1>(f[q][1]);
                fn[3] = lane_shift<-1>(f[q][3]);
                fn[5] = lane_shift<1>(f[q][5]);
                fn[6] = lane_shift<-1>(f[q][6]);
                fn[7] = lane_shift<-1>(f[q][7]);
                fn[8] = lane_shift<1>(f[q][8]);
                const double part = eps_part_d2q9(du, fn, r);
                ge += own ? part : 0.0;
            }
            load_f(j + 1, q);
        }
    }
#pragma unroll
    for (int q = 0; q < R; ++q)
        if (owned(q) && own) {
            const MsAddr<true> to((y0 - S + top + q) * g.nx + x);
#pragma unroll
            for (int i = 0; i < 9; ++i) to.store_cached(dst, i, lam[q][i]);
        }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) ge += __shfl_xor(ge, o, 64);
    if (lane == 0) sums[wave] = ge;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < waves; ++w) s += sums[w];
        partials[blockIdx.x] = s;
        for (int i = (int)gridDim.x + (int)blockIdx.x; i < ntab; i += (int)gridDim.x)
            partials[i] = 0.0;
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

// How a run of `nsteps` in passes of up to `limit` goes.
//
// Tiles of kTall rows and more lose to the march in passes of at most four steps, unless
// they save a launch (us a call, tiles and march: 512^2, 23 rows, 2 steps 8.6 and 8.0,
// 4 steps 10.5 and 10.1, but 3 steps 9.7 and 13.5; 700^2 2 steps 13.5 and 11.3, 4 steps
// 16.7 and 13.2; 450^2, 18 rows, 7.2 and 7.5, 9.1 and 9.7).
//
// Passes hand on FORM_MOM, with which a run of three launches and more takes three
// kernels, the first reading FORM_TWIN.  Where a launch takes little more than to fetch
// its kernel, runs of three to five hand on FORM_TWIN, which takes two kernels, and so do
// those of the march (us a call, FORM_MOM and FORM_TWIN: tiles, 17 steps, 256^2 21.7 and
// 20.3, 512^2 42.2 and 36.0, 600^2, 32 rows, 47.1 and 44.4; 650^2, 37 rows, 48.1 and
// 49.3, 40^2 14.9 and 15.3).  So do marches in the
// Infinity Cache of no more rows than the 16 of halo that a wave expands for them, longer
// runs on small grids only (us a call: 16323 x 7, 200 steps 358 and 351; 13000 x 12, 25
// steps 66.9 and 64.3; 40000 x 16, 25 steps 91.2 and 88.2, 200 steps 592 and 609).
TilePlan tile_plan(const Geo& g, int64_t nsteps, int limit) {
    constexpr int kShort = 5, kTall = 20, kTallest = 36;
    constexpr int64_t kSmall = (int64_t)1 << 18;
    TilePlan p{false, pass_form(2, g)};
    if (limit < 2 || nsteps < 2) return p;
    const int rows = tile_rows(g);
    const int log2 = __builtin_ctz((unsigned)limit);
    const int64_t passes = (nsteps + limit - 1) >> log2;
    const int64_t march = (nsteps >> log2) + __builtin_popcount((unsigned)(nsteps & (limit - 1)));
    auto few = [](int64_t launches) { return launches >= 3 && launches <= 5; };
    if (rows == 0) {
        if (g.ny <= 2 * MAX_STEPS_PER_PASS && d2q9_cached_stores(g) &&
            (g.V <= kSmall || few(march)))
            p.form = FORM_TWIN;
        return p;
    }
    p.tiles = rows < kTall || passes * 4 < nsteps || passes < march;
    if (rows >= kShort && rows < kTallest && (!p.tiles || few(passes)))
        p.form = FORM_TWIN;
    return p;
}

// Tile shape of a launch: rows per wave, waves and blocks.
struct TileShape {
    int R, waves, nstrips;
    dim3 grid, block;
    size_t lds;
};
static TileShape tile_shape(const Geo& g, int rows, int nsteps) {
    TileShape s;
    const int w = 64 - 2 * nsteps;
    s.nstrips = (g.nx + w - 1) / w;
    s.R = (rows + 2 * nsteps + TILE_MAX_WAVES - 1) / TILE_MAX_WAVES;
    s.waves = (rows + 2 * nsteps + s.R - 1) / s.R;
    s.grid = dim3((unsigned)(s.nstrips * ((g.ny + rows - 1) / rows)));
    s.block = dim3(64 * s.waves);
    s.lds = (size_t)2 * s.waves * 6 * TILE_ROW * sizeof(double);  // at most 51 KB
    return s;
}

hipError_t launch_tile(int nsteps, const Geo& g, const Rates& r, const double* src, double* dst,
                       hipStream_t st, int in, int out) {
    const int rows = tile_rows(g);
    if (nsteps < 2 || nsteps > MAX_STEPS_PER_PASS || rows == 0) return hipErrorInvalidValue;
    const TileShape s = tile_shape(g, rows, nsteps);
    return dispatch_form(in, [&](auto fi) {
        return dispatch_form(out, [&](auto fo) {
            constexpr int IN = decltype(fi)::value, OUT = decltype(fo)::value;
            switch (s.R) {
#define LBM_TILE(RR)                                                                            \
    case RR:                                                                                    \
        hipLaunchKernelGGL((k_tile_d2q9<RR, IN, OUT>), s.grid, s.block, s.lds, st, src, dst, g, \
                           r, nsteps, rows, s.nstrips);                                         \
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

hipError_t launch_tile_all(int nsteps, const Geo& g, const Rates& r, const double* src,
                           double* out, int64_t stride, hipStream_t st, bool rin) {
    const int rows = tile_rows(g);
    if (nsteps < 1 || nsteps > MAX_STEPS_PER_PASS || rows == 0) return hipErrorInvalidValue;
    const TileShape s = tile_shape(g, rows, nsteps);
    return dispatch_io(rin, false, [&](auto ri, auto) {
        constexpr int IN = decltype(ri)::value ? FORM_TWIN : FORM_FULL;
        switch (s.R) {
#define LBM_TILE(RR)                                                                              \
    case RR:                                                                                      \
        hipLaunchKernelGGL((k_tile_d2q9_all<RR, IN>), s.grid, s.block, s.lds, st, src, out,       \
                           stride, g, r, nsteps, rows, s.nstrips);                                \
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
}

// Tiles where TILE_ADJOINT_ROWS rows a wave hold five steps (us a step of forward and
// backward, march and tiles of up to 8 steps: 40^2 6.60 and 4.04, 256^2 8.15 and 5.92,
// 512^2 15.85 and 12.75, 600^2 19.8 and 16.0). Otherwise the march, in us a segment of m
// steps, march and tiles:
// - one or two steps, and three on short tiles, which take no more launches by single
//   steps (m = 2: 320^2 20.6 and 24.1, 512^2 32.8 and 36.0; m = 3: 256^2 20.1 and 21.3,
//   but 700^2 66.6 and 60.8);
// - passes of two steps, unless the tiles are short (limit 2, m = 45: 400^2, 15 rows, 435
//   and 493; 256^2, 7 rows, 314 and 275; no limit, 720^2, where two steps fit, 803 and 995);
// - long segments of passes of three or four steps on rows of whole 64-byte lines, which
//   the march's strips start on (m = 45: 2000 x 250 780 and 826, 4000 x 120 729 and 752,
//   but 710^2 960 and 864; m = 17: 318 and 305, 297 and 289).
int tile_adjoint_steps(const Geo& g, int limit, int64_t m) {
    constexpr int kShort = 12, kThree = 15, kLong = 20;
    const int rows = tile_rows(g);
    if (rows == 0 || m < (rows < kThree ? 4 : 3)) return 0;
    int fit = MAX_STEPS_PER_PASS;
    while (fit > 1 && tile_shape(g, rows, fit).R > TILE_ADJOINT_ROWS) --fit;
    const int most = std::min(limit, fit);
    if (most < 3) return most == 2 && rows < kShort ? 2 : 0;
    return fit >= 5 || g.nx % 8 != 0 || m <= kLong ? most : 0;
}

int64_t tile_adjoint_table(const Geo& g) {
    const int rows = tile_rows(g);
    return rows == 0 ? 0 : (int64_t)tile_shape(g, rows, MAX_STEPS_PER_PASS).grid.x;
}

hipError_t launch_tile_adjoint(int nsteps, const Geo& g, const Rates& r, const double* lam_in,
                               double* lam_out, const double* ftop, int64_t stride,
                               const double* ckpt, double* partials, int64_t ntab,
                               hipStream_t st) {
    const int rows = tile_rows(g);
    if (nsteps < 1 || nsteps > MAX_STEPS_PER_PASS || rows == 0) return hipErrorInvalidValue;
    const TileShape s = tile_shape(g, rows, nsteps);
    if ((int64_t)s.grid.x > ntab || ntab > (int64_t)INT32_MAX) return hipErrorInvalidValue;
    switch (s.R) {
#define LBM_TILE(RR)                                                                             \
    case RR:                                                                                     \
        hipLaunchKernelGGL((k_tile_adjoint_d2q9<RR>), s.grid, s.block, s.lds, st, lam_in,        \
                           lam_out, ftop, stride, ckpt, partials, (int)ntab, g, r, nsteps, rows, \
                           s.nstrips);                                                           \
        break;
        LBM_TILE(1)
        LBM_TILE(2)
        LBM_TILE(3)
        LBM_TILE(4)
        LBM_TILE(5)
        LBM_TILE(6)
#undef LBM_TILE
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace lbm
