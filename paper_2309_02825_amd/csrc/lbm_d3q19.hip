// D3Q19 passes of two steps.
#include <algorithm>
#include <cmath>

#include "lbm_device.h"

namespace lbm {
namespace {

// ---------------------------------------------------------------------------
// S D3Q19 time steps per pass over HBM.
//
// The 2-D scheme above one dimension up: a block of MS3_TX x MS3_TY threads
// owns a tile of (MS3_TX - 2S) x (MS3_TY - 2S) output columns (x, y) plus an
// S-wide halo, thread (tx, ty) owns one column in every stage, and the block
// marches along z through a segment of planes.  A row of the tile (fixed y)
// is one wave, lane tx = column x: the ten populations with e_x != 0 are
// pulled from lane tx - e_x by DPP lane shifts, as in the D2Q9 passes; the
// ten with e_y != 0 (the xy edges after their x shift) then go through LDS
// to row ty + e_y; the three with e_x = e_y = 0 stay in their thread.  Planes
// are delayed in registers by e_z (0, 1 or 2 iterations).  Register pressure
// limits S to 2 (190 VGPRs when only the 13 independent populations are
// loaded, 217 otherwise; two waves per SIMD, so one 512-thread block per
// CU); each block uses 2 x 10 x 512 doubles of LDS.
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int m3_ex(int i) { return Lat<3>::E[i][0]; }
__host__ __device__ constexpr int m3_ey(int i) { return Lat<3>::E[i][1]; }
__host__ __device__ constexpr int m3_ez(int i) { return Lat<3>::E[i][2]; }
// index of population i among those with its e_z
__host__ __device__ constexpr int m3_zslot(int i) {
    int s = 0;
    for (int j = 0; j < i; ++j) s += m3_ez(j) == m3_ez(i);
    return s;
}
constexpr int M3_Z0 = 9, M3_ZP = 5;  // populations with e_z = 0 and with e_z = +1
constexpr int M3_THREADS = MS3_TX * MS3_TY;
static_assert(MS3_TX == 64, "a tile row of the D3Q19 pass is one wave (DPP lane shifts along x)");

template <int S>
struct Ms3State {
    double pre[19];            // next input plane (prefetched)
    double z[S][M3_Z0];        // e_z = 0 populations of the previous plane, per stage input
    double u[2][S][M3_ZP];     // e_z = +1 populations of the planes of each parity
};

// y-movers (e_y != 0): the 10 populations exchanged through LDS
__host__ __device__ constexpr bool m3_ymover(int i) { return m3_ey(i) != 0; }
__host__ __device__ constexpr int m3_yslot(int i) {
    int s = 0;
    for (int j = 0; j < i; ++j) s += m3_ymover(j);
    return s;
}
constexpr int M3_YMOVERS = m3_yslot(19);
static_assert(M3_YMOVERS == 10, "D3Q19 has 10 populations with e_y != 0");

// Whether plane i of a post-collision state (population i, or its twin)
// holds a population with e_y = ey.
__host__ __device__ constexpr bool m3_plane_holds(int i, int ey) {
    for (int p = 0; p < 19; ++p)
        if (twin<3>(p) == i && m3_ey(p) == ey) return true;
    return false;
}
__host__ __device__ constexpr int m3_planes_holding(int ey) {
    int n = 0;
    for (int i = 0; i < 19; ++i) n += twin<3>(i) == i && m3_plane_holds(i, ey);
    return n;
}
static_assert(m3_planes_holding(1) == 5 && m3_planes_holding(-1) == 5,
              "an edge row of the tile passes on 5 of the 13 independent planes");

// With only the 13 independent populations, one input plane (z-plane zp) of
// the column col through a buffer resource over that z-plane's chunks
// (32-bit offsets).  The first tile row passes on only its populations with
// e_y = +1 and the last only those with e_y = -1; the planes they do not
// need get an out-of-range offset, so the hardware drops those loads (no
// memory access, the register reads 0) and every wave still issues the same
// instructions: the two edge rows fetch 5 of the 13 planes.
__device__ __forceinline__ void m3_load_plane(double (&pre)[19], const double* src,
                                              int64_t plane, int zp, int col, int ty) {
    const int64_t n0 = (int64_t)zp * plane;
    const int64_t c0 = n0 >> 12, c1 = (n0 + plane - 1) >> 12;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<double*>(src) + c0 * 19 * 4096, (short)0,
        (int)((c1 - c0 + 1) * 19 * 4096 * 8), 0x00020000);
    const int64_t kk = n0 + col;
    const unsigned base = (unsigned)((((kk >> 12) - c0) * 19 * 4096 + (kk & 4095)) * 8);
#pragma unroll
    for (int i = 0; i < 19; ++i)
        if (form_holds<3>(FORM_TWIN, i)) {
            const bool need = (ty != 0 || m3_plane_holds(i, 1)) &&
                              (ty != MS3_TY - 1 || m3_plane_holds(i, -1));
            const unsigned off = need ? base + (unsigned)(i * 4096 * 8) : 0x80000000u;
            pre[i] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0));
        }
}

// The planes of FORM_MOM.
__device__ __forceinline__ void m3_planes(const Mom3& m, double (&p)[19]) {
    p[0] = m.th;
    p[1] = m.jx;
    p[2] = m.jy;
    p[3] = m.jz;
    p[4] = m.hPx;
    p[5] = m.hPy;
    p[6] = m.hPz;
    p[7] = m.Pxy;
    p[8] = m.Pxz;
    p[9] = m.Pyz;
}

// One iteration k of the march.  x shift by DPP (pull from lane tx - e_x), then y shift
// through LDS.  BUF: the input planes come through m3_load_plane (FORM_TWIN only).
template <int S, int P, int IN, int OUT, bool BUF = false>
__device__ __forceinline__ void ms3_plane(Ms3State<S>& st, double* lds, int k,
                                          const double* __restrict__ src, double* __restrict__ dst,
                                          const Geo& g, int col, int zs, int x0, int y0,
                                          const FoldedRates& r) {
    static_assert(IN != FORM_MOM && (!BUF || IN == FORM_TWIN), "buffer loads serve the reduced state only");
    // a tile row is one wave: ty is uniform across it, and saying so lets the
    // per-row choices (edge-row loads, y exchange) compile to scalar selects
    // and branches instead of lane-masked ones
    const int tid = threadIdx.x, tx = tid % MS3_TX;
    const int ty = __builtin_amdgcn_readfirstlane(tid / MS3_TX);
    const int64_t plane = (int64_t)g.nx * g.ny;
    double f[19];
#pragma unroll
    for (int i = 0; i < 19; ++i) f[i] = st.pre[IN == FORM_TWIN ? twin<3>(i) : i];
    if constexpr (BUF) {
        m3_load_plane(st.pre, src, plane, wrapi(zs - S + k + 1, g.nz), col, ty);
    } else {
        const int64_t base = (int64_t)wrapi(zs - S + k + 1, g.nz) * plane + col;
#pragma unroll
        for (int i = 0; i < 19; ++i)
            if (form_holds<3>(IN, i)) st.pre[i] = src[slot<19>(i, base)];
    }
    // pull along x (every lane takes part; the edge lanes receive zeros,
    // which reach only halo columns, never a stored output)
#pragma unroll
    for (int i = 0; i < 19; ++i)
        if (m3_ex(i) != 0) f[i] = m3_ex(i) == 1 ? lane_shift<1>(f[i]) : lane_shift<-1>(f[i]);
#pragma unroll
    for (int i = 0; i < 19; ++i)
        if (m3_ymover(i)) {
            const int cy = ty + m3_ey(i);
            if (cy >= 0 && cy < MS3_TY) lds[m3_yslot(i) * M3_THREADS + cy * MS3_TX + tx] = f[i];
        }
    __syncthreads();
#pragma unroll
    for (int j = 1; j <= S; ++j) {
        double in[19];
        const double* rd = lds + ((j - 1) & 1) * M3_YMOVERS * M3_THREADS;
#pragma unroll
        for (int i = 0; i < 19; ++i) {
            const double v = m3_ymover(i) ? rd[m3_yslot(i) * M3_THREADS + tid] : f[i];
            if (m3_ez(i) == -1) {
                in[i] = v;
            } else if (m3_ez(i) == 0) {
                in[i] = st.z[j - 1][m3_zslot(i)];
                st.z[j - 1][m3_zslot(i)] = v;
            } else {
                in[i] = st.u[P][j - 1][m3_zslot(i)];
                st.u[P][j - 1][m3_zslot(i)] = v;
            }
        }
        if (k >= 2 * j) {
            Mom3 mom;
            moments_d3q19(in, r, mom);
            if (j < S || OUT != FORM_MOM)
                expand_d3q19(mom, r, in);
            else
                m3_planes(mom, in);
            if (j < S) {
                double* wr = lds + (j & 1) * M3_YMOVERS * M3_THREADS;
#pragma unroll
                for (int i = 0; i < 19; ++i) {
                    double v = in[i];
                    if (m3_ex(i) != 0) v = m3_ex(i) == 1 ? lane_shift<1>(v) : lane_shift<-1>(v);
                    f[i] = v;
                    if (m3_ymover(i)) {
                        const int cy = ty + m3_ey(i);
                        if (cy >= 0 && cy < MS3_TY) wr[m3_yslot(i) * M3_THREADS + cy * MS3_TX + tx] = v;
                    }
                }
            } else if (tx >= S && tx < MS3_TX - S && ty >= S && ty < MS3_TY - S &&
                       x0 - S + tx < g.nx && y0 - S + ty < g.ny) {
                const int64_t kk = (int64_t)wrapi(zs - 2 * S + k, g.nz) * plane +
                                   (int64_t)(y0 - S + ty) * g.nx + (x0 - S + tx);
#pragma unroll
                for (int i = 0; i < 19; ++i)
                    if (form_holds<3>(OUT, i))
                        __builtin_nontemporal_store(in[i], dst + slot<form_planes<3>(OUT)>(i, kk));
            }
        }
        if (j < S) __syncthreads();
    }
    if (S & 1) __syncthreads();
}

template <int S, int IN, int OUT, bool BUF>
__global__ void __launch_bounds__(M3_THREADS) k_steps_d3q19(const double* __restrict__ src,
                                                            double* __restrict__ dst, Geo g,
                                                            Rates r, int lz, int ntx, int nty) {
    __shared__ double lds[2 * M3_YMOVERS * M3_THREADS];
    const unsigned t = xcd_remap(blockIdx.x, gridDim.x);
    const unsigned ntile = (unsigned)ntx * (unsigned)nty;
    const int tile = (int)(t % ntile), seg = (int)(t / ntile);
    const int x0 = (tile % ntx) * tile_width3(S), y0 = (tile / ntx) * tile_height3(S);
    const int zs = seg * lz, ze = min(zs + lz, g.nz);
    const int tx = threadIdx.x % MS3_TX;
    const int ty = __builtin_amdgcn_readfirstlane((int)threadIdx.x / MS3_TX);
    const int col = wrapi(y0 - S + ty, g.ny) * g.nx + wrapi(x0 - S + tx, g.nx);
    const int kend = ze - zs + 2 * S - 1;
    const FoldedRates fr = folded(r);
    Ms3State<S> st;
    {
        const int64_t base = (int64_t)wrapi(zs - S, g.nz) * g.nx * g.ny + col;
#pragma unroll
        for (int i = 0; i < 19; ++i)
            if (form_holds<3>(IN, i)) st.pre[i] = src[slot<19>(i, base)];
    }
#pragma unroll
    for (int j = 0; j < S; ++j) {
#pragma unroll
        for (int a = 0; a < M3_Z0; ++a) st.z[j][a] = 0.0;
#pragma unroll
        for (int a = 0; a < M3_ZP; ++a) st.u[0][j][a] = st.u[1][j][a] = 0.0;
    }
    // plane pairs in the loop, a last odd plane after it (as in ms_tile)
    int k = 0;
    for (; k + 1 <= kend; k += 2) {
        ms3_plane<S, 0, IN, OUT, BUF>(st, lds, k, src, dst, g, col, zs, x0, y0, fr);
        ms3_plane<S, 1, IN, OUT, BUF>(st, lds, k + 1, src, dst, g, col, zs, x0, y0, fr);
    }
    if (k <= kend) ms3_plane<S, 0, IN, OUT, BUF>(st, lds, k, src, dst, g, col, zs, x0, y0, fr);
}

}  // namespace

// Planes per segment of a D3Q19 pass over `tiles` (x, y) tiles: a block marches its
// planes one after the other, four more than it stores, and the chip runs one block
// per CU at a time, so the cost of a choice is rounds x (planes + 4), with whole
// rounds while there are few.  At most 64 planes (512^3, with planes 19 apart: 64 planes
// 2,797 us a step, 128 2,829).  100^3, 12 planes (one round) against the 16 of a rule
// without rounds: 24.7 and 30.1 us a step.
static int segment_planes(int nz, int64_t tiles, double* plane_rounds = nullptr) {
    const int cus = compute_units();
    int best = nz;
    double best_cost = 1e300;
    for (int nseg = (nz + 63) / 64; nseg <= nz; ++nseg) {
        const int lz = (nz + nseg - 1) / nseg;
        if (nseg > 1 && lz < 4) break;
        double rounds = (double)(tiles * ((nz + lz - 1) / lz)) / cus;
        if (rounds < 8.0) rounds = std::ceil(rounds);
        const double cost = rounds * (lz + 4);
        if (cost < best_cost * 0.999) {
            best_cost = cost;
            best = lz;
        }
    }
    if (plane_rounds) *plane_rounds = best_cost;
    return best;
}

bool march3_fits(const Geo& g) {
    // buffer addressing needs the chunks of one z-plane under 2 GiB (planes up to
    // about 14 M nodes)
    return ((int64_t)g.nx * g.ny / CHUNK + 2) * 19 * CHUNK * 8 < ((int64_t)1 << 31);
}

template <int S>
static hipError_t launch_steps3_t(const Geo& g, const Rates& r, const double* src, double* dst,
                                  hipStream_t st, int in, int out, int lz) {
    const int ntx = (g.nx + tile_width3(S) - 1) / tile_width3(S);
    const int nty = (g.ny + tile_height3(S) - 1) / tile_height3(S);
    const int64_t nseg = (g.nz + lz - 1) / lz;  // every segment non-empty
    const int64_t nb = (int64_t)ntx * nty * nseg;
    if (nb > (int64_t)UINT32_MAX) return hipErrorInvalidValue;
    const bool buf = march3_fits(g);
    const dim3 grid((unsigned)nb), block(M3_THREADS);
    return dispatch_form(out, [&](auto fo) {
        constexpr int OUT = decltype(fo)::value;
        if (in == FORM_FULL)
            hipLaunchKernelGGL((k_steps_d3q19<S, FORM_FULL, OUT, false>), grid, block, 0, st, src,
                               dst, g, r, lz, ntx, nty);
        else if (buf)
            hipLaunchKernelGGL((k_steps_d3q19<S, FORM_TWIN, OUT, true>), grid, block, 0, st, src,
                               dst, g, r, lz, ntx, nty);
        else
            hipLaunchKernelGGL((k_steps_d3q19<S, FORM_TWIN, OUT, false>), grid, block, 0, st, src,
                               dst, g, r, lz, ntx, nty);
        return hipGetLastError();
    });
}

static int64_t march3_tiles(const Geo& g) {
    return (int64_t)((g.nx + MARCH3_W - 1) / MARCH3_W) * ((g.ny + MARCH3_H - 1) / MARCH3_H);
}

// Two steps: from FORM_MOM on the taller tiles of k_march_d3q19; from 19 or 13 planes,
// the first launch of a call and every one where passes hand on FORM_TWIN (plan3), on the
// 8-row tiles.
hipError_t launch_steps3(int nsteps, const Geo& g, const Rates& r, const double* src, double* dst,
                         hipStream_t st, int in, int out, const Plan3& plan) {
    if (g.nw != 1 || nsteps != 2 || plan.lz_first < 1 || plan.lz < 1) return hipErrorInvalidValue;
    if (in == FORM_MOM) {
        if (!march3_fits(g)) return hipErrorInvalidValue;  // pass_form
        return launch_march3(g, r, src, dst, st, plan.lz, out);
    }
    return launch_steps3_t<2>(g, r, src, dst, st, in, out, plan.lz_first);
}

// How a run goes, by an estimate in us of two steps.  A pass takes 4 and 2.1 for a plane
// of the march (a block alone on its CU), or 2.3 for a plane of the 8-row tiles and 1 for
// the ends of segments.  Those are faster where they march no more planes, on few planes
// and on rows of columns, while what they move (FORM_TWIN) stays in the Infinity Cache (us
// for 24 steps, 8-row tiles and march: 322 x 154 x 4 224 and 250, 303 x 154 x 3 185 and
// 221; 337 x 185 x 4, two rounds of 8-row tiles, 408 and 269; 1000 x 4 x 1000, beyond the
// cache, 2,647 and 2,479).  Two single steps take 7, one for 42 thousand nodes and one for
// 40 thousand threads of their launch grids, at least one for 480 blocks, and beyond the
// cache one for 10 thousand nodes (two steps, single and in passes: 40^3 9.9 and 20.9,
// 64^3 19.5 and 21.6, 72^3 28.8 and 26.4, 2 x 76 x 232 37.6 and 33.3, 1 x 1 x 65535 123
// and 481).
Plan3 plan3(const Geo& g) {
    const int64_t first = (int64_t)((g.nx + tile_width3(2) - 1) / tile_width3(2)) *
                          ((g.ny + tile_height3(2) - 1) / tile_height3(2));
    const bool cached = states_fit_cache(3, g);
    Plan3 p;
    double planes_first, planes;
    p.lz_first = segment_planes(g.nz, first, &planes_first);
    p.lz = segment_planes(g.nz, march3_tiles(g), &planes);
    p.form = cached && planes_first <= planes ? (int)FORM_TWIN : pass_form(3, g);
    const double pass = p.form == FORM_TWIN ? 2.3 * planes_first + (p.lz_first < g.nz)
                                            : 4.0 + 2.1 * planes;
    const double blocks = (double)launch_shape(3, g).nblocks;
    double single = std::max(7.0 + (double)g.V / 42000.0 + blocks * 256.0 / 40000.0,
                             blocks / 480.0);
    if (!cached) single = std::max(single, (double)g.V / 10000.0);
    p.passes = pass < single;
    return p;
}

}  // namespace lbm
