// D3Q19 passes of two steps whose columns keep partial sums.
#include "lbm_device.h"

namespace lbm {
namespace {

// ---------------------------------------------------------------------------
// Two D3Q19 steps per pass over HBM, FORM_MOM to any form.
//
// A block of 12 waves owns a tile of 64 x 12 (x, y) columns, 60 x 8 of them
// outputs, and marches along z; a wave is one row of the tile, a thread one column.
// In iteration k it takes in plane zs - 2 + k (ten values per column, loaded one
// iteration ahead), stage 1 completes the plane behind it and stage 2 the one
// behind that, which is stored.
//
// Exchange: along x by DPP lane shifts, along y through LDS: a row hands out the six
// populations with e_y != 0 that have no twin and reads ten, one column to the side
// where e_x != 0.  Two LDS buffers (one per stage), one barrier each.
//
// Along z a column keeps, per stage, the partial sums (MarchSums) of the plane that
// waits for its e_z = -1 populations and the five e_z = +1 populations for the
// plane after it: 14 doubles where a delay of the populations takes 19.  That
// leaves room for three waves per SIMD (168 registers) and a tile 12 rows high for
// 8 outputs, against 8 for 4 in k_steps_d3q19: a quarter less is computed and
// loaded per output.  What bounds it: at 512^3 memory (21.5 GB algorithmic in
// 4.91 ms, 4.4 TB/s, with a halo of half as much again in the reads); on small grids
// the 2.1 us of a plane: 192 VALU instructions a wave and 32 LDS accesses, two
// barriers.  us a step, 8-row tiles of 13 populations and these of 10 quantities: 512^3
// 3,413 and 2,455, 256^3 444 and 314, 100^3 42.2 and 25 (with these tiles and 13
// planes' strides 512^3 took 2,797).  Two rows per thread (16-row tiles) spilled 41
// registers and took twice the time.
// ---------------------------------------------------------------------------
constexpr int MARCH_WAVES = MARCH3_H + 4;
constexpr int MARCH_LINE = 66;  // a row of 64 doubles in LDS and one to each side

struct MarchSums {
    double xp, xm, yp, ym, zp, Pxy, Pxz, Pyz, T;
    double up[5];  // f_3, f_11, f_12, f_15, f_16 on their way to the next plane
};

// The thirteen populations of a column that have no twin, by their index:
// rest, +x +y +z -x -y -z, xy (+,+) (-,+), xz (+,+) (-,+), yz (+,+) (-,+).
struct MarchPops {
    double f0, px, py, pz, mx, my, mz, xy, yx, xz, zx, yz, zy;
};
__device__ __forceinline__ void march_expand(const Mom3& m, const FoldedRates& r, MarchPops& p) {
    double f[19];
    expand_d3q19(m, r, f);
    p = MarchPops{f[0], f[1], f[2], f[3], f[4], f[5], f[6], f[7], f[8], f[11], f[12], f[15], f[16]};
}

constexpr int MARCH_LINES = 6;
__device__ __forceinline__ void march_publish(const MarchPops& p, double* line) {
    line[0 * MARCH_LINE] = p.py;  // f_2
    line[1 * MARCH_LINE] = p.my;  // f_5
    line[2 * MARCH_LINE] = p.xy;  // f_7 and f_9
    line[3 * MARCH_LINE] = p.yx;  // f_8 and f_10
    line[4 * MARCH_LINE] = p.yz;  // f_15 and f_17
    line[5 * MARCH_LINE] = p.zy;  // f_16 and f_18
}

// What a row pulls from its y neighbours.
struct MarchPull {
    double f2, f7, f8, f15, f18;   // from row y - 1
    double f5, f9, f10, f16, f17;  // from row y + 1
};

// Streams one plane of one row into its sums and gives the quantities of the plane
// that it completes.
__device__ __forceinline__ void march_plane(MarchSums& s, const MarchPops& p, const MarchPull& q,
                                            const FoldedRates& r, Mom3& m) {
    // e_z = -1: completes the plane behind
    const double f13 = lane_shift<-1>(p.xz), f14 = lane_shift<1>(p.zx);
    const double xp = s.xp + f14, xm = s.xm + f13, yp = s.yp + q.f18, ym = s.ym + q.f17;
    const double zm = (p.mz + f13) + (f14 + q.f17) + q.f18;
    const double Px = xp + xm, Py = yp + ym, Pz = s.zp + zm;
    m.jx = xp - xm;
    m.jy = yp - ym;
    m.jz = s.zp - zm;
    m.th = (s.T + (p.mz + (q.f17 + q.f18))) + Px;
    m.Pxy = s.Pxy;
    m.Pxz = s.Pxz + (f13 - f14);
    m.Pyz = s.Pyz + (q.f17 - q.f18);
    const double tt = r.ct * m.th;
    m.hPx = fma(r.cp, Px, tt);
    m.hPy = fma(r.cp, Py, tt);
    m.hPz = fma(r.cp, Pz, tt);
    // e_z = 0 and, from the plane before, e_z = +1: the sums of this plane
    const double f1 = lane_shift<1>(p.px), f4 = lane_shift<-1>(p.mx);
    const double f3 = s.up[0], f11 = s.up[1], f12 = s.up[2], f15 = s.up[3], f16 = s.up[4];
    s.xp = (f1 + q.f7) + (q.f10 + f11);
    s.xm = (f4 + q.f8) + (q.f9 + f12);
    s.yp = (q.f2 + q.f7) + (q.f8 + f15);
    s.ym = (q.f5 + q.f9) + (q.f10 + f16);
    s.zp = (f3 + f11) + (f12 + f15) + f16;
    s.Pxy = (q.f7 + q.f9) - (q.f8 + q.f10);
    s.Pxz = f11 - f12;
    s.Pyz = f15 - f16;
    s.T = (p.f0 + (q.f2 + q.f5)) + (f3 + (f15 + f16));
    // e_z = +1: for the next plane
    s.up[0] = p.pz;
    s.up[1] = lane_shift<1>(p.xz);
    s.up[2] = lane_shift<-1>(p.zx);
    s.up[3] = q.f15;
    s.up[4] = q.f16;
}

// One stage of a row; up / dn: the lines of the rows y - 1 and y + 1 at this lane.
__device__ __forceinline__ void march_stage(MarchSums& s, const MarchPops& p, const double* up,
                                            const double* dn, const FoldedRates& r, Mom3& m) {
    MarchPull q;
    q.f2 = up[0 * MARCH_LINE];
    q.f7 = up[2 * MARCH_LINE - 1];
    q.f8 = up[3 * MARCH_LINE + 1];
    q.f15 = up[4 * MARCH_LINE];
    q.f18 = up[5 * MARCH_LINE];
    q.f5 = dn[1 * MARCH_LINE];
    q.f9 = dn[2 * MARCH_LINE + 1];
    q.f10 = dn[3 * MARCH_LINE - 1];
    q.f16 = dn[5 * MARCH_LINE];
    q.f17 = dn[4 * MARCH_LINE];
    march_plane(s, p, q, r, m);
}

// One z-plane of a chunked D3Q19 buffer as a buffer resource, and the byte offset of
// population 0 of a node of it.
template <int Q>
struct MarchPlane {
    __amdgpu_buffer_rsrc_t rs;
    int64_t n0, c0;
    __device__ __forceinline__ MarchPlane(const double* buf, int64_t plane, int z) {
        n0 = (int64_t)z * plane;
        c0 = n0 >> LOG2_CHUNK;
        const int64_t c1 = (n0 + plane - 1) >> LOG2_CHUNK;
        rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(buf) + c0 * Q * CHUNK, (short)0,
                                               (int)((c1 - c0 + 1) * Q * CHUNK * 8), 0x00020000);
    }
    __device__ __forceinline__ unsigned offset(int col) const {
        const int kk = (int)(n0 - (c0 << LOG2_CHUNK)) + col;  // node within the plane's chunks
        return (unsigned)(((kk >> LOG2_CHUNK) * Q * (int)CHUNK + (kk & ((int)CHUNK - 1))) * 8);
    }
};
typedef unsigned int MarchU2 __attribute__((__vector_size__(8)));  // a double as buffer data

template <int OUT>
__global__ void __launch_bounds__(64 * MARCH_WAVES)
k_march_d3q19(const double* __restrict__ src, double* __restrict__ dst, Geo g, Rates rates, int lz,
              int ntx, int nty) {
    __shared__ double lds[2 * MARCH_WAVES * MARCH_LINES * MARCH_LINE];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const unsigned t = xcd_remap(blockIdx.x, gridDim.x);
    const unsigned ntile = (unsigned)ntx * (unsigned)nty;
    const int tile = (int)(t % ntile), seg = (int)(t / ntile);
    const int x0 = (tile % ntx) * MARCH3_W, y0 = (tile / ntx) * MARCH3_H;
    const int zs = seg * lz, ze = min(zs + lz, g.nz);
    const int64_t plane = (int64_t)g.nx * g.ny;
    const FoldedRates r = folded(rates);
    const int gx = wrapi(x0 - 2 + lane, g.nx);
    const int col = wrapi(y0 - 2 + wave, g.ny) * g.nx + gx;
    double* line = lds + wave * MARCH_LINES * MARCH_LINE + 1 + lane;
    // (the outermost waves read their own lines: any value, it stays in the halo)
    const double* up = lds + max(wave - 1, 0) * MARCH_LINES * MARCH_LINE + 1 + lane;
    const double* dn = lds + min(wave + 1, MARCH_WAVES - 1) * MARCH_LINES * MARCH_LINE + 1 + lane;
    constexpr int BUF = MARCH_WAVES * MARCH_LINES * MARCH_LINE;
    const int x = x0 - 2 + lane, y = y0 - 2 + wave;
    const bool own = wave >= 2 && wave < MARCH_WAVES - 2 && y < g.ny && lane >= 2 && lane < 62 &&
                     x < g.nx;
    const bool edge = wave == 0 || wave == MARCH_WAVES - 1;
    Mom3 pre;
    // The first and the last row of the tile only pass on their populations with
    // e_y = +1 and -1, which need theta, j_y, hP_y, P_xy and P_yz: the other five
    // planes get an out-of-range offset, which reads nothing.
    auto load = [&](int z) {
        const MarchPlane<form_planes<3>(FORM_MOM)> pl(src, plane, wrapi(z, g.nz));
        const unsigned off = pl.offset(col), trim = edge ? 0x80000000u : off;
        auto get = [&](unsigned o, int i) {
            return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(
                                                  pl.rs, o, i * (int)CHUNK * 8, 0));
        };
        pre.th = get(off, 0);
        pre.jy = get(off, 2);
        pre.hPy = get(off, 5);
        pre.Pxy = get(off, 7);
        pre.Pyz = get(off, 9);
        pre.jx = get(trim, 1);
        pre.jz = get(trim, 3);
        pre.hPx = get(trim, 4);
        pre.hPz = get(trim, 6);
        pre.Pxz = get(trim, 8);
    };
    load(zs - 2);
    // waited for here, so that the loop is entered with no load in flight and its
    // own waits can leave the stores of the iteration before in flight
    asm volatile("" : "+v"(pre.th), "+v"(pre.jx), "+v"(pre.jy), "+v"(pre.jz), "+v"(pre.hPx));
    asm volatile("" : "+v"(pre.hPy), "+v"(pre.hPz), "+v"(pre.Pxy), "+v"(pre.Pxz), "+v"(pre.Pyz));
    MarchSums s1 = MarchSums{0, 0, 0, 0, 0, 0, 0, 0, 0, {0, 0, 0, 0, 0}}, s2 = s1;
    // stage j holds valid planes from iteration 2j on; before that it works on
    // zeros and nothing is stored
    const int kend = ze - zs + 3;
    auto march = [&](auto stores) {
        for (int k = 0; k <= kend; ++k) {
            MarchPops p;
            march_expand(pre, r, p);
            load(zs - 1 + k);  // unused in the last iteration (in bounds: wrapped)
            march_publish(p, line);
            __syncthreads();
            Mom3 m;
            march_stage(s1, p, up, dn, r, m);
            march_expand(m, r, p);
            march_publish(p, line + BUF);
            __syncthreads();
            march_stage(s2, p, up + BUF, dn + BUF, r, m);
            if constexpr (decltype(stores)::value) {
                const MarchPlane<form_planes<3>(OUT)> pl(dst, plane, max(zs + k - 4, zs));
                const unsigned off = own && k >= 4 ? pl.offset(y * g.nx + x) : 0x80000000u;
                auto put = [&](int i, double v) {
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(MarchU2, v), pl.rs,
                                                          off, i * (int)CHUNK * 8, 2);
                };
                if constexpr (OUT == FORM_MOM) {
                    put(0, m.th);
                    put(1, m.jx);
                    put(2, m.jy);
                    put(3, m.jz);
                    put(4, m.hPx);
                    put(5, m.hPy);
                    put(6, m.hPz);
                    put(7, m.Pxy);
                    put(8, m.Pxz);
                    put(9, m.Pyz);
                } else {
                    double f[19];
                    expand_d3q19(m, r, f);
#pragma unroll
                    for (int i = 0; i < 19; ++i)
                        if (form_holds<3>(OUT, i)) put(i, f[i]);
                }
            }
        }
    };
    // The rows that own outputs and the halo rows run loops of their own, and lanes
    // that own none, and every lane while the pipeline fills, store to an
    // out-of-range offset, which writes nothing: behind a branch in the loop the
    // memory counter has to serve both of its sides, and every iteration waits for
    // its own stores.
    if (wave >= 2 && wave < MARCH_WAVES - 2)
        march(std::true_type{});
    else
        march(std::false_type{});
}

}  // namespace

hipError_t launch_march3(const Geo& g, const Rates& r, const double* src, double* dst,
                         hipStream_t st, int lz, int out) {
    const int ntx = (g.nx + MARCH3_W - 1) / MARCH3_W, nty = (g.ny + MARCH3_H - 1) / MARCH3_H;
    const int64_t nb = (int64_t)ntx * nty * ((g.nz + lz - 1) / lz);
    if (nb > (int64_t)UINT32_MAX) return hipErrorInvalidValue;
    return dispatch_form(out, [&](auto fo) {
        hipLaunchKernelGGL((k_march_d3q19<decltype(fo)::value>), dim3((unsigned)nb),
                           dim3(64 * MARCH_WAVES), 0, st, src, dst, g, r, lz, ntx, nty);
        return hipGetLastError();
    });
}

}  // namespace lbm
