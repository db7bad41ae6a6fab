// Device helpers shared by the kernel sources: node and neighbour indexing, the
// XCD-aware tile order, lane shifts and block reductions.
#pragma once

#include <type_traits>

#include "lbm_kernels.h"

namespace lbm {
namespace {

constexpr int BX = BLOCK_X;
constexpr int BY = BLOCK_Y;
constexpr int B1 = BLOCK_1D;

// Offsets of the neighbour x - e (e = -1, 0, +1) along each axis, periodic:
// s[a][e + 1] = ((x_a - e) mod n_a) * (stride of axis a in the node index).
struct Nbr {
    int s[4][3];
};

template <int D>
__device__ __forceinline__ Nbr make_nbr(const int (&c)[4], const Geo& g) {
    Nbr nb;
    const int n[4] = {g.nx, g.ny, g.nz, g.nw};
    int stride = 1;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        if (a < D) {
            const int m = c[a] == 0 ? n[a] - 1 : c[a] - 1;
            const int p = c[a] == n[a] - 1 ? 0 : c[a] + 1;
            nb.s[a][0] = p * stride;
            nb.s[a][1] = c[a] * stride;
            nb.s[a][2] = m * stride;
            stride *= n[a];
        } else {
            nb.s[a][0] = nb.s[a][1] = nb.s[a][2] = 0;
        }
    }
    return nb;
}

// Node index of x - e_i (pull source) and x + e_i (push target).
template <int D>
__device__ __forceinline__ int pull_index(const Nbr& nb, int i) {
    int k = 0;
#pragma unroll
    for (int a = 0; a < D; ++a) k += nb.s[a][Lat<D>::E[i][a] + 1];
    return k;
}
template <int D>
__device__ __forceinline__ int push_index(const Nbr& nb, int i) {
    int k = 0;
#pragma unroll
    for (int a = 0; a < D; ++a) k += nb.s[a][1 - Lat<D>::E[i][a]];
    return k;
}

__device__ __forceinline__ int64_t block_linear() {
    return (int64_t)blockIdx.x + (int64_t)gridDim.x * ((int64_t)blockIdx.y + (int64_t)gridDim.y * blockIdx.z);
}

// Workgroups are dispatched round-robin over the 8 XCDs of the chip (linear
// block b runs on XCD b mod 8), each with its own L2.  Neighbouring tiles
// along x share the cache lines of the x +- 1 halo, so every XCD is given one
// contiguous range of tiles (x fastest) instead of every eighth tile.
constexpr unsigned NXCD = 8;
__device__ __forceinline__ unsigned xcd_remap(unsigned b, unsigned nb) {
    const unsigned q = nb / NXCD, r = nb % NXCD;
    const unsigned c = b % NXCD, slot = b / NXCD;
    return c * q + (c < r ? c : r) + slot;
}

template <int D>
__device__ __forceinline__ bool thread_node(const Geo& g, int (&c)[4]) {
    const unsigned nb = gridDim.x * gridDim.y * gridDim.z;
    const unsigned b = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    const unsigned t = xcd_remap(b, nb);
    const unsigned tx = t % gridDim.x;
    const unsigned rest = t / gridDim.x;
    c[2] = c[3] = 0;
    if constexpr (D == 1) {
        c[0] = (int)(tx * B1 + threadIdx.x);
        c[1] = 0;
    } else {
        c[0] = (int)(tx * blockDim.x + threadIdx.x);
        c[1] = (int)((rest % gridDim.y) * blockDim.y + threadIdx.y);
        if constexpr (D >= 3) {
            const unsigned zw = rest / gridDim.y;  // grid.z runs over n_z * n_w
            if (D == 4 && (g.nz & 7) == 0 && (g.nw & 7) == 0) {
                // (z, w) planes in 8 x 8 patches, so that the blocks running
                // at the same time (about 64 planes of 64 x 64 nodes) hold
                // both the z and the w neighbours of most of their nodes in
                // L2: a twin is pulled from its partner's plane at the node
                // the partner's own pull does not read (64^4: +6 %)
                const unsigned p = zw >> 6, q = zw & 63, npz = (unsigned)g.nz >> 3;
                c[2] = (int)((p % npz) * 8 + (q & 7));
                c[3] = (int)((p / npz) * 8 + (q >> 3));
            } else {
                c[2] = (int)(zw % (unsigned)g.nz);
                c[3] = (int)(zw / (unsigned)g.nz);
            }
        }
    }
    return c[0] < g.nx && c[1] < g.ny;
}

__device__ __forceinline__ int node_index(const Geo& g, const int (&c)[4]) {
    return ((c[3] * g.nz + c[2]) * g.ny + c[1]) * g.nx + c[0];
}

// Deterministic sum over the 256 threads of a block; result valid in thread 0.
__device__ __forceinline__ double block_sum(double v) {
    __shared__ double sh[4];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    const int tid = threadIdx.x + threadIdx.y * blockDim.x;
    if ((tid & 63) == 0) sh[tid >> 6] = v;
    __syncthreads();
    return tid == 0 ? (sh[0] + sh[1]) + (sh[2] + sh[3]) : 0.0;
}

__device__ __forceinline__ int wrapi(int v, int n) {
    v %= n;
    return v < 0 ? v + n : v;
}

__host__ __device__ constexpr int ms_ex(int i) { return Lat<2>::E[i][0]; }
__host__ __device__ constexpr int ms_ey(int i) { return Lat<2>::E[i][1]; }
// index of population i among those with the same e_y
__host__ __device__ constexpr int ms_yslot(int i) {
    int s = 0;
    for (int j = 0; j < i; ++j) s += ms_ey(j) == ms_ey(i);
    return s;
}

// value of a double in the lane on the left (DIR = +1) or right (DIR = -1)
template <int DIR>
__device__ __forceinline__ double lane_shift(double x) {
    constexpr int ctrl = DIR == 1 ? 0x138 : 0x130;  // wave_shr:1 : wave_shl:1
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xffffffff), ctrl, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), ctrl, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// value of a double in the lane on the left (DIR = +1) or right (DIR = -1),
// rotating around the wave (lane 0 takes lane 63 and vice versa)
template <int DIR>
__device__ __forceinline__ double lane_rotate(double x) {
    constexpr int ctrl = DIR == 1 ? 0x13C : 0x134;  // wave_ror:1 : wave_rol:1
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xffffffff), ctrl, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), ctrl, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

template <typename F>
hipError_t dispatch(int d, F&& f) {
    switch (d) {
        case 1: return f(std::integral_constant<int, 1>{});
        case 2: return f(std::integral_constant<int, 2>{});
        case 3: return f(std::integral_constant<int, 3>{});
        case 4: return f(std::integral_constant<int, 4>{});
        default: return hipErrorInvalidValue;
    }
}

// (rin, wout) as template arguments of a kernel.
template <typename F>
hipError_t dispatch_io(bool rin, bool wout, F&& f) {
    if (rin)
        return wout ? f(std::true_type{}, std::true_type{}) : f(std::true_type{}, std::false_type{});
    return wout ? f(std::false_type{}, std::true_type{}) : f(std::false_type{}, std::false_type{});
}

// A buffer form (FORM_*) as a template argument.
template <typename F>
hipError_t dispatch_form(int form, F&& f) {
    switch (form) {
        case FORM_FULL: return f(std::integral_constant<int, FORM_FULL>{});
        case FORM_TWIN: return f(std::integral_constant<int, FORM_TWIN>{});
        case FORM_MOM: return f(std::integral_constant<int, FORM_MOM>{});
        default: return hipErrorInvalidValue;
    }
}

}  // namespace
}  // namespace lbm
