// Block sizes, tiles, node indices and the workgroup sum shared by the device
// kernels.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace dgmg {

constexpr int kWG = 256;

__device__ __forceinline__ int xcd_tile(int bid, int nblk) {
    // bijective remap of [0, nblk): XCD x = bid % 8 gets tiles [x*q + min(x,r), ...)
    const int x = bid & 7, k = bid >> 3;
    const int q = nblk >> 3, r = nblk & 7;
    return x * q + (x < r ? x : r) + k;
}

// spatial dimension of a block size (Q1..Q3 in 2D: 4, 9, 16; in 3D: 8, 27, 64)
template <int B>
constexpr int dim_of() {
    return (B == 8 || B == 27 || B == 64) ? 3 : 2;
}

// Cells per tile: 256 / b, but 8 (two whole cells per wave) for b = 25.  The
// values that a cell gathers are then shared by lane shuffles, which is worth
// the idle lanes: axis-ELL level of 1024 cells, FP64 step 8.7 -> 7.1 us and
// residual 10.8 -> 6.2 us, FP32 5.6 -> 4.9 and 6.5 -> 4.6 us.  b = 27 keeps 9
// cells that straddle waves: with 8 its FP64 level products gain as much (slots,
// 1728 cells, step 38.4 -> 28.5 us), but in mixed precision the narrower
// workgroups cost a time step of 64^3 Q2 boxes 9.93 ms instead of 9.89.
__host__ __device__ constexpr int tile_cells(int b) { return b == 25 ? 8 : kWG / b; }

template <typename T, int B>
struct Tile {
    static constexpr int TC = tile_cells(B);  // cells per tile / workgroup
    static constexpr int TR = TC * B;         // rows per tile
};

// Nodes per axis of a block size.
__host__ __device__ constexpr int ax_nodes_1d(int b, int d) { return d == 2 ? (b == 4 ? 2 : b == 9 ? 3 : b == 16 ? 4 : 5) : (b == 8 ? 2 : b == 27 ? 3 : 4); }
// coordinate of node j along axis a, and its index among the nodes of a face normal to a
__host__ __device__ constexpr int node_coord(int j, int a, int q) { return a == 0 ? j % q : a == 1 ? (j / q) % q : j / (q * q); }
__host__ __device__ constexpr int node_tan(int j, int a, int q) {
    return a == 0 ? (j / q) % q + q * (j / (q * q)) : a == 1 ? j % q + q * (j / (q * q)) : j % (q * q);
}

// Orders one wave's LDS accesses at the compiler level.  Only lanes of one
// wave exchange data through the buffers it guards, and LDS executes a
// wave's instructions in issue order, so no barrier is needed.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Workgroup sum of a double into partial[blockIdx.x] (deterministic order).
// NT: threads of the workgroup; one slot per wave (the cell kernels run three
// to seven).
template <int NT = kWG>
__device__ __forceinline__ void wg_sum_store(double v, double* partial) {
    constexpr int NW = NT / 64;
    __shared__ double red[NW];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) red[w] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int k = 0; k < NW; ++k) s += red[k];
        partial[blockIdx.x] = s;
    }
}

}  // namespace dgmg
