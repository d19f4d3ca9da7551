// What the kernels on the packed 3D fields share: the operator's description,
// cells across a block's edges, and how many planes a z-marching workgroup takes.
#pragma once

#include <algorithm>

#include "internal.h"
#include "wave.h"

namespace mbp {

__device__ __forceinline__ int xcd_remap3(int g, int n) {
    int x = g & 7, l = g >> 3;
    int per = n >> 3, rem = n & 7;
    return x * per + min(x, rem) + l;
}

__device__ __forceinline__ long long cell3(const DBlock& b, int nz, int k, int j, int i) {
    return (long long)nz * b.off + ((long long)k * b.ny + j) * b.nx + i;
}

// Sum over one workgroup; the result is valid in thread 0.
__device__ __forceinline__ double wg_sum(double v, double* red) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    const int t = threadIdx.x + threadIdx.y * blockDim.x;
    const int w = t >> 6, nw = (blockDim.x * blockDim.y + 63) >> 6;
    __syncthreads();
    if ((t & 63) == 0) red[w] = v;
    __syncthreads();
    double s = 0.0;
    if (t == 0)
        for (int k = 0; k < nw; ++k) s += red[k];
    return s;
}

// (L_h - alpha) p at cell (b, k, j, i) and its diagonal coefficient.  x-y
// neighbours beyond a joined face come from the partner block; beyond a wall
// the coefficient already holds the boundary condition (Neumann: none,
// Dirichlet: folded into the diagonal).  z ends: periodic wrap, or a mirror
// ghost (Neumann +p, Dirichlet -p) one cell away.
struct Op3 {
    const DBlock* B;
    const double* dp;
    int nz;
    double idz2;
    int zlo, zhi;  // MBP_PERIODIC / MBP_NEUMANN / MBP_DIRICHLET
    double alpha;
};

// Cell (ii, jj) of block b, which may lie one cell outside the block: its
// offset at plane 0 and its plane stride (the partner's cell across a joined
// face).  False beyond a wall (the coupling is zero) and diagonally outside.
__device__ __forceinline__ bool ring_cell(const Op3& o, const DBlock& b, int ii, int jj, long long& off, int& stride) {
    const bool xin = ii >= 0 && ii < b.nx, yin = jj >= 0 && jj < b.ny;
    int n = -1;
    off = (long long)o.nz * b.off + (long long)jj * b.nx + ii;
    stride = b.nx * b.ny;
    if (xin && yin) return true;
    if (yin && ii == -1) n = b.nbr[XM];
    else if (yin && ii == b.nx) n = b.nbr[XP];
    else if (xin && jj == -1) n = b.nbr[YM];
    else if (xin && jj == b.ny) n = b.nbr[YP];
    if (n < 0) return false;
    const DBlock& p = o.B[n];
    const int pi = ii < 0 ? p.nx - 1 : ii == b.nx ? 0 : ii, pj = jj < 0 ? p.ny - 1 : jj == b.ny ? 0 : jj;
    off = (long long)o.nz * p.off + (long long)pj * p.nx + pi;
    stride = p.nx * p.ny;
    return true;
}

// Plane index of z neighbour k (periodic wrap) or -1 where the ghost rule
// applies (its coupling is folded into the diagonal).
__device__ __forceinline__ int zplane(const Op3& o, int k) {
    if (k >= 0 && k < o.nz) return k;
    if (o.zlo == MBP_PERIODIC) return (k + o.nz) % o.nz;
    return -1;
}

// A z-marching workgroup owns one x-y tile and a chunk of planes.  The chunk is
// as short as it takes to fill the chip, as every chunk reads two planes more than
// it owns.  Sweeps of the 256^3 multigrid solve with 1024 / 2048 / 4096 workgroups
// wanted: 23.3 / 22.2 / 23.3 ms; with 32 planes whatever the level 44.7 ms.
constexpr int kZMost = 32;     // most planes of a chunk
constexpr int kZWgs = 2048;    // workgroups a launch aims at (eight a CU)

// Planes per workgroup (even) for a level of ntiles x-y tiles and nz planes.
inline int zchunk(int ntiles, int nz) {
    const int n = std::max(1, (kZWgs + ntiles - 1) / std::max(1, ntiles));  // chunks wanted
    const int c = ((nz + n - 1) / n + 1) & ~1;
    return std::min(kZMost, std::max(2, c));
}

}  // namespace mbp
