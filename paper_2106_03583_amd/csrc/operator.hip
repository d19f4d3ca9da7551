// The 3D operator on the packed fields: out = (L_h - alpha) p, and the check of
// a solve, |f - shift - (L_h - alpha) p| and |f - shift|.
#include "op3.h"

namespace mbp {

// A workgroup owns one 64 x 16 x-y tile and marches a chunk of planes; a thread
// keeps its four cells' values at planes k-1, k, k+1 in registers and the plane-k
// tile, with a one-cell ring, is in LDS (two copies: one barrier a step).  The
// next plane is loaded during this plane's work.
//
// Bound by memory: p in once and out (or f) once.  One workgroup a plane and
// tile, five loads a cell, had the neighbours' planes from L2 and a chain of
// per-cell edge branches: 190 us (apply) and 183 us (check) at 320 x 256 x 256,
// 1.8 TB/s; now 78 us each (4.3 TB/s; a large copy reaches 4.9).  A subtraction
// beside the guarded load of f made the compiler wait for every load: 102 us.
//
// NORM: per-workgroup partial sums of (f - shift - (L_h - alpha) p)^2 into part[w]
// and of (f - shift)^2 into part[nw + w], nw = workgroups of the launch.
template <bool NORM>
__global__ void __launch_bounds__(256)
k_operator(Op3 o, const int4* __restrict__ tiles, int ntiles, const double* __restrict__ p,
           const double* __restrict__ f, double shift, double* __restrict__ out, double* __restrict__ part,
           int chunk) {
    __shared__ double sp2[2][kTileY + 2][kTileX + 2];
    const int4 t = tiles[xcd_remap3(blockIdx.x, ntiles)];
    const DBlock b = o.B[t.x];
    const int k0 = blockIdx.y * chunk, k1 = min(k0 + chunk, o.nz);
    // a wave is one row group: its rows and their coefficients are uniform
    const int tx = threadIdx.x, ty = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int tid = ty * kTileX + tx;
    const int i = t.y + tx;
    const bool in_i = i < b.nx;
    const double* dp = o.dp;
    constexpr int R = kTileY / kRowsPerPass;
    const int plane = b.nx * b.ny;
    const bool per = o.zlo == MBP_PERIODIC;
    const double glo = o.zlo == MBP_NEUMANN ? 1.0 : -1.0, ghi = o.zhi == MBP_NEUMANN ? 1.0 : -1.0;
    const double wxm = in_i ? dp[b.cx + i] : 0.0, wxp = in_i ? dp[b.cx + b.nx + i] : 0.0;
    const double dx = in_i ? dp[b.cx + 2 * b.nx + i] : 0.0;
    bool act[R], ok[R];
    double wym[R], wyp[R], d[R];
    long long at[R];  // own cell, or the cell across a joined edge in a ragged tile
    long long fo[R];  // own cell, of an inactive one the block's first
    int st[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int j = t.z + ty + kRowsPerPass * r, jc = min(j, b.ny - 1);
        act[r] = in_i && j < b.ny;
        wym[r] = dp[b.cy + jc];
        wyp[r] = dp[b.cy + b.ny + jc];
        d[r] = dx + dp[b.cy + 2 * b.ny + jc] - o.alpha;
        ok[r] = ring_cell(o, b, i, j, at[r], st[r]);
        if (!ok[r]) at[r] = (long long)o.nz * b.off;  // loads need no branch: masked where they are used
        fo[r] = (long long)o.nz * b.off + (act[r] ? (long long)j * b.nx + i : 0);
    }
    // the tile's ring: one cell of 160 threads
    long long rat = 0;
    int rst = 0;
    bool rok = false;
    const int side = tid < 2 * kTileX ? tid / kTileX : (tid - 2 * kTileX) / kTileY;
    const int along = tid < 2 * kTileX ? tid % kTileX : (tid - 2 * kTileX) % kTileY;
    if (tid < 2 * kTileX) rok = ring_cell(o, b, t.y + along, side == 0 ? t.z - 1 : t.z + kTileY, rat, rst);
    else if (tid < 2 * kTileX + 2 * kTileY)
        rok = ring_cell(o, b, side == 0 ? t.y - 1 : t.y + kTileX, t.z + along, rat, rst);
    if (!rok) rat = (long long)o.nz * b.off;
    auto load = [&](int kp, double* v) {
        const int q = max(0, zplane(o, kp));
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = p[at[r] + (long long)q * st[r]];
    };
    auto loadf = [&](int kp, double* v) {
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = f[fo[r] + (long long)kp * plane];
    };
    double pm[R], pc[R], pp[R], pn[R], fc[R], fn[R];
    double rc = p[rat + (long long)k0 * rst];
    load(k0 - 1, pm);
    load(k0, pc);
    load(k0 + 1, pp);
    if (NORM) loadf(k0, fc);
    double rr = 0.0, ff = 0.0;
    for (int k = k0; k < k1; ++k) {
        double(*sp)[kTileX + 2] = sp2[k & 1];
#pragma unroll
        for (int r = 0; r < R; ++r) sp[ty + kRowsPerPass * r + 1][tx + 1] = ok[r] ? pc[r] : 0.0;
        if (tid < 2 * kTileX) sp[side == 0 ? 0 : kTileY + 1][along + 1] = rok ? rc : 0.0;
        else if (tid < 2 * kTileX + 2 * kTileY) sp[along + 1][side == 0 ? 0 : kTileX + 1] = rok ? rc : 0.0;
        if (k + 1 < k1) {
            load(k + 2, pn);
            if (NORM) loadf(k + 1, fn);
            rc = p[rat + (long long)(k + 1) * rst];
        }
        __syncthreads();
        const bool lo = !per && k == 0, hi = !per && k == o.nz - 1;  // mirrored ghosts
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int ly = ty + kRowsPerPass * r + 1, lx = tx + 1;
            const double v = pc[r], zm = lo ? glo * v : pm[r], zp = hi ? ghi * v : pp[r];
            const double a = wxm * sp[ly][lx - 1] + wxp * sp[ly][lx + 1] + wym[r] * sp[ly - 1][lx] +
                             wyp[r] * sp[ly + 1][lx] + d[r] * v + (zm - 2.0 * v + zp) * o.idz2;
            if (act[r]) {
                if (NORM) {
                    const double fv = fc[r] - shift, res = fv - a;
                    rr += res * res;
                    ff += fv * fv;
                } else {
                    out[fo[r] + (long long)k * plane] = a;
                }
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            pm[r] = pc[r];
            pc[r] = pp[r];
            pp[r] = pn[r];
            fc[r] = fn[r];
        }
    }
    if (NORM) {
        __shared__ double red[8];
        const long long w = (long long)blockIdx.y * gridDim.x + blockIdx.x;
        const long long nw = (long long)gridDim.y * gridDim.x;
        const double sr = wg_sum(rr, red);
        if (tid == 0) part[w] = sr;
        const double sf = wg_sum(ff, red);
        if (tid == 0) part[nw + w] = sf;
    }
}

// out[0] = sqrt(sum part[0, n)), out[1] = sqrt(sum part[n, 2n)).
__global__ void __launch_bounds__(1024) k_resnorm_finish(const double* __restrict__ part, long long n,
                                                         double* __restrict__ out) {
    __shared__ double red[16];
    for (int h = 0; h < 2; ++h) {
        double acc = 0.0;
        for (long long e = threadIdx.x; e < n; e += blockDim.x) acc += part[h * n + e];
        for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
        __syncthreads();
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
        __syncthreads();
        if (threadIdx.x == 0) {
            double s2 = 0.0;
            for (int w = 0; w < int(blockDim.x >> 6); ++w) s2 += red[w];
            out[h] = sqrt(s2);
        }
    }
}

namespace {
Op3 op_of(const mbp_plan* P) {
    return Op3{P->d_blk + P->levels[0].blk_off, P->d_dbl, P->g.nz, 1.0 / (P->g.dz * P->g.dz), P->g.zlo, P->g.zhi,
               P->opt.helmholtz};
}
}  // namespace

// One pair of sums per tile and plane at most; the chunked march writes fewer.
size_t resnorm_scratch_doubles(const mbp_plan* P) {
    return 2 * size_t(P->levels[0].ntiles) * size_t(P->g.nz);
}

void launch_resnorm3d(const mbp_plan* P, const double* f, const double* p, double shift, double* part,
                      double* out, hipStream_t s) {
    const Level& L = P->levels[0];
    const int chunk = zchunk(L.ntiles, P->g.nz);
    const dim3 g(unsigned(L.ntiles), unsigned((P->g.nz + chunk - 1) / chunk));
    hipLaunchKernelGGL(k_operator<true>, g, dim3(kTileX, kRowsPerPass), 0, s, op_of(P), P->d_tiles + L.tile_off,
                       L.ntiles, p, f, shift, nullptr, part, chunk);
    hipLaunchKernelGGL(k_resnorm_finish, dim3(1), dim3(1024), 0, s, part, (long long)g.x * g.y, out);
}

void launch_apply3d(const mbp_plan* P, const double* p, double* out, hipStream_t s) {
    const Level& L = P->levels[0];
    const int chunk = zchunk(L.ntiles, P->g.nz);
    const dim3 g(unsigned(L.ntiles), unsigned((P->g.nz + chunk - 1) / chunk));
    hipLaunchKernelGGL(k_operator<false>, g, dim3(kTileX, kRowsPerPass), 0, s, op_of(P), P->d_tiles + L.tile_off,
                       L.ntiles, p, nullptr, 0.0, out, nullptr, chunk);
}

}  // namespace mbp
