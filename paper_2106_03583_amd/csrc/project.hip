// Pressure projection around the Poisson solve: the fractional step of
// Eqs. (3)-(6) on the staggered grid (Sec. 2; velocities on cell faces),
//     rhs = D u* / (gamma dt),   L_h Phi = rhs,   u = u* - gamma dt G Phi,
// after which D u vanishes to the solver's tolerance (the check of Sec. 4.1).
// D is the finite-volume divergence (face flux differences over the cell
// width) and G the face gradient, so D G = L_h with the boundary rules of
// the solver: a Neumann face keeps its velocity (G Phi = 0), a Dirichlet face
// sees the mirrored ghost -Phi one cell width away, a joined or periodic face
// the partner's cell at half the two widths.  A face shared by two blocks is
// stored (and updated) in both.
//
// Face fields are packed block after block: u (nz, ny, nx + 1), v (nz, ny + 1,
// nx), w (nz, ny, nx) for periodic z (face k - 1/2, cyclic) else (nz + 1, ny, nx).
#include "op3.h"

namespace mbp {

namespace {

__device__ __forceinline__ int xcd_remap_pj(int g, int n) {
    int x = g & 7, l = g >> 3;
    int per = n >> 3, rem = n & 7;
    return x * per + min(x, rem) + l;
}

struct PjArgs {
    const DBlock* B;  // finest-level blocks
    const int4* tiles;
    int ntiles;
    const double* dp;
    const int* pt;    // per block {dcx, dcy, gx, gy, rows before, columns before}
    int nz, nzw;      // cells and z faces per column
    double dz;
    int zper, zlo, zhi;
};

__device__ __forceinline__ long long uoff(const PjArgs& a, const DBlock& b, int bi) {
    return (long long)a.nz * (b.off + a.pt[6 * bi + 4]);
}
__device__ __forceinline__ long long voff(const PjArgs& a, const DBlock& b, int bi) {
    return (long long)a.nz * (b.off + a.pt[6 * bi + 5]);
}
__device__ __forceinline__ long long woff(const PjArgs& a, const DBlock& b) { return (long long)a.nzw * b.off; }
__device__ __forceinline__ long long coff(const PjArgs& a, const DBlock& b) { return (long long)a.nz * b.off; }

}  // namespace

// out = scale * D(u, v, w) on every cell.
__global__ void __launch_bounds__(256)
k_divergence(PjArgs a, const double* __restrict__ u, const double* __restrict__ v, const double* __restrict__ w,
             double scale, double* __restrict__ out) {
    const int k = blockIdx.y;
    const int4 t = a.tiles[xcd_remap_pj(blockIdx.x, a.ntiles)];
    const int bi = t.x;
    const DBlock b = a.B[bi];
    const int i = t.y + threadIdx.x;
    if (i >= b.nx) return;
    const double* dcx = a.dp + a.pt[6 * bi + 0];
    const double* dcy = a.dp + a.pt[6 * bi + 1];
    const double* ub = u + uoff(a, b, bi);
    const double* vb = v + voff(a, b, bi);
    const double* wb = w + woff(a, b);
    const int k1 = a.zper ? (k + 1) % a.nz : k + 1;
    const double idz = 1.0 / a.dz;
    for (int r = threadIdx.y; r < kTileY; r += kRowsPerPass) {
        const int j = t.z + r;
        if (j >= b.ny) break;
        const long long ui = ((long long)k * b.ny + j) * (b.nx + 1) + i;
        const long long vi = ((long long)k * (b.ny + 1) + j) * b.nx + i;
        const long long wi = ((long long)k * b.ny + j) * b.nx + i;
        const long long wi1 = ((long long)k1 * b.ny + j) * b.nx + i;
        const double d = (ub[ui + 1] - ub[ui]) / dcx[i] + (vb[vi + b.nx] - vb[vi]) / dcy[j] + (wb[wi1] - wb[wi]) * idz;
        out[coff(a, b) + ((long long)k * b.ny + j) * b.nx + i] = scale * d;
    }
}

namespace {

// Phi at (ii, jj) of block b, which may be one cell outside along one axis: the
// partner's cell across a joined face, the mirrored ghost -Phi of the cell inside
// across a Dirichlet wall (a Neumann wall's face coefficient is zero).  Offset at
// plane 0, plane and row strides, sign.
struct PhiSide {
    long long off, plane;
    int row;
    double sign;
};
__device__ __forceinline__ PhiSide phi_side(const PjArgs& a, const DBlock& b, int ii, int jj) {
    int f = -1;
    if (ii < 0) f = XM;
    else if (ii >= b.nx) f = XP;
    else if (jj < 0) f = YM;
    else if (jj >= b.ny) f = YP;
    const int nb = f == XM ? b.nbr[XM] : f == XP ? b.nbr[XP] : f == YM ? b.nbr[YM] : f == YP ? b.nbr[YP] : -1;
    if (nb >= 0) {
        const DBlock& n = a.B[nb];
        const int ni = f == XM ? n.nx - 1 : f == XP ? 0 : ii;
        const int nj = f == YM ? n.ny - 1 : f == YP ? 0 : jj;
        return PhiSide{coff(a, n) + (long long)nj * n.nx + ni, (long long)n.ny * n.nx, n.nx, 1.0};
    }
    const int ci = min(max(ii, 0), b.nx - 1), cj = min(max(jj, 0), b.ny - 1);
    return PhiSide{coff(a, b) + (long long)cj * b.nx + ci, (long long)b.ny * b.nx, b.nx, f < 0 ? 1.0 : -1.0};
}

}  // namespace

// u -= gdt G Phi on every face of the block: each cell updates its lower x,
// y and z faces, the last cell of a row / column / z column also the upper
// one.  Faces with a zero coefficient (Neumann walls) are left untouched.
//
// Bound by memory: Phi in, three fields in and out.  A wave marches 64 columns x
// four rows through a chunk of planes, so Phi below in z and, within the four
// rows, below in y stays in registers and Phi to the left comes from the next
// lane; what lies outside (the row under the group, lane 0's left column) is
// addressed once, a plane stride apart.  One cell a thread and plane, each face
// resolving its neighbour, took 278 us at 256 x 192 x 256 (2.5 TB/s); now 141 us
// (5.0 TB/s).
__global__ void __launch_bounds__(256)
k_gradient_update(PjArgs a, const double* __restrict__ phi, double gdt, double* __restrict__ u,
                  double* __restrict__ v, double* __restrict__ w, int chunk) {
    constexpr int R = kTileY / kRowsPerPass;
    const int4 t = a.tiles[xcd_remap_pj(blockIdx.x, a.ntiles)];
    const int bi = t.x;
    const DBlock b = a.B[bi];
    const int i = t.y + threadIdx.x, ic = min(i, b.nx - 1);
    const int j0 = t.z + R * __builtin_amdgcn_readfirstlane(threadIdx.y);  // rows j0 .. j0 + R - 1
    if (j0 >= b.ny) return;
    const int rows = min(R, b.ny - j0);
    const int k0 = blockIdx.y * chunk, k1 = min(k0 + chunk, a.nz);
    const double* gx = a.dp + a.pt[6 * bi + 2];
    const double* gy = a.dp + a.pt[6 * bi + 3];
    const int nx = b.nx;
    const long long plane = (long long)b.ny * nx, uplane = (long long)b.ny * (nx + 1), vplane = plane + nx;
    const double* pb = phi + coff(a, b) + (long long)j0 * nx + ic;
    double* ub = u + uoff(a, b, bi) + (long long)j0 * (nx + 1) + ic;
    double* vb = v + voff(a, b, bi) + (long long)j0 * nx + ic;
    double* wb = w + woff(a, b) + (long long)j0 * nx + ic;
    const double gz = gdt * (1.0 / a.dz);
    const bool in = i < nx, first = threadIdx.x == 0, last = i == nx - 1;
    const double gl = gx[ic], gr = gx[nx];
    const bool left = in && gl != 0.0, right = last && gr != 0.0;
    double gb[R + 1];
#pragma unroll
    for (int r = 0; r <= R; ++r) gb[r] = gy[min(j0 + r, b.ny)];
    const bool top = j0 + rows == b.ny && gy[b.ny] != 0.0;
    // lane 0's left column, the last column's right, the rows below and above
    const PhiSide sl = phi_side(a, b, t.y - 1, j0), sr = phi_side(a, b, nx, j0);
    const PhiSide sb = phi_side(a, b, 0, j0 - 1), su = phi_side(a, b, 0, b.ny);
    double pm[R], pc[R], pn[R];
    {
        const int km = k0 > 0 ? k0 - 1 : a.zper ? a.nz - 1 : 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int ro = min(r, rows - 1) * nx;
            pm[r] = pb[km * plane + ro];
            pc[r] = pb[k0 * plane + ro];
        }
    }
    for (int k = k0; k < k1; ++k) {
        double uv[R], vv[R], wv[R], lv[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int rc = min(r, rows - 1);
            if (k + 1 < k1) pn[r] = pb[(k + 1) * plane + rc * nx];
            uv[r] = ub[k * uplane + (long long)rc * (nx + 1)];
            vv[r] = vb[k * vplane + rc * nx];
            wv[r] = wb[k * plane + rc * nx];
            lv[r] = first ? sl.sign * phi[sl.off + k * sl.plane + rc * sl.row] : 0.0;
        }
        const double below = sb.sign * phi[sb.off + k * sb.plane + ic];
        const bool zface = a.zper || k > 0 || a.zlo == MBP_DIRICHLET;
        const bool ghost = !a.zper && k == 0;  // mirrored: -Phi
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double l = from_left(pc[r]);
            if (r < rows) {
                const double pl = first ? lv[r] : l, pb1 = r ? pc[r ? r - 1 : 0] : below;
                if (left) ub[k * uplane + r * (nx + 1)] = uv[r] - gdt * gl * (pc[r] - pl);
                if (right) {
                    const double pr = sr.sign * phi[sr.off + k * sr.plane + r * sr.row];
                    ub[k * uplane + r * (nx + 1) + 1] -= gdt * gr * (pr - pc[r]);
                }
                if (in && gb[r] != 0.0) vb[k * vplane + r * nx] = vv[r] - gdt * gb[r] * (pc[r] - pb1);
                if (in && zface) wb[k * plane + r * nx] = wv[r] - gz * (pc[r] - (ghost ? -pc[r] : pm[r]));
                if (in && top && r == rows - 1) {
                    const double pu = su.sign * phi[su.off + k * su.plane + ic];
                    vb[k * vplane + (r + 1) * nx] -= gdt * gy[b.ny] * (pu - pc[r]);
                }
                if (in && k == a.nz - 1 && !a.zper && a.zhi == MBP_DIRICHLET)
                    wb[(k + 1) * plane + r * nx] -= gz * (-pc[r] - pc[r]);
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            pm[r] = pc[r];
            pc[r] = pn[r];
        }
    }
}

namespace {
PjArgs pj_args(const mbp_plan* P) {
    const Level& L = P->levels[0];
    const bool per = P->g.zkind == Z_PP;
    return PjArgs{P->d_blk + L.blk_off, P->d_tiles + L.tile_off, L.ntiles, P->d_dbl, P->d_int + P->proj_tab,
                  P->g.nz, per ? P->g.nz : P->g.nz + 1, P->g.dz, per ? 1 : 0, P->g.zlo, P->g.zhi};
}
}  // namespace

void velocity_offsets(const mbp_plan* P, int64_t* uo, int64_t* vo, int64_t* wo) {
    const int nz = P->g.nz, nzw = P->g.zkind == Z_PP ? nz : nz + 1;
    int64_t a = 0, c = 0, e = 0;
    for (int b = 0; b <= P->g.nb; ++b) {
        if (uo) uo[b] = a;
        if (vo) vo[b] = c;
        if (wo) wo[b] = e;
        if (b == P->g.nb) break;
        const int64_t nx = P->g.nx[b], ny = P->g.ny[b];
        a += int64_t(nz) * ny * (nx + 1);
        c += int64_t(nz) * (ny + 1) * nx;
        e += int64_t(nzw) * ny * nx;
    }
}

void launch_divergence(const mbp_plan* P, const double* u, const double* v, const double* w, double scale,
                       double* out, hipStream_t s) {
    const Level& L = P->levels[0];
    hipLaunchKernelGGL(k_divergence, dim3(L.ntiles, P->g.nz), dim3(kTileX, kRowsPerPass), 0, s, pj_args(P), u, v, w,
                       scale, out);
}

void launch_gradient_update(const mbp_plan* P, const double* phi, double gdt, double* u, double* v, double* w,
                            hipStream_t s) {
    const Level& L = P->levels[0];
    const int chunk = zchunk(L.ntiles, P->g.nz);
    hipLaunchKernelGGL(k_gradient_update, dim3(L.ntiles, (P->g.nz + chunk - 1) / chunk), dim3(kTileX, kRowsPerPass), 0,
                       s, pj_args(P), phi, gdt, u, v, w, chunk);
}

}  // namespace mbp
