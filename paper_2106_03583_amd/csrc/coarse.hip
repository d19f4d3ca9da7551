// The levels that fit in LDS, one workgroup per mode: a V-cycle from zero (the
// coarse end of every V-cycle), or, when the whole hierarchy fits, complete
// solves.
//
// What bounds it is latency: a few thousand cells per mode, five or so levels,
// and a barrier after every colour.  So no phase does index arithmetic and a
// phase waits for little but its neighbours' values: each thread owns a few red
// and a few black cells of the top level for the whole launch (offsets of the
// neighbours, rhs, iterate, diagonal and its reciprocal in registers; the
// separable couplings in LDS tables) and at most one of each colour on the
// levels below.  A relaxation is four LDS reads, a multiply by the reciprocal
// (with one residual correction) and one LDS write.  Levels of at most 64 cells
// of a colour run in one wave without barriers, together with the exact coarsest
// solve, whose matrices sit in LDS.  The black cells' residual after a sweep is
// rounding, so the restriction takes the red ones: each writes its weighted
// residual to a slot of its 2 x 2 patch, and the coarse cell's owner adds the
// slots (no atomics, fixed order).  A correction is added to the black cells
// only, since the red ones are relaxed from black neighbours next.
//
// Records and tables are built by the host for any layout with full 2 : 1
// coarsening in every block (joined blocks, odd counts, odd periodic rings with
// their two extra colours); the generic kernels of mg.hip run the others.
#include <algorithm>
#include <cmath>
#include <map>
#include <mutex>
#include <utility>

#include "internal.h"
#include "wave.h"

namespace mbp {

// One cell: its offset in the level's plane, the places of its neighbours in the
// LDS iterate (another one's where there is none: the coupling is zero), its
// entries in the level's x and y tables, the slot of its residual, the places of
// the four coarse values of its correction (bit 15: negated), and as a coarse
// cell the first patch of its rhs (gp: patch row pitch, bits 14 / 15: an odd last
// column / row adds the next patch too).  Cells sit in LDS in the order of their
// records, colour by colour (the coarsest level's in plane order): a colour's
// neighbouring cells then read and write neighbouring words.
struct Raw {  // the words of a record that a smoothing cell needs, unpacked on use
    unsigned w[6];
    __device__ __forceinline__ int self() const { return int(w[0] & 0xffffu); }
};
struct CRec {
    unsigned short self, n[4], xi, yi, s;
    unsigned short c[4], g, gp, pad[2];
    __device__ __forceinline__ Raw words() const {
        const unsigned* u = reinterpret_cast<const unsigned*>(this);
        return Raw{{u[0], u[1], u[2], u[3], u[4], u[5]}};
    }
};
static_assert(sizeof(CRec) == 32, "eight words a record");

constexpr int kTab = 6;  // x / y table entry: lower and upper coupling, diagonal, restriction weight, lower prolongation weight

// One level as the kernel reads it (in the int pool).
struct CLev {
    int ncell;       // cells
    int n0, n1, n2, n3;  // cells per colour (n2, n3: odd rings only); records are stored colour by colour
    int rec;         // first record (int pool offset)
    int lrec;        // ... in the LDS copy, -1: not there
    int ltab;        // first table entry in the LDS copy
    int p, s;        // LDS element offsets of the iterate and of the residual slots
    int ns;          // slots per patch: 2, or 4 on a level with odd rings
    int odd;
};
static_assert(sizeof(CLev) == 48, "three 16-byte reads");

template <typename T>
struct CArgs {
    const int* ip;
    const double* dp;
    int lev, nl, ls;   // CLev array (int pool), levels, first level of the single-wave part (nl: none)
    int nc;
    const double* cwl;
    const double* cwr;
    const double* cmu;
    double cmumax;
    int wt, wlds;      // transposed coarsest matrices (double pool offset), copied to LDS or not
    int oT, oRed, oMu, oW, oP, oTab, oRec;  // byte offsets of the LDS parts
    int nslot, oS;     // residual slots (elements), first one (element of the P part)
    int tab0, ntab, rec0, nrec;        // pool ranges of the LDS copies (entries, records)
    T* pL;
    const T* fL;
    long long planeL;
    const double* shift;
    const int* act;
    const int* nact;
    int ncyc;          // V-cycles from zero
    // complete solves
    const double* sabs;
    int maxc;
    double rtol2, etol2;
    int* cyc;
    double* rnorm;
    double* fnorm;
};

namespace {

template <typename T>
struct Cell {
    int n[4], s;
    T w[4];
    T d, inv;  // diagonal with the shift and its reciprocal
    T rw;
    unsigned c01, c23;
    T wx, wy;
};

// The level descriptors are never written while a kernel runs: through the
// constant address space they come by scalar loads.
typedef __attribute__((address_space(4))) const CLev clev_t;
__device__ __forceinline__ CLev level_at(const CLev* lev, int k) {
    const clev_t* c = (const clev_t*)lev + k;
    CLev L;
    L.ncell = c->ncell;
    L.n0 = c->n0;
    L.n1 = c->n1;
    L.n2 = c->n2;
    L.n3 = c->n3;
    L.rec = c->rec;
    L.lrec = c->lrec;
    L.ltab = c->ltab;
    L.p = c->p;
    L.s = c->s;
    L.ns = c->ns;
    L.odd = c->odd;
    return L;
}

struct View {
    const CRec* rec;    // LDS copies
    const void* tab;
    double* b;          // coarsest rhs
    double* t;
    double* red;
    const double* w;    // LDS matrices
    const double* mu;   // coarsest eigenvalues (nc <= 64)
    const CLev* lev;
};

template <bool WG>
__device__ __forceinline__ void csync() {
    if constexpr (WG) {
        __syncthreads();
    } else {  // one wave: LDS keeps its order, only the compiler must
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

__device__ __forceinline__ double recip(double d) {
    double r = __builtin_amdgcn_rcp(d);
    r = fma(r, fma(-d, r, 1.0), r);
    return fma(r, fma(-d, r, 1.0), r);
}
__device__ __forceinline__ float recip(float d) {
    const float r = __builtin_amdgcn_rcpf(d);
    return fmaf(r, fmaf(-d, r, 1.0f), r);
}

template <typename T>
__device__ __forceinline__ T around(const Cell<T>& x, const T* p) {
    return x.w[0] * p[x.n[0]] + x.w[1] * p[x.n[1]] + x.w[2] * p[x.n[2]] + x.w[3] * p[x.n[3]];
}
// t / d with the reciprocal at hand and one residual correction
template <typename T>
__device__ __forceinline__ T solve_for(T t, T d, T inv) {
    const T q = t * inv;
    return fma(fma(-d, q, t), inv, q);
}
template <typename T>
__device__ __forceinline__ T signed_at(const T* p, unsigned c) {
    const T v = p[c & 0x7fffu];
    return (c & 0x8000u) ? -v : v;
}
template <typename T>
__device__ __forceinline__ T prolong(const Cell<T>& x, const T* pc) {
    const T e00 = signed_at(pc, x.c01 & 0xffffu), e10 = signed_at(pc, x.c01 >> 16);
    const T e01 = signed_at(pc, x.c23 & 0xffffu), e11 = signed_at(pc, x.c23 >> 16);
    return x.wy * (x.wx * e00 + (T(1) - x.wx) * e10) + (T(1) - x.wy) * (x.wx * e01 + (T(1) - x.wx) * e11);
}

// rhs of a coarse cell: the slots of its patches, in order
template <typename T>
__device__ __forceinline__ T gather(const T* S, int ns, const CRec& r) {
    const int g = r.g, gp = r.gp & 0x3fff;
    auto patch = [&](int k) __attribute__((always_inline)) -> T {
        const T* q = S + ns * k;
        return ns == 2 ? q[0] + q[1] : (q[0] + q[1]) + (q[2] + q[3]);
    };
    T v = patch(g);
    if (r.gp & 0x4000) v += patch(g + 1);
    if (r.gp & 0x8000) {
        v += patch(g + gp);
        if (r.gp & 0x4000) v += patch(g + gp + 1);
    }
    return v;
}

template <typename T>
__device__ __forceinline__ CRec rec_of(const CArgs<T>& a, const View& v, const CLev& L, int k) {
    if (L.lrec >= 0) return v.rec[L.lrec + k];
    return reinterpret_cast<const CRec*>(a.ip + L.rec)[k];
}
// All of a cell but its diagonal (what a caller does not use is not read)
template <typename T>
__device__ __forceinline__ void couplings(Cell<T>& x, const View& v, const CLev& L, const Raw& r) {
    x.n[0] = int(r.w[0] >> 16);
    x.n[1] = int(r.w[1] & 0xffffu);
    x.n[2] = int(r.w[1] >> 16);
    x.n[3] = int(r.w[2] & 0xffffu);
    x.s = int(r.w[3] >> 16);
    x.c01 = r.w[4];
    x.c23 = r.w[5];
    const T* t = static_cast<const T*>(v.tab) + kTab * L.ltab;
    const T* xt = t + kTab * int(r.w[2] >> 16);
    const T* yt = t + kTab * int(r.w[3] & 0xffffu);
    x.w[0] = xt[0];
    x.w[1] = xt[1];
    x.w[2] = yt[0];
    x.w[3] = yt[1];
    x.rw = xt[3] * yt[3];
    x.wx = xt[4];
    x.wy = yt[4];
}
template <typename T>
__device__ __forceinline__ void cell_of(Cell<T>& x, const View& v, const CLev& L, const Raw& r, T sig) {
    couplings(x, v, L, r);
    const T* t = static_cast<const T*>(v.tab) + kTab * L.ltab;
    x.d = t[kTab * int(r.w[2] >> 16) + 2] + t[kTab * int(r.w[3] & 0xffffu) + 2] + sig;
    x.inv = recip(x.d);
}

// ---- levels with odd rings: four colours, everything read per phase ----

template <typename T, bool WG>
__device__ __forceinline__ void odd_smooth(const CArgs<T>& a, const View& v, const CLev& L, T* p, const T* S, int ns, const T* fg, T sig,
                           int tid, int nthr) {
    const int cnt[4] = {L.n0, L.n1, L.n2, L.n3};
    int base = 0;
#pragma unroll 1
    for (int c = 0; c < 4; ++c) {
#pragma unroll 1
        for (int k = tid; k < cnt[c]; k += nthr) {
            const CRec r = rec_of(a, v, L, base + k);
            Cell<T> x;
            cell_of(x, v, L, r.words(), sig);
            const T f = fg ? fg[r.self] : gather(S, ns, r);
            p[base + k] = solve_for(f - around(x, p), x.d, x.inv);
        }
        base += cnt[c];
        csync<WG>();
    }
}
template <typename T, bool WG>
__device__ __forceinline__ void odd_down(const CArgs<T>& a, const View& v, const CLev& L, T* p, T* Sl, const T* S, int ns, const T* fg,
                         T sig, bool zero, int tid, int nthr) {
    if (zero) {
        for (int k = tid; k < L.ncell; k += nthr) p[k] = T(0);
        csync<WG>();
    }
    odd_smooth<T, WG>(a, v, L, p, S, ns, fg, sig, tid, nthr);
#pragma unroll 1
    for (int k = tid; k < L.ncell; k += nthr) {
        const CRec r = rec_of(a, v, L, k);
        Cell<T> x;
        cell_of(x, v, L, r.words(), sig);
        const T f = fg ? fg[r.self] : gather(S, ns, r);
        Sl[x.s] = x.rw * (f - (around(x, p) + x.d * p[k]));
    }
    csync<WG>();
}
template <typename T, bool WG>
__device__ __forceinline__ void odd_up(const CArgs<T>& a, const View& v, const CLev& L, T* p, const T* pc, const T* S, int ns, const T* fg,
                       T sig, int tid, int nthr) {
#pragma unroll 1
    for (int k = tid; k < L.ncell; k += nthr) {
        const CRec r = rec_of(a, v, L, k);
        Cell<T> x;
        cell_of(x, v, L, r.words(), sig);
        p[k] += prolong(x, pc);
    }
    csync<WG>();
    odd_smooth<T, WG>(a, v, L, p, S, ns, fg, sig, tid, nthr);
}

// ---- levels below the top: at most one cell of each colour per thread ----

// What a thread holds of a level: loaded before the barrier that ends the
// previous level's work, so that the record and table reads overlap it.
template <typename T>
struct Mine {
    CRec rr, rb;
    Cell<T> r, b;
};
template <typename T>
__device__ __forceinline__ void load_mine(Mine<T>& x, const CArgs<T>& a, const View& v, const CLev& L, T sig, int tid) {
    // threads without a cell load the last one (and never write it)
    x.rr = rec_of(a, v, L, min(tid, L.n0 - 1));
    x.rb = rec_of(a, v, L, L.n0 + min(tid, L.n1 - 1));
    cell_of(x.r, v, L, x.rr.words(), sig);
    cell_of(x.b, v, L, x.rb.words(), sig);
}

template <typename T, bool WG>
__device__ __forceinline__ void down(const Mine<T>& x, const CLev& L, T* p, T* Sl, const T* S, int ns, int tid) {
    const T fr = gather(S, ns, x.rr), fb = gather(S, ns, x.rb);
    const T pr = solve_for(fr, x.r.d, x.r.inv);
    if (tid < L.n0) p[tid] = pr;
    csync<WG>();
    const T q = solve_for(fb - around(x.b, p), x.b.d, x.b.inv);
    if (tid < L.n1) p[L.n0 + tid] = q;
    csync<WG>();
    const T w = x.r.rw * (fr - (around(x.r, p) + x.r.d * pr));
    if (tid < L.n0) Sl[x.r.s] = w;
}
template <typename T, bool WG>
__device__ __forceinline__ void up(const Mine<T>& x, const CLev& L, T* p, const T* pc, const T* S, int ns, int tid) {
    const T fr = gather(S, ns, x.rr), fb = gather(S, ns, x.rb);
    T q = p[L.n0 + min(tid, L.n1 - 1)] + prolong(x.b, pc);
    if (tid < L.n1) p[L.n0 + tid] = q;
    csync<WG>();
    q = solve_for(fr - around(x.r, p), x.r.d, x.r.inv);
    if (tid < L.n0) p[tid] = q;
    csync<WG>();
    q = solve_for(fb - around(x.b, p), x.b.d, x.b.inv);
    if (tid < L.n1) p[L.n0 + tid] = q;
}

// Exact coarsest solve in float64, x = Wl diag(1 / (mu + sigma)) Wr b, the null
// mode (mu + sigma = 0) dropped.  One wave, one row per lane (nc <= 64), or the
// workgroup with eight lanes per row.
template <typename T, bool WG>
__device__ __forceinline__ void coarsest(const CArgs<T>& a, const View& v, const CLev& L, T* p, const T* S, int ns, double sig,
                                         int tid, int nthr) {
    const int nc = a.nc;
#pragma unroll 1
    for (int k = tid; k < nc; k += nthr) {
        const CRec r = rec_of(a, v, L, k);
        v.b[r.self] = double(gather(S, ns, r));
    }
    csync<WG>();
    const double tiny = 1e-11 * (a.cmumax + fabs(sig));
    if constexpr (!WG) {
        const double* wr = a.wlds ? v.w : a.dp + a.wt;
        const double* wl = wr + nc * nc;
        const int k = min(tid, nc - 1);
        const double d = v.mu[k] + sig;
        const double rd = fabs(d) > tiny ? recip(d) : 0.0;  // the null mode is dropped
        double s0 = 0.0, s1 = 0.0;
        int j = 0;
#pragma unroll 4
        for (; j + 2 <= nc; j += 2) {
            s0 += wr[j * nc + k] * v.b[j];
            s1 += wr[(j + 1) * nc + k] * v.b[j + 1];
        }
        if (j < nc) s0 += wr[j * nc + k] * v.b[j];
        if (tid < nc) v.t[tid] = solve_for(s0 + s1, d, rd);
        csync<WG>();
        s0 = s1 = 0.0;
#pragma unroll 4
        for (j = 0; j + 2 <= nc; j += 2) {
            s0 += wl[j * nc + k] * v.t[j];
            s1 += wl[(j + 1) * nc + k] * v.t[j + 1];
        }
        if (j < nc) s0 += wl[j * nc + k] * v.t[j];
        if (tid < nc) p[tid] = T(s0 + s1);
    } else {
        const int g = tid & 7, rows = nthr / 8;
#pragma unroll 1
        for (int pass = 0; pass < 2; ++pass) {
            const double* W = pass == 0 ? a.cwr : a.cwl;
            const double* x = pass == 0 ? v.b : v.t;
#pragma unroll 1
            for (int k0 = 0; k0 < nc; k0 += rows) {
                const int k = k0 + tid / 8;
                double acc = 0.0;
                if (k < nc) {
                    const double* row = W + (long long)k * nc;
#pragma unroll 4
                    for (int j = g; j < nc; j += 8) acc += row[j] * x[j];
                }
                for (int o = 1; o < 8; o <<= 1) acc += __shfl_xor(acc, o);
                if (k < nc && g == 0) {
                    const double d = a.cmu[k] + sig;
                    if (pass == 0) v.t[k] = fabs(d) > tiny ? acc / d : 0.0;
                    else p[k] = T(acc);
                }
            }
            if (pass == 0) csync<WG>();
        }
    }
}

// Everything below the top level: its rhs sits in the top level's slots, whose
// last writes are published by the first barrier here; the last barrier
// publishes the correction.
template <typename T, bool ODD>
__device__ __forceinline__ void below(const CArgs<T>& a, const View& v, T* P, double sigd, int tid, int nthr) {
    const T sig = T(sigd);
    const int last = a.nl - 1, ls = a.ls;
    CLev L, U;
    Mine<T> x;
    auto fetch = [&](int k) __attribute__((always_inline)) {
        L = level_at(v.lev, k);
        U = level_at(v.lev, k - 1);
        if (k < last && !(ODD && L.odd)) load_mine(x, a, v, L, sig, tid);
    };
    fetch(1);
    __syncthreads();
    auto downward = [&](auto wg, int from, int to, int n) __attribute__((always_inline)) {
        constexpr bool WG = decltype(wg)::value;
#pragma unroll 1
        for (int k = from; k < to; ++k) {
            if (ODD && L.odd) odd_down<T, WG>(a, v, L, P + L.p, P + L.s, P + U.s, U.ns, nullptr, sig, true, tid, n);
            else down<T, WG>(x, L, P + L.p, P + L.s, P + U.s, ODD ? U.ns : 2, tid);
            fetch(k + 1);
            csync<WG>();
        }
    };
    auto upward = [&](auto wg, int from, int to, int n) __attribute__((always_inline)) {
        constexpr bool WG = decltype(wg)::value;
#pragma unroll 1
        for (int k = from; k > to; --k) {
            const T* pc = P + level_at(v.lev, k + 1).p;
            if (ODD && L.odd) odd_up<T, WG>(a, v, L, P + L.p, pc, P + U.s, U.ns, nullptr, sig, tid, n);
            else up<T, WG>(x, L, P + L.p, pc, P + U.s, ODD ? U.ns : 2, tid);
            if (k > 1) fetch(k - 1);
            csync<WG>();
        }
    };
    auto solve = [&](auto wg, int n) __attribute__((always_inline)) {
        constexpr bool WG = decltype(wg)::value;
        coarsest<T, WG>(a, v, L, P + L.p, P + U.s, ODD ? U.ns : 2, sigd, tid, n);
        if (last > 1) fetch(last - 1);
        csync<WG>();
    };
    if (ls >= a.nl) {
        downward(std::true_type{}, 1, last, nthr);
        solve(std::true_type{}, nthr);
        upward(std::true_type{}, last - 1, 0, nthr);
        return;
    }
    downward(std::true_type{}, 1, ls, nthr);
    if (tid < 64) {
        downward(std::false_type{}, ls, last, 64);
        solve(std::false_type{}, 64);
        upward(std::false_type{}, last - 1, ls - 1, 64);
    } else if (ls > 1) {
        fetch(ls - 1);
    }
    __syncthreads();
    upward(std::true_type{}, ls - 1, 0, nthr);
}

// Sums of x and y over the workgroup, in every thread (two barriers; a third
// must pass before the scratch is used again).
__device__ __forceinline__ double2 wg_sum(double x, double y, double* red, int nthr) {
    x = wave_sum63(x);
    y = wave_sum63(y);
    if ((threadIdx.x & 63) == 63) {
        red[2 * (threadIdx.x >> 6)] = x;
        red[2 * (threadIdx.x >> 6) + 1] = y;
    }
    __syncthreads();
    double2 s = make_double2(0.0, 0.0);
    for (int w = 0; w < (nthr >> 6); ++w) {
        s.x += red[2 * w];
        s.y += red[2 * w + 1];
    }
    return s;
}

// The modes first, first + stride, ... of the active list.  NC: cells of each
// colour per thread on the top level; KEEP: 2, their neighbours and couplings
// stay in registers, 1, their diagonals and reciprocals do, 0, neither.  ODD: the
// hierarchy has odd rings on some level (the others do without that code: its
// registers).
template <typename T, int NC, int KEEP, bool ODD, bool FULL>
__device__ __forceinline__ void coarse_body(const CArgs<T>& a, int first, int stride) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int nact = *a.nact;
    if (first >= nact) return;
    const int tid = threadIdx.x;
    const int nthr = __builtin_amdgcn_readfirstlane(int(blockDim.x));
    View v;
    v.b = reinterpret_cast<double*>(lds_raw);
    v.t = reinterpret_cast<double*>(lds_raw + a.oT);
    v.red = reinterpret_cast<double*>(lds_raw + a.oRed);
    double* W = reinterpret_cast<double*>(lds_raw + a.oW);
    v.w = W;
    T* P = reinterpret_cast<T*>(lds_raw + a.oP);
    T* tab = reinterpret_cast<T*>(lds_raw + a.oTab);
    v.tab = tab;
    CRec* rec = reinterpret_cast<CRec*>(lds_raw + a.oRec);
    v.rec = rec;
    double* mu = reinterpret_cast<double*>(lds_raw + a.oMu);
    v.mu = mu;
    v.lev = reinterpret_cast<const CLev*>(a.ip + a.lev);
    if (a.nc <= 64)
        for (int i = tid; i < a.nc; i += nthr) mu[i] = a.cmu[i];
    // tables, records and matrices; empty slots stay zero for the whole launch
    for (int i = tid; i < a.ntab * kTab; i += nthr) tab[i] = T(a.dp[a.tab0 + i]);
    {
        const int4* s = reinterpret_cast<const int4*>(a.ip + a.rec0);
        int4* d = reinterpret_cast<int4*>(rec);
        for (int i = tid; i < 2 * a.nrec; i += nthr) d[i] = s[i];
    }
    if (a.wlds)
        for (int i = tid; i < 2 * a.nc * a.nc; i += nthr) W[i] = a.dp[a.wt + i];
    for (int i = tid; i < a.nslot; i += nthr) P[a.oS + i] = T(0);
    const CLev L = level_at(v.lev, 0);
    T* p = P + L.p;
    T* Sl = P + L.s;
    const T* pc = P + level_at(v.lev, 1).p;
    const CRec* trec = reinterpret_cast<const CRec*>(a.ip + L.rec);
    __syncthreads();

    // the thread's cells of the top level, red then black: the records stay in
    // registers (their correction words only for the black ones)
    Raw raw[2][NC];
    if (!(ODD && L.odd)) {
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int m = 0; m < NC; ++m) {
                const int n = c ? L.n1 : L.n0;
                raw[c][m] = trec[(c ? L.n0 : 0) + min(tid + m * nthr, n - 1)].words();
            }
    }
    Cell<T> kept[2][KEEP == 2 ? NC : 1];
    if constexpr (KEEP == 2) {
        if (!(ODD && L.odd)) {
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int m = 0; m < NC; ++m) couplings(kept[c][m], v, L, raw[c][m]);
        }
    }
    T dk[2][KEEP ? NC : 1], ik[2][KEEP ? NC : 1];  // this mode's diagonals and reciprocals
    auto get = [&](int c, int m, T sig) __attribute__((always_inline)) -> Cell<T> {
        Cell<T> x;
        if constexpr (KEEP == 0) {
            cell_of(x, v, L, raw[c][m], sig);
        } else {
            if constexpr (KEEP == 2) x = kept[c][m];
            else couplings(x, v, L, raw[c][m]);
            x.d = dk[c][m];
            x.inv = ik[c][m];
        }
        return x;
    };
    // with four cells the phases run them two by two: all at once they spill
    auto apart = [&](int m) __attribute__((always_inline)) {
        if (NC > 2 && m > 0 && true) __builtin_amdgcn_sched_barrier(0);
    };
    auto at = [&](int c, int m) { return (c ? L.n0 : 0) + tid + m * nthr; };  // the cell's place
    auto mine = [&](int c, int m) { return tid + m * nthr < (c ? L.n1 : L.n0); };

    for (int item = first; item < nact; item += stride) {
        const int q = __builtin_amdgcn_readfirstlane(a.act[item]);
        const double sigd = a.shift[q];
        const T sig = T(sigd);
        const T* fq = a.fL + q * a.planeL;
        T* pq = a.pL + q * a.planeL;
        T f[2][NC], x[2][NC];
        double fn = 0.0;
        if (!(ODD && L.odd)) {
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int m = 0; m < NC; ++m) {
                    const int o = raw[c][m].self();
                    f[c][m] = fq[o];
                    x[c][m] = FULL ? pq[o] : T(0);
                    if constexpr (KEEP != 0) {
                        Cell<T> y;
                        cell_of(y, v, L, raw[c][m], sig);
                        dk[c][m] = y.d;
                        ik[c][m] = y.inv;
                    }
                }
        }
        __syncthreads();  // the last mode's reads are over
        if constexpr (FULL) {
            double fs = 0.0;
            if (!(ODD && L.odd)) {
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int m = 0; m < NC; ++m)
                        if (mine(c, m)) {
                            p[at(c, m)] = x[c][m];
                            fs += double(f[c][m]) * double(f[c][m]);
                        }
            } else {
                for (int k = tid; k < L.ncell; k += nthr) {
                    const int o = trec[k].self;
                    p[k] = pq[o];
                    fs += double(fq[o]) * double(fq[o]);
                }
            }
            fn = wg_sum(fs, 0.0, v.red, nthr).x;
            __syncthreads();
        }
        double rn = 0.0;
        const double sa = FULL ? a.sabs[q] : 0.0;
        int c = 0;
        for (;; ++c) {
            if constexpr (FULL) {
                // the test of every cycle: residual and solution over all cells
                double rs = 0.0, ps = 0.0;
                if (!(ODD && L.odd)) {
#pragma unroll
                    for (int k = 0; k < 2; ++k)
#pragma unroll
                        for (int m = 0; m < NC; ++m) {
                            const Cell<T> y = get(k, m, sig);
                            const T r = f[k][m] - (around(y, p) + y.d * x[k][m]);
                            if (mine(k, m)) {
                                rs += double(r) * double(r);
                                ps += double(x[k][m]) * double(x[k][m]);
                            }
                        }
                } else {
                    for (int k = tid; k < L.ncell; k += nthr) {
                        const CRec r = rec_of(a, v, L, k);
                        Cell<T> y;
                        cell_of(y, v, L, r.words(), sig);
                        const T z = fq[r.self] - (around(y, p) + y.d * p[k]);
                        rs += double(z) * double(z);
                        ps += double(p[k]) * double(p[k]);
                    }
                }
                const double2 sums = wg_sum(rs, ps, v.red, nthr);
                rn = sums.x;
                const double pn = sums.y;
                const bool err_ok = a.etol2 < 0.0 || 4.0 * rn <= a.etol2 * sa * sa * pn;
                if ((rn <= a.rtol2 * fn && err_ok) || c >= a.maxc) break;
            } else {
                if (c >= a.ncyc) break;
            }
            const bool zero = !FULL && c == 0;
            if (ODD && L.odd) {
                odd_down<T, true>(a, v, L, p, Sl, nullptr, 2, fq, sig, zero, tid, nthr);
            } else {
#pragma unroll
                for (int m = 0; m < NC; ++m) {
                    apart(m);
                    const Cell<T> y = get(0, m, sig);
                    const T t = zero ? f[0][m] : f[0][m] - around(y, p);
                    x[0][m] = solve_for(t, y.d, y.inv);
                    if (mine(0, m)) p[at(0, m)] = x[0][m];
                }
                __syncthreads();
#pragma unroll
                for (int m = 0; m < NC; ++m) {
                    apart(m);
                    const Cell<T> y = get(1, m, sig);
                    x[1][m] = solve_for(f[1][m] - around(y, p), y.d, y.inv);
                    if (mine(1, m)) p[at(1, m)] = x[1][m];
                }
                __syncthreads();
#pragma unroll
                for (int m = 0; m < NC; ++m) {
                    apart(m);
                    const Cell<T> y = get(0, m, sig);
                    const T w = y.rw * (f[0][m] - (around(y, p) + y.d * x[0][m]));
                    if (mine(0, m)) Sl[y.s] = w;
                }
            }
            below<T, ODD>(a, v, P, sigd, tid, nthr);
            if (ODD && L.odd) {
                odd_up<T, true>(a, v, L, p, pc, nullptr, 2, fq, sig, tid, nthr);
            } else {
#pragma unroll
                for (int m = 0; m < NC; ++m) {
                    apart(m);
                    const Cell<T> y = get(1, m, sig);
                    x[1][m] += prolong(y, pc);
                    if (mine(1, m)) p[at(1, m)] = x[1][m];
                }
                __syncthreads();
#pragma unroll
                for (int m = 0; m < NC; ++m) {
                    apart(m);
                    const Cell<T> y = get(0, m, sig);
                    x[0][m] = solve_for(f[0][m] - around(y, p), y.d, y.inv);
                    if (mine(0, m)) p[at(0, m)] = x[0][m];
                }
                __syncthreads();
#pragma unroll
                for (int m = 0; m < NC; ++m) {
                    apart(m);
                    const Cell<T> y = get(1, m, sig);
                    x[1][m] = solve_for(f[1][m] - around(y, p), y.d, y.inv);
                    if (mine(1, m)) p[at(1, m)] = x[1][m];
                }
            }
            if (FULL || c + 1 < a.ncyc) __syncthreads();
        }
        if (!(ODD && L.odd)) {
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int m = 0; m < NC; ++m)
                    if (mine(k, m)) pq[raw[k][m].self()] = x[k][m];
        } else {
            for (int k = tid; k < L.ncell; k += nthr) pq[trec[k].self] = p[k];
        }
        if (FULL && tid == 0) {
            a.cyc[q] = c;
            a.rnorm[q] = rn;
            a.fnorm[q] = fn;
        }
    }
}

}  // namespace

template <typename T, int NC, int KEEP, bool ODD, bool FULL>
__global__ void __launch_bounds__(kCoarseThreads) k_coarse(const CArgs<T> a) {
    coarse_body<T, NC, KEEP, ODD, FULL>(a, blockIdx.x, gridDim.x);
}

template <int NC, int KEEP, bool ODD>
__global__ void __launch_bounds__(kCoarseThreads) k_coarse_group(const GEnt* __restrict__ e, int n,
                                                       const CArgs<float>* __restrict__ jobs) {
    int bx, by;
    const int j = group_locate(e, n, bx, by);
    coarse_body<float, NC, KEEP, ODD, false>(jobs[j], bx, 1 << 30);
}

// ------------------------------- host side -------------------------------

namespace {

// Offset of coarse value (I, J) of block b, one cell beyond a face allowed
// (y first, as the prolongation resolves it); bit 15 set where it is negated.
unsigned short coarse_ref(const mbp_plan* P, const Level& C, int b, int I, int J) {
    bool neg = false;
    int k = b;
    auto blk = [&]() -> const DBlock& { return P->hblk[C.blk_off + k]; };
    if (J < 0) {
        if (blk().nbr[YM] >= 0) { k = blk().nbr[YM]; J = blk().ny - 1; }
        else { neg ^= blk().bc[YM] == MBP_DIRICHLET; J = 0; }
    } else if (J >= blk().ny) {
        if (blk().nbr[YP] >= 0) { k = blk().nbr[YP]; J = 0; }
        else { neg ^= blk().bc[YP] == MBP_DIRICHLET; J = blk().ny - 1; }
    }
    if (I < 0) {
        if (blk().nbr[XM] >= 0) { k = blk().nbr[XM]; I = blk().nx - 1; }
        else { neg ^= blk().bc[XM] == MBP_DIRICHLET; I = 0; }
    } else if (I >= blk().nx) {
        if (blk().nbr[XP] >= 0) { k = blk().nbr[XP]; I = 0; }
        else { neg ^= blk().bc[XP] == MBP_DIRICHLET; I = blk().nx - 1; }
    }
    return (unsigned short)((blk().off + J * blk().nx + I) | (neg ? 0x8000 : 0));
}

}  // namespace

// Records and tables of levels L .. of the plan, appended to the pools; nothing
// where the levels do not fit the form.
void coarse_build(mbp_plan* P, int L, int64_t elem) {
    CoarseInfo& ci = P->coarse;
    ci = CoarseInfo{};
    if (!coarse_fits(P, L, elem)) return;
    const Geometry& g = P->g;
    const int nl = P->nlev - L, nb = g.nb;
    std::vector<CLev> lev(nl);
    std::vector<int> patches(nl), first(nl + 1, 0);  // first record of each level
    for (int k = 0; k < nl; ++k) first[k + 1] = first[k] + int(P->levels[L + k].plane);
    std::vector<unsigned short> place(first[nl]);  // plane offset -> place in the LDS iterate
    // records go straight to the int pool, tables to the double pool
    while (P->hint.size() & 3) P->hint.push_back(0);
    const int words = int(sizeof(CRec) / sizeof(int)), r0 = int(P->hint.size());
    P->hint.resize(P->hint.size() + size_t(first[nl]) * words, 0);
    CRec* recs = reinterpret_cast<CRec*>(P->hint.data() + r0);
    ci.tab0 = int(P->hdbl.size());
    std::vector<int> pgrid;  // patches of the level above: first of each block, row pitch
    int elems = 0;
    for (int k = 0; k < nl; ++k) {
        const Level& F = P->levels[L + k];
        CLev& cl = lev[k];
        cl = CLev{};
        cl.ncell = int(F.plane);
        cl.odd = F.odd ? 1 : 0;
        cl.ns = F.odd ? 4 : 2;
        cl.p = elems;
        elems += cl.ncell;
        std::vector<int> xb(nb), yb(nb), pg(2 * nb);
        int ne = 0, np = 0;
        for (int b = 0; b < nb; ++b) { xb[b] = ne; ne += F.nx[b]; }
        for (int b = 0; b < nb; ++b) { yb[b] = ne; ne += F.ny[b]; }
        for (int b = 0; b < nb; ++b) {
            pg[2 * b] = np;
            pg[2 * b + 1] = (F.nx[b] + 1) / 2;
            np += pg[2 * b + 1] * ((F.ny[b] + 1) / 2);
        }
        const size_t t0 = P->hdbl.size();
        P->hdbl.resize(t0 + size_t(ne) * kTab, 0.0);
        cl.ltab = ci.ntab;
        ci.ntab += ne;
        const bool transfer = k + 1 < nl;
        // a ring of odd length (of one block or several) has one face whose two
        // sides would share colours: its lower side takes the extra ones
        auto ends = [&](const DBlock& d, bool& ox, bool& oy) {
            const int kx = d.nbr[XP], ky = d.nbr[YP];
            ox = kx >= 0 && ((d.par + d.nx + P->hblk[F.blk_off + kx].par) & 1);
            oy = ky >= 0 && ((d.par + d.ny + P->hblk[F.blk_off + ky].par) & 1);
        };
        // cells per colour (the coarsest level's records are read in plane order)
        int n[4] = {0, 0, 0, 0};
        if (!transfer) n[0] = cl.ncell;
        for (int b = 0; b < nb && transfer; ++b) {
            const DBlock& d = P->hblk[F.blk_off + b];
            bool ox, oy;
            ends(d, ox, oy);
            const int mx = d.nx - (ox ? 1 : 0), my = d.ny - (oy ? 1 : 0);
            n[d.par] += (mx * my + 1) / 2;
            n[d.par ^ 1] += mx * my / 2;
            for (int j = 0; j < my && ox; ++j) ++n[2 + ((mx + j + d.par) & 1)];
            for (int i = 0; i < d.nx && oy; ++i) ++n[2 + ((i + my + d.par) & 1)];
        }
        cl.n0 = n[0];
        cl.n1 = n[1];
        cl.n2 = n[2];
        cl.n3 = n[3];
        CRec* rec = recs + first[k];
        unsigned short* pl = place.data() + first[k];
        int next[4] = {0, n[0], n[0] + n[1], n[0] + n[1] + n[2]};  // places by colour
        for (int b = 0; b < nb; ++b) {
            const DBlock& d = P->hblk[F.blk_off + b];
            const DBlock* e = transfer ? &P->hblk[P->levels[L + k + 1].blk_off + b] : nullptr;
            bool ox, oy;
            ends(d, ox, oy);
            auto entry = [&](int e, int c, int n, int i, int rw, int pw) {
                double* t = &P->hdbl[t0 + size_t(e + i) * kTab];
                t[0] = P->hdbl[c + i];
                t[1] = P->hdbl[c + n + i];
                t[2] = P->hdbl[c + 2 * n + i];
                if (transfer) {
                    t[3] = P->hdbl[rw + i];
                    t[4] = P->hdbl[pw + i];
                }
            };
            for (int i = 0; i < d.nx; ++i) entry(xb[b], d.cx, d.nx, i, d.rwx, d.pwx);
            for (int j = 0; j < d.ny; ++j) entry(yb[b], d.cy, d.ny, j, d.rwy, d.pwy);
            for (int j = 0; j < d.ny; ++j)
                for (int i = 0; i < d.nx; ++i) {
                    const int self = d.off + j * d.nx + i;
                    int c = (i + j + d.par) & 1;
                    if ((ox && i == d.nx - 1) || (oy && j == d.ny - 1)) c += 2;
                    const int to = next[transfer ? c : 0]++;
                    pl[self] = (unsigned short)to;
                    CRec r{};
                    r.self = (unsigned short)self;
                    const bool inner = i > 0 && i < d.nx - 1 && j > 0 && j < d.ny - 1;
                    if (inner) {
                        r.n[0] = (unsigned short)(self - 1);
                        r.n[1] = (unsigned short)(self + 1);
                        r.n[2] = (unsigned short)(self - d.nx);
                        r.n[3] = (unsigned short)(self + d.nx);
                    }
                    auto other = [&](int f, int ii, int jj) {
                        if (ii >= 0 && ii < d.nx && jj >= 0 && jj < d.ny) return d.off + jj * d.nx + ii;
                        const int o = d.nbr[f];
                        if (o < 0) return self;
                        const DBlock& e = P->hblk[F.blk_off + o];
                        return e.off + (f == YM ? e.ny - 1 : f == YP ? 0 : j) * e.nx + (f == XM ? e.nx - 1 : f == XP ? 0 : i);
                    };
                    if (!inner) {
                        r.n[0] = (unsigned short)other(XM, i - 1, j);
                        r.n[1] = (unsigned short)other(XP, i + 1, j);
                        r.n[2] = (unsigned short)other(YM, i, j - 1);
                        r.n[3] = (unsigned short)other(YP, i, j + 1);
                        // a missing neighbour (coupling zero) stands for one that exists, of
                        // the other colour: the cell itself may not be written yet
                        int some = self;
                        for (int k4 = 0; k4 < 4; ++k4)
                            if (r.n[k4] != self) some = r.n[k4];
                        for (int k4 = 0; k4 < 4; ++k4)
                            if (r.n[k4] == self) r.n[k4] = (unsigned short)some;
                    }
                    r.xi = (unsigned short)(xb[b] + i);
                    r.yi = (unsigned short)(yb[b] + j);
                    const int patch = pg[2 * b] + (j / 2) * pg[2 * b + 1] + i / 2;
                    r.s = (unsigned short)(cl.ns == 2 ? 2 * patch + (j & 1) : 4 * patch + 2 * (j & 1) + (i & 1));
                    if (transfer) {
                        const int I = P->hint[d.pcx + i], J = P->hint[d.pcy + j];
                        if (I >= 0 && I + 1 < e->nx && J >= 0 && J + 1 < e->ny) {
                            const int at = e->off + J * e->nx + I;
                            r.c[0] = (unsigned short)at;
                            r.c[1] = (unsigned short)(at + 1);
                            r.c[2] = (unsigned short)(at + e->nx);
                            r.c[3] = (unsigned short)(at + e->nx + 1);
                        } else {
                            for (int c = 0; c < 4; ++c)
                                r.c[c] = coarse_ref(P, P->levels[L + k + 1], b, I + (c & 1), J + (c >> 1));
                        }
                    }
                    if (k > 0) {
                        const Level& U = P->levels[L + k - 1];
                        r.g = (unsigned short)(pgrid[2 * b] + j * pgrid[2 * b + 1] + i);
                        r.gp = (unsigned short)(pgrid[2 * b + 1] | (i == d.nx - 1 && U.nx[b] > 2 * d.nx ? 0x4000 : 0) |
                                                (j == d.ny - 1 && U.ny[b] > 2 * d.ny ? 0x8000 : 0));
                    }
                    rec[to] = r;
                }
        }
        pgrid = pg;
        patches[k] = np;
    }
    // neighbours and coarse values by place
    for (int k = 0; k < nl; ++k) {
        const unsigned short* pl = place.data() + first[k];
        const unsigned short* below = k + 1 < nl ? place.data() + first[k + 1] : nullptr;
        for (int i = first[k]; i < first[k + 1]; ++i) {
            for (unsigned short& o : recs[i].n) o = pl[o];
            if (below)
                for (unsigned short& o : recs[i].c) o = (unsigned short)((o & 0x8000) | below[o & 0x7fff]);
        }
    }
    // threads: two cells of each colour each, or as many as kCoarseThreads threads need
    const int n = std::max(lev[0].n0, lev[0].n1);
    ci.ncell = n;
    ci.nthr = coarse_threads(n);
    ci.per = n <= 2 * ci.nthr ? 2 : 4;
    for (const CLev& c : lev) ci.odd |= c.odd;
    ci.oS = elems;
    for (int k = 0; k + 1 < nl; ++k) {
        lev[k].s = elems;
        elems += lev[k].ns * patches[k];
    }
    ci.nslot = elems - ci.oS;
    // records in LDS from the second level on where that costs no workgroup of
    // the CU (its 8 waves of this kernel), else from the third
    const int64_t share = P->lds_limit / std::max(1, kCoarseThreads / ci.nthr);
    const int first_rec = coarse_lds_need(P, L, elem) + int64_t(lev[1].ncell) * 32 <= share ? 1 : 2;
    for (int k = 0; k < nl; ++k) {
        lev[k].rec = r0 + first[k] * words;
        if (k == first_rec) ci.rec0 = lev[k].rec;
        lev[k].lrec = k >= first_rec ? ci.nrec : -1;
        if (k >= first_rec) ci.nrec += lev[k].ncell;
    }
    ci.lev = int(P->hint.size());
    for (const CLev& c : lev) {
        const int* s = reinterpret_cast<const int*>(&c);
        P->hint.insert(P->hint.end(), s, s + sizeof(CLev) / sizeof(int));
    }
    const int nc = P->coarse_n;
    ci.wt = int(P->hdbl.size());
    if (nc <= 64)  // transposed: a lane reads column k of the product's row j
        for (const std::vector<double>* w : {&P->coarse_wr, &P->coarse_wl})
            for (int j = 0; j < nc; ++j)
                for (int k = 0; k < nc; ++k) P->hdbl.push_back((*w)[size_t(k) * nc + j]);
    ci.nl = nl;
    ci.ls = nl;
    if (nc <= 64) {
        ci.ls = nl - 1;
        while (ci.ls > 1 && std::max(lev[ci.ls - 1].n0, lev[ci.ls - 1].n1) <= 64) --ci.ls;
    }
    ci.wlds = nc <= kCoarseInLds ? 1 : 0;
    auto up16 = [](int64_t x) { return (x + 15) & ~int64_t(15); };
    int64_t o = up16(int64_t(nc) * 8);
    ci.oT = int(o);
    o += up16(int64_t(nc) * 8);
    ci.oRed = int(o);
    o += 128;
    ci.oMu = int(o);
    if (nc <= 64) o += up16(int64_t(nc) * 8);
    ci.oW = int(o);
    if (ci.wlds) o += 2 * int64_t(nc) * nc * 8;
    ci.oP = int(o);
    o = up16(o + elems * elem);
    ci.oTab = int(o);
    o = up16(o + int64_t(ci.ntab) * kTab * elem);
    ci.oRec = int(o);
    o += int64_t(ci.nrec) * 32;
    ci.bytes = o;
    ci.ok = 1;
}

namespace {

template <typename T>
CArgs<T> coarse_args(const mbp_plan* P, int L, T* pL, const T* fL, const int* act, const int* nact) {
    const CoarseInfo& ci = P->coarse;
    CArgs<T> a{};
    a.ip = P->d_int;
    a.dp = P->d_dbl;
    a.lev = ci.lev;
    a.nl = ci.nl;
    a.ls = ci.ls;
    a.nc = P->coarse_n;
    a.cwl = P->d_cwl;
    a.cwr = P->d_cwr;
    a.cmu = P->d_cmu;
    for (double mu : P->coarse_mu) a.cmumax = std::max(a.cmumax, std::fabs(mu));
    a.wt = ci.wt;
    a.wlds = ci.wlds;
    a.oT = ci.oT;
    a.oRed = ci.oRed;
    a.oMu = ci.oMu;
    a.oW = ci.oW;
    a.oP = ci.oP;
    a.oTab = ci.oTab;
    a.oRec = ci.oRec;
    a.nslot = ci.nslot;
    a.oS = ci.oS;
    a.tab0 = ci.tab0;
    a.ntab = ci.ntab;
    a.rec0 = ci.rec0;
    a.nrec = ci.nrec;
    a.pL = pL;
    a.fL = fL;
    a.planeL = P->levels[L].plane;
    a.shift = P->d_shift;
    a.act = act;
    a.nact = nact;
    a.ncyc = 1;
    return a;
}

// Workgroups of a kernel on the chip at once (taken once per kernel, threads,
// LDS size and device), with the kernel's LDS limit raised on the way.
int coarse_slots(const void* kernel, int nthr, size_t lds) {
    static std::mutex mu;
    static std::map<std::pair<std::pair<int, const void*>, std::pair<int, size_t>>, int> cache;
    int dev = 0;
    (void)hipGetDevice(&dev);
    std::lock_guard<std::mutex> lock(mu);
    const auto key = std::make_pair(std::make_pair(dev, kernel), std::make_pair(nthr, lds));
    auto it = cache.find(key);
    if (it != cache.end()) return it->second;
    int most = 0, per_cu = 0, ncu = 0;
    if (hipDeviceGetAttribute(&most, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess)
        (void)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, most);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, nthr, lds) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        per_cu = 1;
        ncu = 256;
    }
    return cache[key] = std::max(1, per_cu) * std::max(1, ncu);
}

template <typename T, int NC, int KEEP, bool ODD, bool FULL>
void launch(const mbp_plan* P, const CArgs<T>& a, int nitems, hipStream_t s) {
    const void* fn = reinterpret_cast<const void*>(k_coarse<T, NC, KEEP, ODD, FULL>);
    const CoarseInfo& ci = P->coarse;
    const int slots = coarse_slots(fn, ci.nthr, size_t(ci.bytes));
    // modes per workgroup: equal shares of the rounds the chip needs anyway
    const int per = (nitems + slots - 1) / slots, grid = (nitems + per - 1) / per;
    hipLaunchKernelGGL((k_coarse<T, NC, KEEP, ODD, FULL>), dim3(grid), dim3(ci.nthr), size_t(ci.bytes), s, a);
}

// What stays in registers is what fits 256 of them.
template <typename T, bool FULL>
void launch_form(const mbp_plan* P, const CArgs<T>& a, int nitems, hipStream_t s) {
    constexpr bool F32 = sizeof(T) == 4;
    if (P->coarse.odd) launch<T, 4, 0, true, FULL>(P, a, nitems, s);
    else if (P->coarse.per == 2) launch<T, 2, F32 ? 2 : 1, false, FULL>(P, a, nitems, s);
    else launch<T, 4, F32 ? 1 : 0, false, FULL>(P, a, nitems, s);
}

}  // namespace

template <typename T>
void launch_coarse(const mbp_plan* P, int L, T* pL, const T* fL, int ncyc, const int* act, const int* nact, int nitems,
                   hipStream_t s) {
    CArgs<T> a = coarse_args<T>(P, L, pL, fL, act, nact);
    a.ncyc = ncyc;
    launch_form<T, false>(P, a, nitems, s);
}
template void launch_coarse<double>(const mbp_plan*, int, double*, const double*, int, const int*, const int*, int,
                                    hipStream_t);
template void launch_coarse<float>(const mbp_plan*, int, float*, const float*, int, const int*, const int*, int,
                                   hipStream_t);

void launch_coarse_full(const mbp_plan* P, double* p, const double* f, const int* act, const int* nact, int nitems, int maxc,
                        double rtol2, double etol2, int* cyc, double* rnorm, double* fnorm, hipStream_t s) {
    CArgs<double> a = coarse_args<double>(P, 0, p, f, act, nact);
    a.sabs = P->d_sabs;
    a.maxc = maxc;
    a.rtol2 = rtol2;
    a.etol2 = etol2;
    a.cyc = cyc;
    a.rnorm = rnorm;
    a.fnorm = fnorm;
    launch_form<double, true>(P, a, nitems, s);
}

// The LDS stage of the problems of one form (0: two cells of a colour per thread,
// 1: four, 2: odd rings), one launch: threads and LDS of the largest.  A hierarchy that
// fits LDS whole runs all of its inner cycles in the launch of the first (k = 0), as
// alone; every launch starts from zero.
GStage group_coarse32(GroupBlob& gb, const std::vector<SolveCtx*>& cs, int form, int k, int inner) {
    std::vector<CArgs<float>> jobs;
    std::vector<int> gx, gy;
    GStage st;
    int64_t bytes = 0;
    int nthr = 64;
    for (const SolveCtx* c : cs) {
        const mbp_plan* P = c->P;
        if (!P->coarse.ok || (P->coarse.odd ? 2 : P->coarse.per == 2 ? 0 : 1) != form) continue;
        const int L = P->lds_level32;
        if (L == 0 && k > 0) continue;
        CArgs<float> a = coarse_args<float>(P, L, P->p32[L], P->f32[L], P->d_act, P->d_nact);
        if (L == 0) a.ncyc = inner;
        jobs.push_back(a);
        gx.push_back(c->nitems);
        gy.push_back(1);
        bytes = std::max(bytes, P->coarse.bytes);
        nthr = std::max(nthr, P->coarse.nthr);
    }
    if (!jobs.empty()) st = group_build(gb, G_COARSE0 + form, jobs, gx, gy);
    st.kind = G_COARSE0 + form;
    st.lds = size_t(bytes);
    st.threads = nthr;
    if (!jobs.empty())
        (void)coarse_slots(form == 0   ? reinterpret_cast<const void*>(k_coarse_group<2, 2, false>)
                           : form == 1 ? reinterpret_cast<const void*>(k_coarse_group<4, 1, false>)
                                       : reinterpret_cast<const void*>(k_coarse_group<4, 0, true>),
                           nthr, size_t(bytes));
    return st;
}

void group_launch_coarse(const GStage& st, const unsigned char* dev, hipStream_t s) {
    if (st.wgs <= 0) return;
    const GEnt* e = reinterpret_cast<const GEnt*>(dev + st.ent_off);
    const CArgs<float>* j = reinterpret_cast<const CArgs<float>*>(dev + st.job_off);
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(st.wgs), dim3(st.threads), st.lds, s, e, st.nent, j); };
    if (st.kind == G_COARSE0) go(k_coarse_group<2, 2, false>);
    else if (st.kind == G_COARSE0 + 1) go(k_coarse_group<4, 1, false>);
    else go(k_coarse_group<4, 0, true>);
}

}  // namespace mbp
