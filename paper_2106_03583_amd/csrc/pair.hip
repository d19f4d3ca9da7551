// Pair march: the red-black sweeps of the global-memory levels with two
// neighbouring cells per lane, all in registers.
//
// One wave owns a strip of one block and one mode: 128 columns (two per
// lane), of which the outer ones are halo, and a run of rows.  It marches down
// the strip with a ring of rows in registers; row k arrives while the stages
// below it work on rows k-1, k-2, ... of the same step:
//   A  pre-smoothing sweep (red row k-1, black row k-2),
//   C  bilinear coarse-grid correction (row k-3) and the post-smoothing sweep
//      (red k-4, black k-5); row k-5 is then the cycle's iterate and is stored,
//   B  the next cycle's pre-smoothing sweep (red k-6, black k-7),
//   R  residual of row k-8 (k-3 without C and B), area-weighted and summed
//      into the coarse rhs.
// Three forms: PRE = A R, POST = A C, CYCLE = A C B R.  The pre-smoothed iterate
// is never stored: whoever needs it smooths the stored iterate again, which
// costs arithmetic the memory-bound march has to spare, so a V-cycle reads p, f
// and the coarse correction and writes p and the coarse rhs once on the finest
// level (28 B per FP64 cell in one launch instead of 52 B in two), and reads f
// twice, the correction once and writes p and the coarse rhs once on a coarse
// level (28 B instead of 44 B).
//
// Why two cells per lane: the cells of one colour in a row are then one slot
// of every lane, so a colour's relaxation is one full-width pass per row, one
// x neighbour is in the lane and the other one DPP shift away.  No barrier and
// no LDS traffic in the dependent chain; LDS holds only the coefficient tables
// (per strip: x per row region and lane, y per column region and row), so that
// lanes in neighbouring blocks, walls and cells that do not exist take no
// branches: a missing cell has zero couplings and a huge diagonal and stays 0.
// Loads are buffer loads whose out-of-range lanes return 0.
//
// The last sweep of an FP32 correction solve (ADD) adds its rows to the FP64 iterate:
// 25 B a cell instead of 13 B and a pass of 20 B that read them again (eight-block
// obstacle: 94 + 41 -> 106 us a refinement step).  Four FP64 rows ahead, and six of p
// and f instead of eight, as eight of both spilled: 7 % slower than two passes.
//
// What bounds it: memory.  512 x 512 x 1024 box, FP64, all 1024 modes: the first
// cycle launch moves 20 B per cell in 1.32 ms (4.1 TB/s; a device copy reaches
// 4.9), the later ones 28 B at 4.3 TB/s; the two strip launches they replace
// (k_tile, k_tile_corr) took 2.1 ms together on the average of the solve's
// active sets against 0.99 ms for the cycle form.  Whole solves before and
// after: box 51.3 -> 27.8 ms, three-block L-shape 3 x 256^2 x 512 25.7 -> 13.5 ms,
// eight-block obstacle (mixed) 12.5 -> 7.0 ms, 24 uneven boxes in one mixed batch
// 31.8 -> 18.7 ms.
//
// Levels qualify when every block has at least 8 cells both ways and odd counts end
// at walls (pairs and coarse cells then align in every block, and the halo stays
// inside the neighbour); the strip kernels of march.hip run the others.  An odd
// count leaves one cell alone in the last lane, or row, as the third child of the
// last coarse cell: forms of their own (ODD), since what they add (a masked store a
// row, a shift in the restriction, a select in the interpolation) costs even planes
// registers.  203 x 157, 90 modes: 34 + 41 us of strip sweeps a cycle -> 40 us, a
// lockstep solve 2.20 -> 1.51 ms.
#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>
#include <utility>

#include "internal.h"
#include "wave.h"

namespace mbp {

// One strip: geometry and the places of its tables.
struct PTile {
    int x0, w, y0, y1;     // output columns and rows of the block
    int bnx, bny, off;     // block size, first cell in the plane
    int ncx, ncy, coff;    // the same of the next level
    int xt, yt, ot;        // x table, y table (double pool), offsets (int pool)
    int hl;                // halo lanes on each side
    int pad[2];
};

namespace {

constexpr int kRing = 16;        // register rows (static indices: the march is unrolled over the ring)
constexpr int kPad = 24;         // rows of the y tables beyond each end of the block
constexpr int kUp = 18;          // rows of the LDS copy above the strip's first
constexpr int kDown = 8;         // and below its last
constexpr int kYw = 6;           // y table: ym, yp, yd, restriction weight, prolongation weights lo, hi
constexpr int kXw = 3 * 2 * 64 * 2, kXd = 3 * 2 * 64, kXp = 3 * 64 * 4, kXr = 2 * 64;
constexpr int kXTab = kXw + kXd + kXp + kXr;  // x table: couplings, diagonals, prolongation, restriction
constexpr int kOTab = 3 * 64 * 4;             // offsets: base, stride, coarse base, coarse stride
constexpr int kNoCell = -0x7fffffff - 1;
constexpr unsigned kDead = 0x7fff0000u;  // byte offset past every plane (the host keeps planes below 2^30 bytes)

}  // namespace

template <typename T>
struct PArgs {
    const PTile* tiles;
    int ntiles;
    const double* dp;
    const int* ip;
    T* pa;              // iterate in / out: pa -> pb, or pb -> pa when *cycle says so
    T* pb;
    const int* cycle;   // convergence tests so far (nullptr: pa -> pb): the V-cycle after test t
                        // reads buffer (t - 1) & 1, so a recorded graph replays correctly
    const T* f;
    const T* ec;        // coarse correction
    T* fc;              // coarse rhs
    long long plane, plane_c;
    const double* shift;
    const int* act;
    const int* nact;
    double* part;       // per (mode, strip) squared residual and solution
    int* nparts;        // strips of this launch, for the reduction
    double* sum;        // ADD: the FP64 iterate that takes the result (its plane as of p)
    int first;          // ADD: it is zero so far and need not be read
};

namespace {

template <typename T>
struct alignas(2 * sizeof(T)) Pr {
    T v[2];
};
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const void* p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, int(bytes), 0x00020000);
}
__device__ __forceinline__ Pr<double> load_pair(__amdgpu_buffer_rsrc_t r, unsigned o, double) {
    return __builtin_bit_cast(Pr<double>, __builtin_amdgcn_raw_buffer_load_b128(r, int(o), 0, 0));
}
__device__ __forceinline__ Pr<float> load_pair(__amdgpu_buffer_rsrc_t r, unsigned o, float) {
    return __builtin_bit_cast(Pr<float>, __builtin_amdgcn_raw_buffer_load_b64(r, int(o), 0, 0));
}
__device__ __forceinline__ double load_one(__amdgpu_buffer_rsrc_t r, unsigned o, double) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, int(o), 0, 0));
}
__device__ __forceinline__ float load_one(__amdgpu_buffer_rsrc_t r, unsigned o, float) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, int(o), 0, 0));
}
// The whole offset goes in the vector operand: with a scalar offset register
// beside it the compiler lets the data registers of a 16-byte store be
// overwritten at once, and such stores wrote wrong values here.
__device__ __forceinline__ void store_pair(__amdgpu_buffer_rsrc_t r, unsigned o, Pr<double> v) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, int(o), 0, 0);
}
__device__ __forceinline__ void store_pair(__amdgpu_buffer_rsrc_t r, unsigned o, Pr<float> v) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, int(o), 0, 0);
}
__device__ __forceinline__ void store_one(__amdgpu_buffer_rsrc_t r, unsigned o, double v) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, int(o), 0, 0);
}
__device__ __forceinline__ void store_one(__amdgpu_buffer_rsrc_t r, unsigned o, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, int(o), 0, 0);
}

// The march of one wave.  FORM bits: see the file comment.
enum { kPre = 0, kPost = 1, kCycle = 2 };

// ADD (FP32, the last sweep of a correction solve): the result is added to the FP64
// iterate instead of being stored; the iterate's rows are loaded kSum steps ahead.
template <typename T, int FORM, bool ZIN, bool NRM, bool ADD = false, bool ODD = false>
struct March {
    static constexpr bool C = FORM != kPre, R = FORM != kPost;
    // rows loaded ahead: at most the ring minus the rows the last stage still reads.  Six
    // in the odd forms too: with eight, hipcc 7.2 overwrites the black value of one row of
    // the sixteen in the FP32 PRE form from zero before its only use (following every
    // loaded register of that form through its assembly: row 5's upper half has no
    // reader; with six, and in the even forms, every one has), and two of eight
    // restricted rows were wrong.  tests/test_gpu_cycle_cells.py holds every form to a
    // single cycle's values, cell by cell.
    static constexpr int kAhead = FORM == kCycle || ADD || ODD ? 6 : 8;

    // strip constants
    int lane, y0, y1, bny, ncy, kend;
    unsigned out_p, out_c, row_p, row_c;  // byte offsets of the lane's output cells and row pitches
    const T* yb;        // the lane's y table at the current base row
    const T* sXw;
    const T* sXd;
    const T* sW;
    T sig, wr0, wr1;
    __amdgpu_buffer_rsrc_t rp, rq, rf, re, rc;
    bool outl;
    // ODD (some block's count is odd): the last coarse cell of such a row or column
    // has three children, the third alone in its lane (row)
    bool oy, out1, lastc;   // odd rows; both cells of the lane are output; lane of the last coarse cell
    unsigned out_1;         // the lone cell
    // moving state
    int kc;                               // row of ring slot 0
    Pr<T> p[kRing], f[kRing];
    Pr<T> xlo, xhi;
    T e[4];
    unsigned vo, vs, vo1, vs1, vo2, vs2;  // next row to load: offset, pitch; the same past each face
    unsigned co, cs, co1, cs1, co2, cs2;  // coarse rows
    T acc;
    double nrm, pnr;
    static constexpr int kSum = 4;
    __amdgpu_buffer_rsrc_t rsl, rss;      // ADD: the FP64 plane, for loads and stores
    unsigned out_s, row_s;
    Pr<double> sum[kSum];

    static __device__ __forceinline__ unsigned pick(bool c, unsigned a, unsigned b) { return c ? a : b; }
    __device__ __forceinline__ bool inside(int r) const { return (r >= y0) & (r < y1); }
    __device__ __forceinline__ int region(int r, int n) const { return (r >= 0) + (r >= n); }

    // The compiler may keep a row's coefficients and reciprocals from one step
    // for the next stages that need them; the cycle form has no registers for
    // that, so each of its steps reads through an offset the compiler cannot
    // see through (kFresh).
    static constexpr bool kFresh = FORM == kCycle;
    int z;

    // off-diagonal sum of the row at lag LAG, slot S, and its diagonal
    template <int U, int LAG, int S>
    __device__ __forceinline__ T around(T& d) const {
        constexpr int i = (U - LAG) & (kRing - 1), up = (i + 1) & (kRing - 1), dn = (i - 1) & (kRing - 1);
        const int rr = region(kc + U - LAG, bny);
        const T* y = yb + kYw * (U - LAG) + z;
        const Pr<T> xw = *reinterpret_cast<const Pr<T>*>(sXw + ((rr * 2 + S) * 64 + lane) * 2 + z);
        const Pr<T> yw = *reinterpret_cast<const Pr<T>*>(y);
        d = sXd[(rr * 2 + S) * 64 + lane + z] + y[2] + sig;
        const T l = S == 0 ? from_left(p[i].v[1]) : p[i].v[0];
        const T r = S == 0 ? p[i].v[1] : from_right(p[i].v[0]);
        return xw.v[0] * l + xw.v[1] * r + yw.v[0] * p[dn].v[S] + yw.v[1] * p[up].v[S];
    }
    // the same where every p around is zero: the diagonal only
    template <int U, int LAG, int S>
    __device__ __forceinline__ T diag() const {
        const int rr = region(kc + U - LAG, bny);
        return sXd[(rr * 2 + S) * 64 + lane + z] + (yb + kYw * (U - LAG) + z)[2] + sig;
    }
    template <int U, int LAG, int S>
    __device__ __forceinline__ void relax() {
        constexpr int i = (U - LAG) & (kRing - 1);
        T d;
        const T o = around<U, LAG, S>(d);
        p[i].v[S] = div_nr(f[i].v[S] - o, d);
    }

    __device__ __forceinline__ void advance_load(int k, unsigned& o) {
        // offset of row k for this lane; rows past the last one needed are not read
        // (pick takes values: a conditional on members would select addresses
        // and keep the whole state in memory)
        vo = pick(k == 0, vo1, pick(k == bny, vo2, vo + vs));
        vs = pick(k == 0, vs1, pick(k == bny, vs2, vs));
        o = pick(k > kend, kDead, vo);
    }
    __device__ __forceinline__ void advance_coarse(int j, unsigned& o) {
        co = pick(j == 0, co1, pick(j == ncy, co2, co + cs));
        cs = pick(j == 0, cs1, pick(j == ncy, cs2, cs));
        o = co;
    }

    template <int U>
    __device__ __forceinline__ bool step() {
        constexpr int M = kRing - 1;
        constexpr int S0 = U & 1, S1 = S0 ^ 1;
        const int k = kc + U;
        if (S0 == 0 && k > kend) return false;
        z = 0;
        if constexpr (kFresh) asm volatile("v_mov_b32 %0, 0" : "=v"(z));
        // A: red cells of row k-1 (slot (k-1) & 1), black cells of row k-2
        if constexpr (ZIN) {
            constexpr int i = (U - 1) & M;
            p[i].v[S1] = div_nr(f[i].v[S1], diag<U, 1, S1>());
            p[i].v[S0] = T(0);
        } else {
            relax<U, 1, S1>();
        }
        relax<U, 2, S1>();
        if constexpr (C) {
            // coarse rows: a new one every second row, x-interpolated once
            if constexpr (S0 == 0) {
                constexpr int ie = (U >> 1) & 3;
                const int j = (k - 2) >> 1;
                const T* w = sW + (region(j, ncy) * 64 + lane) * 4;
                const Pr<T> w0 = *reinterpret_cast<const Pr<T>*>(w), w1 = *reinterpret_cast<const Pr<T>*>(w + 2);
                const T l = from_left(e[ie]);
                T r = from_right(e[ie]);
                if (ODD) r = lastc ? l : r;
                // (the last two rows of an odd count lie between the last two coarse rows)
                if (!ODD || !(oy & (j >= ncy))) {
                    xlo = xhi;
                    xhi.v[0] = w0.v[0] * l + w0.v[1] * e[ie];
                    xhi.v[1] = w1.v[0] * e[ie] + w1.v[1] * r;
                }
                unsigned o;
                advance_coarse(j + 4, o);
                e[ie] = load_one(re, o, T(0));
            }
            {
                constexpr int i = (U - 3) & M;
                const Pr<T> w = *reinterpret_cast<const Pr<T>*>(yb + kYw * (U - 3) + 4 + z);
#pragma unroll
                for (int s = 0; s < 2; ++s) p[i].v[s] += w.v[0] * xlo.v[s] + w.v[1] * xhi.v[s];
            }
            relax<U, 4, S0>();
            relax<U, 5, S0>();
            {
                constexpr int i = (U - 5) & M;
                const int r = k - 5;
                const bool in = inside(r);
                if constexpr (ADD) {
                    constexpr int w = (U - 5) & (kSum - 1);
                    Pr<double> v = sum[w];
                    v.v[0] += double(p[i].v[0]);
                    v.v[1] += double(p[i].v[1]);
                    if (ODD) {
                        store_pair(rss, pick(in & out1, out_s + unsigned(max(r, 0)) * row_s, kDead), v);
                        store_one(rss, pick(in & (out_1 != kDead), out_s + unsigned(max(r, 0)) * row_s, kDead), v.v[0]);
                    } else {
                        store_pair(rss, pick(in, out_s + unsigned(max(r, 0)) * row_s, kDead), v);
                    }
                    const int n = r + kSum;
                    sum[w] = load_pair(rsl, pick(inside(n), out_s + unsigned(max(n, 0)) * row_s, kDead), 0.0);
                } else {
                    store_pair(rq, pick(in, out_p + unsigned(max(r, 0)) * row_p, kDead), p[i]);
                    if (ODD) store_one(rq, pick(in, out_1 + unsigned(max(r, 0)) * row_p, kDead), p[i].v[0]);
                }
                if (NRM) {
                    const T a = p[i].v[0], b = p[i].v[1];
                    const T sum = a * a + (ODD && !out1 ? T(0) : b * b);
                    pnr += double((in & outl) ? sum : T(0));
                }
            }
        }
        if constexpr (FORM == kCycle) {
            {
                // the red residual of the stored iterate is what its next
                // relaxation removes: f - off - d p (the black cells, relaxed
                // last, solve their own equations to rounding)
                constexpr int i = (U - 6) & M;
                T d;
                const T o = around<U, 6, S0>(d);
                const T t = f[i].v[S0] - o;
                if (NRM) {
                    const int r = k - 6;
                    const T res = t - d * p[i].v[S0];
                    const T sq = res * res;
                    nrm += double((inside(r) & (ODD && S0 == 1 ? out1 : outl)) ? sq : T(0));
                }
                p[i].v[S0] = div_nr(t, d);
            }
            relax<U, 7, S0>();
        }
        if constexpr (R) {
            // black residuals are rounding: the restriction takes the red cell
            // of each row, two rows a coarse cell
            constexpr int LAG = FORM == kCycle ? 8 : 3;
            constexpr int S = FORM == kCycle ? S0 : S1;
            constexpr int i = (U - LAG) & M;
            T d;
            const T o = around<U, LAG, S>(d);
            T w = (f[i].v[S] - o - d * p[i].v[S]) * (S == 0 ? wr0 : wr1) * (yb + kYw * (U - LAG) + z)[3];
            const int r = k - LAG;
            const bool in = inside(r);
            if constexpr (S == 0) {
                if (ODD) {
                    const T third = from_right(w);
                    w += lastc ? third : T(0);
                    const bool end = oy & (r == bny - 1);  // third row of the last coarse cell
                    store_one(rc, pick(in & end, out_c + unsigned(max((r >> 1) - 1, 0)) * row_c, kDead), acc + w);
                }
                acc = w;  // even row: the coarse cell's first
            } else {
                acc += w;
                const bool more = ODD && (oy & (r == bny - 2));
                store_one(rc, pick(in & !more, out_c + unsigned(max(r >> 1, 0)) * row_c, kDead), acc);
            }
        }
        // row k + kAhead takes the slot of a row no stage reads any more
        {
            constexpr int i = (U + kAhead) & M;
            unsigned o;
            advance_load(k + kAhead, o);
            if (!ZIN) p[i] = load_pair(rp, o, T(0));
            f[i] = load_pair(rf, o, T(0));
        }
        return true;
    }

    template <int... U>
    __device__ __forceinline__ bool steps(std::integer_sequence<int, U...>) {
        return (step<U>() && ...);
    }
    template <int U>
    __device__ __forceinline__ void preload_row() {
        p[U] = f[U] = Pr<T>{{T(0), T(0)}};
        if constexpr (U < kAhead) {
            unsigned o = vo;
            if constexpr (U > 0) advance_load(kc + U, o);
            if constexpr (!ZIN) p[U] = load_pair(rp, o, T(0));
            f[U] = load_pair(rf, o, T(0));
        }
    }
    template <int... U>
    __device__ __forceinline__ void preload(std::integer_sequence<int, U...>) {
        (preload_row<U>(), ...);
    }
    template <int I>
    __device__ __forceinline__ void preload_coarse(int j0) {
        unsigned o = co;
        if constexpr (I > 0) advance_coarse(j0 + I, o);
        e[I] = load_one(re, o, T(0));
    }
};

template <typename T>
__host__ __device__ constexpr size_t pair_lds_bytes(int rows, bool corr) {
    return (size_t(kXw + kXd + (corr ? kXp : 0)) + 3 * size_t(rows + kUp + kDown) * kYw) * sizeof(T);
}

template <typename T, int FORM, bool ZIN, bool NRM, bool ADD = false, bool ODD = false>
__device__ __forceinline__ void pair_body(const PArgs<T>& a, int bx, int by) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int nact = *a.nact;
    if (4 * by >= nact) return;
    const PTile t = wave_uniform(a.tiles[bx]);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr bool C = FORM != kPre;
    const int nrows = t.y1 - t.y0 + kUp + kDown;
    T* sXw = reinterpret_cast<T*>(lds_raw);
    T* sXd = sXw + kXw;
    T* sW = sXd + kXd;
    T* sY = sW + (C ? kXp : 0);
    const double* xt = a.dp + t.xt;
    for (int i = threadIdx.x; i < kXw + kXd + (C ? kXp : 0); i += 256) sXw[i] = T(xt[i]);
    const int ycol = (t.bny + 2 * kPad) * kYw, yn = nrows * kYw;
    for (int c = 0; c < 3; ++c) {
        const double* yt = a.dp + t.yt + c * ycol + (t.y0 - kUp + kPad) * kYw;
        for (int i = threadIdx.x; i < yn; i += 256) sY[c * yn + i] = T(yt[i]);
    }
    __syncthreads();
    const int mi = 4 * by + wave;
    if (a.nparts && bx == 0 && by == 0 && threadIdx.x == 0) *a.nparts = a.ntiles;
    if (mi >= nact) return;
    const int q = __builtin_amdgcn_readfirstlane(a.act[mi]);

    March<T, FORM, ZIN, NRM, ADD, ODD> m;
    m.lane = lane;
    m.y0 = t.y0;
    m.y1 = t.y1;
    m.bny = t.bny;
    m.ncy = t.ncy;
    m.kc = t.y0 - (FORM == kCycle ? 8 : 4);
    // last row to arrive: the last stage's lag below the strip's last row
    m.kend = t.y1 - 1 + (FORM == kCycle ? 8 : FORM == kPost ? 5 : 3);
    const int c0 = t.x0 - 2 * t.hl + 2 * lane;
    const int cr = c0 < 0 ? 0 : (c0 < t.bnx ? 1 : 2);
    m.yb = sY + cr * yn + (m.kc - t.y0 + kUp) * kYw;
    m.sXw = sXw;
    m.sXd = sXd;
    m.sW = sW;
    m.sig = T(a.shift[q]);
    const double* wr = xt + kXw + kXd + kXp + 2 * lane;
    m.wr0 = T(wr[0]);
    m.wr1 = T(wr[1]);
    m.outl = c0 >= t.x0 && c0 < t.x0 + t.w;
    constexpr unsigned sz = sizeof(T);
    m.out_p = m.outl ? unsigned(t.off + c0) * sz : kDead;
    m.out_c = m.outl ? unsigned(t.coff + (c0 >> 1)) * sz : kDead;
    m.row_p = unsigned(t.bnx) * sz;
    if (ODD) {
        const bool ox = t.bnx & 1, lone = ox & (c0 == t.bnx - 1);
        m.oy = t.bny & 1;
        m.out1 = m.outl & !lone;
        m.lastc = ox & (c0 == t.bnx - 3);
        m.out_1 = m.outl & lone ? m.out_p : kDead;
        m.out_p = lone ? kDead : m.out_p;
        m.out_c = lone ? kDead : m.out_c;
    }
    m.row_c = unsigned(t.ncx) * sz;
    const unsigned pbytes = unsigned(a.plane) * sz, cbytes = unsigned(a.plane_c) * sz;
    const bool swap = a.cycle ? ((*a.cycle - 1) & 1) != 0 : false;
    const long long qo = q * a.plane, qc = q * a.plane_c;
    if (!ZIN) m.rp = plane_rsrc((swap ? a.pb : a.pa) + qo, pbytes);
    if (C && !ADD) m.rq = plane_rsrc((swap ? a.pa : a.pb) + qo, pbytes);
    m.rf = plane_rsrc(a.f + qo, pbytes);
    if (C) m.re = plane_rsrc(a.ec + qc, cbytes);
    if (FORM != kPost) m.rc = plane_rsrc(a.fc + qc, cbytes);
    if constexpr (ADD) {
        // (the first rows are loaded by the steps before the strip's first)
        m.rsl = plane_rsrc(a.sum + qo, a.first ? 0u : unsigned(a.plane) * 8u);
        m.rss = plane_rsrc(a.sum + qo, unsigned(a.plane) * 8u);
        m.out_s = m.outl ? unsigned(t.off + c0) * 8u : kDead;
        m.row_s = unsigned(t.bnx) * 8u;
#pragma unroll
        for (int i = 0; i < m.kSum; ++i) m.sum[i] = Pr<double>{{0.0, 0.0}};
    }
    // row offsets of the lane in each row region
    {
        const int4* ot = reinterpret_cast<const int4*>(a.ip + t.ot);
        const int4 o0 = ot[lane], o1 = ot[64 + lane], o2 = ot[128 + lane];
        auto at = [&](const int4& o, int k) { return o.x == kNoCell ? kDead : unsigned(o.x + k * o.y) * sz; };
        auto pitch = [&](const int4& o) { return o.x == kNoCell ? 0u : unsigned(o.y) * sz; };
        auto cat = [&](const int4& o, int k) { return o.x == kNoCell ? kDead : unsigned(o.z + k * o.w) * sz; };
        auto cpitch = [&](const int4& o) { return o.x == kNoCell ? 0u : unsigned(o.w) * sz; };
        m.vo1 = at(o1, 0);
        m.vs1 = pitch(o1);
        m.vo2 = at(o2, t.bny);
        m.vs2 = pitch(o2);
        const bool below = m.kc < 0;
        m.vo = below ? at(o0, m.kc) : at(o1, m.kc);
        m.vs = below ? pitch(o0) : m.vs1;
        if (C) {
            const int j0 = (m.kc - 2) >> 1;
            m.co1 = cat(o1, 0);
            m.cs1 = cpitch(o1);
            m.co2 = cat(o2, t.ncy);
            m.cs2 = cpitch(o2);
            m.co = j0 < 0 ? cat(o0, j0) : cat(o1, j0);
            m.cs = j0 < 0 ? cpitch(o0) : m.cs1;
            m.template preload_coarse<0>(j0);
            m.template preload_coarse<1>(j0);
            m.template preload_coarse<2>(j0);
            m.template preload_coarse<3>(j0);
        }
    }
    m.xlo = m.xhi = Pr<T>{{T(0), T(0)}};
    m.acc = T(0);
    m.nrm = m.pnr = 0.0;
    m.preload(std::make_integer_sequence<int, kRing>{});
    while (m.steps(std::make_integer_sequence<int, kRing>{})) {
        m.kc += kRing;
        m.yb += kRing * kYw;
    }
    if (NRM) {
        const double n = wave_sum63(m.nrm), s = wave_sum63(m.pnr);
        if (lane == 63) {
            const long long o = 2 * ((long long)q * a.ntiles + bx);
            a.part[o] = n;
            a.part[o + 1] = s;
        }
    }
}

}  // namespace

// Register budgets: the FP64 forms run two waves per SIMD (the cycle form
// holds a 16-row ring of p and f), FP32 three.
template <typename T, int FORM, bool ZIN, bool NRM, bool ADD = false, bool ODD = false>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : 3)))
k_pair(const PArgs<T> args) {
    // strips fastest, each XCD a contiguous range: neighbouring strips share an L2
    const int n = gridDim.x, x = blockIdx.x & 7, l = blockIdx.x >> 3;
    const int id = x * (n >> 3) + min(x, n & 7) + l;
    pair_body<T, FORM, ZIN, NRM, ADD, ODD>(args, id % args.ntiles, id / args.ntiles);
}

template <int FORM, bool ZIN, bool ADD = false, bool ODD = false>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3)))
k_pair_group(const GEnt* __restrict__ e, int n, const PArgs<float>* __restrict__ jobs) {
    int bx, by;
    const int j = group_locate(e, n, bx, by);
    pair_body<float, FORM, ZIN, false, ADD, ODD>(jobs[j], bx, by);
}

// ------------------------------- host side -------------------------------

namespace {

// Rows a strip aims at; each level keeps one strip list per useful entry and
// a launch takes the list that fills the chip best.
constexpr int kRowTargets[] = {16, 32, 48, 64, 96, 128, 192, 256, 384};

// Block met beyond (row region, column region) of block b: the strip kernels'
// rule (the y neighbour's x neighbour, else the x neighbour's y neighbour).
int block_beyond(const Geometry& g, int b, int rr, int cr) {
    const int colb = cr == 1 ? b : g.nbr[b][cr == 0 ? XM : XP];
    if (rr == 1) return colb;
    const int fy = rr == 0 ? YM : YP;
    const int M = g.nbr[b][fy];
    if (cr == 1) return M;
    const int fx = cr == 0 ? XM : XP;
    if (M >= 0 && g.nbr[M][fx] >= 0) return g.nbr[M][fx];
    if (colb >= 0 && g.nbr[colb][fy] >= 0) return g.nbr[colb][fy];
    return -1;
}

}  // namespace

static bool pair_odd(const mbp_plan* P, int l) {
    for (int b = 0; b < P->levels[l].nb; ++b)
        if ((P->levels[l].nx[b] | P->levels[l].ny[b]) & 1) return true;
    return false;
}

// Every block at least 8 x 8, with the aligned 2 : 1 transfer the march assumes
// (fine cells 2I, 2I + 1 between coarse I - 1, I, I + 1), one sweep before and after
// the correction, no extra colours.  An odd count (whose last coarse cell I has the
// children 2I .. 2I + 2, the second between I - 1 and I or beyond I) only where a
// wall ends it: beyond a joined face the pairs of the two blocks would not align.
bool pair_level_ok(const mbp_plan* P, int l) {
    if (P->opt.nu1 != 1 || P->opt.nu2 != 1 || l + 1 >= P->nlev) return false;
    const Level& L = P->levels[l];
    if (!L.cx || !L.cy || !march_level_ok(P, l) || L.plane >= (int64_t(1) << 27)) return false;
    for (int b = 0; b < L.nb; ++b) {
        const DBlock& d = P->hblk[L.blk_off + b];
        if (d.nx < 8 || d.ny < 8 || d.par != 0) return false;
        if (((d.nx & 1) && d.nbr[XP] >= 0) || ((d.ny & 1) && d.nbr[YP] >= 0)) return false;
        auto aligned = [&](int at, int n) {
            const int I = n / 2 - 1;  // last coarse cell
            for (int i = 0; i < n; ++i) {
                const int c = P->hint[at + i];
                if ((n & 1) && i == n - 2) {
                    if (c != I - 1 && c != I) return false;
                } else if ((n & 1) && i == n - 1) {
                    if (c != I) return false;
                } else if (c != ((i & 1) ? i / 2 : i / 2 - 1)) {
                    return false;
                }
            }
            return true;
        };
        if (!aligned(d.pcx, d.nx) || !aligned(d.pcy, d.ny)) return false;
    }
    return true;
}

static size_t most_strips(int nx) { return size_t(nx + 1 + 111) / 112; }  // (the narrower strips)
size_t pair_block_doubles(int nx, int ny) { return 3 * size_t(ny + 2 * kPad) * kYw + most_strips(nx) * kXTab; }
size_t pair_block_ints(int nx) { return most_strips(nx) * (kOTab + 3); }

// Tables and strips of level l; appends to the pools and the strip list.
// halo: lanes of halo on each side (4 for the cycle form, which runs on the
// finest level; 2 otherwise).
void pair_build(mbp_plan* P, int l, int halo, std::vector<unsigned char>& bytes, std::vector<PairSet>& sets) {
    const Level& L = P->levels[l];
    const Level& Lc = P->levels[l + 1];
    const Geometry& g = P->g;
    const int wmax = 128 - 4 * halo;
    auto blk = [&](int b) -> const DBlock& { return P->hblk[L.blk_off + b]; };
    auto sign = [&](int b, int f) { return g.bc[b][f] == MBP_DIRICHLET ? -1.0 : 1.0; };
    std::vector<PTile> strips;  // one per (block, x strip), rows set below
    std::vector<int> owner;
    for (int b = 0; b < L.nb; ++b) {
        const DBlock d = blk(b);
        // y table: the three column regions over the block's rows and kPad more
        const int rows = d.ny + 2 * kPad;
        const int yt = int(P->hdbl.size());
        P->hdbl.resize(P->hdbl.size() + size_t(3) * rows * kYw, 0.0);
        for (int cr = 0; cr < 3; ++cr)
            for (int r = -kPad; r < d.ny + kPad; ++r) {
                double* y = &P->hdbl[yt + (size_t(cr) * rows + r + kPad) * kYw];
                const int rr = r < 0 ? 0 : (r < d.ny ? 1 : 2);
                const int k = block_beyond(g, b, rr, cr);
                y[2] = -1.0;
                if (k < 0) continue;
                const DBlock e = blk(k);
                const int j = rr == 0 ? e.ny + r : (rr == 2 ? r - d.ny : r);
                if (j < 0 || j >= e.ny) continue;
                y[0] = P->hdbl[e.cy + j];
                y[1] = P->hdbl[e.cy + e.ny + j];
                y[2] = P->hdbl[e.cy + 2 * e.ny + j];
                if (cr == 1 && rr == 1) y[3] = P->hdbl[e.rwy + j];
                double lo = P->hdbl[e.pwy + j], hi = 1.0 - lo;
                if (j == 0 && g.nbr[k][YM] < 0) {
                    hi += sign(k, YM) * lo;
                    lo = 0.0;
                }
                if ((e.ny & 1) && j >= e.ny - 2) {
                    // the last two rows of an odd count, between the last two coarse rows
                    if (P->hint[e.pcy + j] == e.ny / 2 - 1) {
                        hi = lo + sign(k, YP) * hi;
                        lo = 0.0;
                    }
                } else if (j == e.ny - 1 && g.nbr[k][YP] < 0) {
                    lo += sign(k, YP) * hi;
                    hi = 0.0;
                }
                y[4] = lo;
                y[5] = hi;
            }
        const int ns = (d.nx + (d.nx & 1) + wmax - 1) / wmax;
        for (int s = 0; s < ns; ++s) {
            PTile t{};
            t.x0 = 2 * int((long long)(d.nx / 2) * s / ns);
            t.w = 2 * int((long long)(d.nx / 2) * (s + 1) / ns) - t.x0;
            if (s + 1 == ns) t.w = d.nx - t.x0;
            t.bnx = d.nx;
            t.bny = d.ny;
            t.off = d.off;
            t.ncx = Lc.nx[b];
            t.ncy = Lc.ny[b];
            t.coff = Lc.off[b];
            t.hl = halo;
            t.yt = yt;
            t.xt = int(P->hdbl.size());
            P->hdbl.resize(P->hdbl.size() + kXTab, 0.0);
            while (P->hint.size() & 3) P->hint.push_back(0);
            t.ot = int(P->hint.size());
            P->hint.resize(P->hint.size() + kOTab, 0);
            for (int rr = 0; rr < 3; ++rr)
                for (int lane = 0; lane < 64; ++lane) {
                    double* xw = &P->hdbl[t.xt];
                    double* xd = xw + kXw;
                    double* xp = xd + kXd;
                    double* xr = xp + kXp;
                    int* o = &P->hint[t.ot + (rr * 64 + lane) * 4];
                    const int c = t.x0 - 2 * halo + 2 * lane;
                    const int cr = c < 0 ? 0 : (c < d.nx ? 1 : 2);
                    const int k = c < t.x0 + t.w + 2 * halo ? block_beyond(g, b, rr, cr) : -1;
                    if (k < 0) {
                        // no cell: no couplings, a diagonal that keeps it at zero
                        xd[(rr * 2) * 64 + lane] = xd[(rr * 2 + 1) * 64 + lane] = 1e30;
                        o[0] = kNoCell;
                        continue;
                    }
                    const DBlock e = blk(k);
                    const int ci = cr == 0 ? e.nx + c : (cr == 2 ? c - d.nx : c);
                    const bool lone = ci + 1 == e.nx;  // the last cell of an odd count
                    for (int sl = 0; sl < 2; ++sl) {
                        if (sl && lone) {
                            xd[(rr * 2 + sl) * 64 + lane] = 1e30;
                            continue;
                        }
                        xw[((rr * 2 + sl) * 64 + lane) * 2] = P->hdbl[e.cx + ci + sl];
                        xw[((rr * 2 + sl) * 64 + lane) * 2 + 1] = P->hdbl[e.cx + e.nx + ci + sl];
                        xd[(rr * 2 + sl) * 64 + lane] = P->hdbl[e.cx + 2 * e.nx + ci + sl];
                    }
                    double wl = P->hdbl[e.pwx + ci], w0e = 1.0 - wl;
                    double w0o = lone ? 0.0 : P->hdbl[e.pwx + ci + 1], wr = lone ? 0.0 : 1.0 - w0o;
                    if (ci == 0 && g.nbr[k][XM] < 0) {
                        w0e += sign(k, XM) * wl;
                        wl = 0.0;
                    }
                    if (lone) {  // its lower coarse cell is the left lane's, beyond is the wall
                        wl += sign(k, XP) * w0e;
                        w0e = 0.0;
                    }
                    if ((e.nx & 1) && ci == e.nx - 3) {
                        // the middle child of the last coarse cell: the third weight goes with
                        // the coarse cell to the left (March::lastc)
                        if (P->hint[e.pcx + ci + 1] == e.nx / 2 - 1) {
                            w0o += sign(k, XP) * wr;
                            wr = 0.0;
                        } else {
                            std::swap(w0o, wr);
                        }
                    }
                    if (ci == e.nx - 2 && g.nbr[k][XP] < 0) {
                        w0o += sign(k, XP) * wr;
                        wr = 0.0;
                    }
                    double* w4 = xp + (rr * 64 + lane) * 4;
                    w4[0] = wl;
                    w4[1] = w0e;
                    w4[2] = w0o;
                    w4[3] = wr;
                    if (rr == 1 && c >= t.x0 && c < t.x0 + t.w) {
                        xr[2 * lane] = P->hdbl[e.rwx + ci];
                        xr[2 * lane + 1] = lone ? 0.0 : P->hdbl[e.rwx + ci + 1];
                    }
                    const int up = rr == 0 ? e.ny : (rr == 2 ? -d.ny : 0);  // row of the neighbour's row 0
                    const int cup = rr == 0 ? Lc.ny[k] : (rr == 2 ? -Lc.ny[b] : 0);
                    o[0] = e.off + up * e.nx + ci;
                    o[1] = e.nx;
                    o[2] = Lc.off[k] + cup * Lc.nx[k] + ci / 2;
                    o[3] = Lc.nx[k];
                }
            strips.push_back(t);
            owner.push_back(b);
        }
    }
    for (int target : kRowTargets) {
        PairSet ps;
        ps.off = int(bytes.size() / sizeof(PTile));
        std::vector<PTile> out;
        // strips of one block side by side, so that neighbours run together
        for (size_t s0 = 0; s0 < strips.size();) {
            size_t s1 = s0;
            while (s1 < strips.size() && owner[s1] == owner[s0]) ++s1;
            const int ny = strips[s0].bny, nseg = (ny + target - 1) / target;
            for (int y = 0; y < nseg; ++y)
                for (size_t s = s0; s < s1; ++s) {
                    PTile t = strips[s];
                    t.y0 = 2 * int((long long)(ny / 2) * y / nseg);
                    t.y1 = y + 1 == nseg ? ny : 2 * int((long long)(ny / 2) * (y + 1) / nseg);
                    ps.rows = std::max(ps.rows, t.y1 - t.y0);
                    out.push_back(t);
                }
            s0 = s1;
        }
        ps.cnt = int(out.size());
        if (!sets.empty() && sets.back().cnt == ps.cnt) break;  // no block is taller than the last target
        const unsigned char* src = reinterpret_cast<const unsigned char*>(out.data());
        bytes.insert(bytes.end(), src, src + out.size() * sizeof(PTile));
        sets.push_back(ps);
    }
}

// Workgroups of a kernel resident on the chip at once with that much LDS
// (taken once per kernel, size and device).
static int pair_slots(const void* kernel, size_t lds) {
    static std::mutex mu;
    static std::map<std::tuple<int, const void*, size_t>, int> cache;
    int dev = 0;
    (void)hipGetDevice(&dev);
    std::lock_guard<std::mutex> lock(mu);
    auto it = cache.find({dev, kernel, lds});
    if (it != cache.end()) return it->second;
    int per_cu = 0, ncu = 0;
    int most = 0;  // the kernel may be launched with any size up to the device's
    if (hipDeviceGetAttribute(&most, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess)
        (void)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, most);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, 256, lds) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        per_cu = 1;
        ncu = 256;
    }
    return cache[{dev, kernel, lds}] = std::max(1, per_cu) * std::max(1, ncu);
}

// The strip list of level l for nitems modes: the one whose rounds of
// workgroups times the rows a workgroup marches (its strip, halo and set-up)
// are fewest; ties go to the taller strips, which read less halo.
template <typename T>
static const PairSet& pair_choose(const mbp_plan* P, int l, int nitems, const void* kernel, bool corr) {
    const std::vector<PairSet>& sets = P->pair_sets[l];
    size_t best = 0;
    long long cost = -1;
    for (size_t i = 0; i < sets.size(); ++i) {
        const size_t lds = pair_lds_bytes<T>(sets[i].rows, corr);
        if (int64_t(lds) > P->lds_limit) continue;
        const long long wgs = (long long)sets[i].cnt * ((nitems + 3) / 4), slots = pair_slots(kernel, lds);
        const long long c = ((wgs + slots - 1) / slots) * (sets[i].rows + 32);
        if (cost < 0 || c <= cost) {
            cost = c;
            best = i;
        }
    }
    return sets[best];
}

template <typename T>
static PArgs<T> pair_args(const mbp_plan* P, int l, const PairSet& set, const T* f, const T* ec, T* fc, T* pa,
                          T* pb, const int* cycle, const int* act, const int* nact, bool norm) {
    PArgs<T> a{};
    a.tiles = reinterpret_cast<const PTile*>(P->d_ptiles) + set.off;
    a.ntiles = set.cnt;
    a.dp = P->d_dbl;
    a.ip = P->d_int;
    a.pa = pa;
    a.pb = pb;
    a.cycle = cycle;
    a.f = f;
    a.ec = ec;
    a.fc = fc;
    a.plane = P->levels[l].plane;
    a.plane_c = P->levels[l + 1].plane;
    a.shift = P->d_shift;
    a.act = act;
    a.nact = nact;
    a.part = norm ? P->d_part : nullptr;
    a.nparts = norm ? P->d_flag + 3 : nullptr;
    return a;
}

template <typename T, int FORM, bool ZIN, bool NRM, bool ADD = false, bool ODD = false>
static void launch_pair(const mbp_plan* P, int l, const T* f, const T* ec, T* fc, T* pa, T* pb, const int* cycle,
                        const int* act, const int* nact, int nitems, hipStream_t s, double* sum = nullptr,
                        bool first = false) {
    if constexpr (!ODD)
        if (pair_odd(P, l)) {
            launch_pair<T, FORM, ZIN, NRM, ADD, true>(P, l, f, ec, fc, pa, pb, cycle, act, nact, nitems, s, sum, first);
            return;
        }
    const void* fn = reinterpret_cast<const void*>(k_pair<T, FORM, ZIN, NRM, ADD, ODD>);
    const PairSet& set = pair_choose<T>(P, l, nitems, fn, FORM != kPre);
    PArgs<T> a = pair_args<T>(P, l, set, f, ec, fc, pa, pb, cycle, act, nact, NRM);
    a.sum = sum;
    a.first = first ? 1 : 0;
    hipLaunchKernelGGL((k_pair<T, FORM, ZIN, NRM, ADD, ODD>), dim3(set.cnt * ((nitems + 3) / 4)), dim3(256),
                       pair_lds_bytes<T>(set.rows, FORM != kPre), s, a);
}

// Pre-smoothing of p (nullptr: zero) and restriction of the residual into fc.
template <typename T>
void pair_pre(const mbp_plan* P, int l, const T* p, const T* f, T* fc, const int* act, const int* nact, int nitems,
              hipStream_t s) {
    T* pp = const_cast<T*>(p);
    if (p) launch_pair<T, kPre, false, false>(P, l, f, nullptr, fc, pp, nullptr, nullptr, act, nact, nitems, s);
    else launch_pair<T, kPre, true, false>(P, l, f, nullptr, fc, nullptr, nullptr, nullptr, act, nact, nitems, s);
}

// Pre-smoothing of p (nullptr: zero) again, correction ec, post-smoothing into pnew.
template <typename T>
void pair_post(const mbp_plan* P, int l, const T* p, T* pnew, const T* f, const T* ec, const int* act, const int* nact,
               int nitems, hipStream_t s) {
    T* pp = const_cast<T*>(p);
    if (p) launch_pair<T, kPost, false, false>(P, l, f, ec, nullptr, pp, pnew, nullptr, act, nact, nitems, s);
    else launch_pair<T, kPost, true, false>(P, l, f, ec, nullptr, nullptr, pnew, nullptr, act, nact, nitems, s);
}

// The same on the finest level, added to the FP64 iterate sum (first: zero so far).
void pair_post_add(const mbp_plan* P, const float* p, double* sum, bool first, const float* f, const float* ec,
                   const int* act, const int* nact, int nitems, hipStream_t s) {
    float* pp = const_cast<float*>(p);
    if (p) launch_pair<float, kPost, false, false, true>(P, 0, f, ec, nullptr, pp, nullptr, nullptr, act, nact, nitems, s, sum, first);
    else launch_pair<float, kPost, true, false, true>(P, 0, f, ec, nullptr, nullptr, nullptr, nullptr, act, nact, nitems, s, sum, first);
}

// The same as pair_post, then the next cycle's pre-smoothing and restriction.  zero: p is
// zero.  FP64: per-strip squared residual and solution sums too.  cycle:
// device count of convergence tests that picks the buffers (see PArgs).
template <typename T>
void pair_cycle(const mbp_plan* P, int l, T* pa, T* pb, const int* cycle, const T* f, const T* ec, T* fc, bool zero,
                const int* act, const int* nact, int nitems, hipStream_t s) {
    auto go = [&](auto z, auto n) {
        launch_pair<T, kCycle, decltype(z)::value, decltype(n)::value>(P, l, f, ec, fc, pa, pb, cycle, act, nact,
                                                                      nitems, s);
    };
    if constexpr (sizeof(T) == 8) {
        if (zero) go(std::true_type{}, std::true_type{});
        else go(std::false_type{}, std::true_type{});
    } else {
        if (zero) go(std::true_type{}, std::false_type{});
        else go(std::false_type{}, std::false_type{});
    }
}

int pair_max_strips(const mbp_plan* P, int l) {
    return P->pair_sets.size() > size_t(l) && !P->pair_sets[l].empty() ? P->pair_sets[l][0].cnt : 0;
}

template void pair_pre<double>(const mbp_plan*, int, const double*, const double*, double*, const int*, const int*,
                               int, hipStream_t);
template void pair_pre<float>(const mbp_plan*, int, const float*, const float*, float*, const int*, const int*, int,
                              hipStream_t);
template void pair_post<double>(const mbp_plan*, int, const double*, double*, const double*, const double*, const int*,
                                const int*, int, hipStream_t);
template void pair_post<float>(const mbp_plan*, int, const float*, float*, const float*, const float*, const int*,
                               const int*, int, hipStream_t);
template void pair_cycle<double>(const mbp_plan*, int, double*, double*, const int*, const double*, const double*,
                                 double*, bool, const int*, const int*, int, hipStream_t);
template void pair_cycle<float>(const mbp_plan*, int, float*, float*, const int*, const float*, const float*, float*,
                                bool, const int*, const int*, int, hipStream_t);

template <bool ODD>
static const void* group_kernel(int kind) {
    switch (kind) {
        case G_PAIR_PRE: return reinterpret_cast<const void*>(k_pair_group<kPre, true, false, ODD>);
        case G_PAIR_POST0: return reinterpret_cast<const void*>(k_pair_group<kPost, true, false, ODD>);
        case G_PAIR_ADD0: return reinterpret_cast<const void*>(k_pair_group<kPost, true, true, ODD>);
        case G_PAIR_ADD: return reinterpret_cast<const void*>(k_pair_group<kPost, false, true, ODD>);
        case G_PAIR_CYCLE0: return reinterpret_cast<const void*>(k_pair_group<kCycle, true, false, ODD>);
        default: return reinterpret_cast<const void*>(k_pair_group<kCycle, false, false, ODD>);
    }
}

// Level `level` of every problem whose level the pair march takes, for inner
// cycle k of the FP32 correction solve: on the way down the pre-smoothing and
// restriction (the finest level's only in cycle 0: later ones were done by
// the cycle form), on the way up the correction and post-smoothing (finest
// level: the cycle form, but the last cycle).  The finest iterate starts from
// zero in p32 and alternates with p32B.  One rows-a-strip target serves the
// whole launch: the fewest rounds of workgroups times rows, as for one problem.
GStage group_pair32(GroupBlob& gb, const std::vector<SolveCtx*>& cs, int level, bool down, int k, int inner) {
    const int l = level;
    const bool last = k + 1 == inner;
    std::vector<const SolveCtx*> in;
    for (const SolveCtx* c : cs)
        if (l < c->P->lds_level32 && c->P->pair_ok[l] && !(down && l == 0 && k > 0)) in.push_back(c);
    const int kind = down ? G_PAIR_PRE
                          : l > 0 ? G_PAIR_POST0
                                  : last ? (k == 0 ? G_PAIR_ADD0 : G_PAIR_ADD) : (k == 0 ? G_PAIR_CYCLE0 : G_PAIR_CYCLE);
    GStage none;
    none.kind = kind;
    if (in.empty()) return none;
    // one launch for all: where one plane is odd, the form that can do both
    bool odd = false;
    for (const SolveCtx* c : in) odd = odd || pair_odd(c->P, l);
    const void* fn = odd ? group_kernel<true>(kind) : group_kernel<false>(kind);
    auto set = [&](const SolveCtx* c, size_t t) -> const PairSet& {
        const std::vector<PairSet>& v = c->P->pair_sets[l];
        return v[std::min(t, v.size() - 1)];
    };
    size_t best = 0, lds = 0;
    long long cost = -1;
    for (size_t t = 0; t < sizeof(kRowTargets) / sizeof(kRowTargets[0]); ++t) {
        long long wgs = 0;
        int rows = 0;
        for (const SolveCtx* c : in) {
            wgs += (long long)set(c, t).cnt * ((c->nitems + 3) / 4);
            rows = std::max(rows, set(c, t).rows);
        }
        const size_t bytes = pair_lds_bytes<float>(rows, !down);
        if (int64_t(bytes) > in[0]->P->lds_limit) break;
        const long long slots = pair_slots(fn, bytes), x = ((wgs + slots - 1) / slots) * (rows + 32);
        if (cost < 0 || x <= cost) {
            cost = x;
            best = t;
            lds = bytes;
        }
    }
    std::vector<PArgs<float>> jobs;
    std::vector<int> gx, gy;
    for (const SolveCtx* c : in) {
        const mbp_plan* P = c->P;
        const PairSet& ps = set(c, best);
        float* pa = l == 0 ? ((k & 1) ? P->p32B[0] : P->p32[0]) : nullptr;
        float* pb = l == 0 ? ((k & 1) ? P->p32[0] : P->p32B[0]) : P->p32[l];
        jobs.push_back(pair_args<float>(P, l, ps, P->f32[l], down ? nullptr : P->p32[l + 1], P->f32[l + 1], pa, pb, nullptr,
                                        P->d_act, P->d_nact, false));
        jobs.back().sum = P->phat;
        gx.push_back(ps.cnt);
        gy.push_back((c->nitems + 3) / 4);
    }
    GStage st = group_build(gb, kind, jobs, gx, gy);
    st.lds = lds;
    st.odd = odd;
    return st;
}

void group_launch_pair(const GStage& st, const unsigned char* dev, hipStream_t s) {
    if (st.wgs <= 0) return;
    const GEnt* e = reinterpret_cast<const GEnt*>(dev + st.ent_off);
    const PArgs<float>* j = reinterpret_cast<const PArgs<float>*>(dev + st.job_off);
    const void* fn = st.odd ? group_kernel<true>(st.kind) : group_kernel<false>(st.kind);
    int n = st.nent;
    void* args[] = {&e, &n, &j};
    (void)hipLaunchKernel(fn, dim3(st.wgs), dim3(256), args, st.lds, s);
}

}  // namespace mbp
