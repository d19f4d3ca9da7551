// Real-to-real transforms along the homogeneous z direction (Algorithm 1,
// first and last loops; Table 1 kinds).  Every kind is reduced to one
// complex FFT of length m = n/2 per z column:
//   periodic  -> discrete Hartley transform from the half-length real DFT;
//   N-N       -> DCT-II by Makhoul's even/odd reordering (inverse DCT-III);
//   D-D       -> DST-II as the DCT-II of (-1)^j x read backwards (DST-III);
//   N-D       -> DCT-IV with the quarter-wave pre/post twiddles (self-inverse);
//   D-N       -> DST-IV as (-1)^q DCT-IV of x reversed (self-inverse).
// All transforms are orthonormal.  The complex FFT is a mixed-radix Stockham
// autosort held in LDS; a workgroup transforms W neighbouring columns, whose
// z rows are read and written as contiguous W-element segments.
#include <algorithm>

#include "internal.h"

namespace mbp {

struct FFTArgs {
    int n, m, kind, W, cs;
    int nstage;
    int radix[16];
    const double* tw;     // e^{-2 pi i t / m}, t < m
    const double* twn;    // e^{-2 pi i k / n}, k <= m
    const double* post;   // e^{-i pi k / (2n)}, k <= n
    const double* pre4;   // e^{-i pi (4k+1) / (4n)}, k < m
    const double* post4;  // e^{-i pi k / n}, k < m
};

struct FTile {
    long long in_base, out_base;  // element offsets of column 0 of the tile
    int in_stride, out_stride;    // distance between consecutive z rows
    int ncol;                     // valid columns (<= W)
    int pad;
};

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cconj(double2 a) { return make_double2(a.x, -a.y); }
// The transform tables are never written while a kernel runs: reading them
// through the constant address space marks the loads invariant, so they may
// move ahead of the stores of earlier results and stay in flight together.
typedef __attribute__((address_space(4))) const double ctab_t;
__device__ __forceinline__ double2 ld2(const double* t, int k) {
    const ctab_t* c = (const ctab_t*)t;
    return make_double2(c[2 * k], c[2 * k + 1]);
}

// Where a transform reads its tables: straight from device memory (through
// the constant address space), or from a copy in LDS.
struct GlobalTab {
    const double* t;
    __device__ __forceinline__ double2 operator()(int k) const { return ld2(t, k); }
};
struct LdsTab {
    const double2* t;
    __device__ __forceinline__ double2 operator()(int k) const { return t[k]; }
};

// a / b for 0 <= a < 2^22 and 1 <= b < 2^12, from the float reciprocal rb of
// b: the float quotient is within one of the true one, and the remainder
// test corrects it.
__device__ __forceinline__ int div_small(int a, int b, float rb) {
    int q = int(float(a) * rb);
    const int r = a - q * b;
    if (r < 0) --q;
    else if (r >= b) ++q;
    return q;
}

// cos and sin of 2 pi t / R for the odd radices with closed-form butterflies
template <int R>
struct Roots;
template <>
struct Roots<3> {
    static constexpr double c[3] = {1.0, -0.5, -0.5};
    static constexpr double s[3] = {0.0, 0.86602540378443864676, -0.86602540378443864676};
};
template <>
struct Roots<5> {
    static constexpr double c[5] = {1.0, 0.30901699437494742410, -0.80901699437494742410,
                                    -0.80901699437494742410, 0.30901699437494742410};
    static constexpr double s[5] = {0.0, 0.95105651629515357212, 0.58778525229247312917,
                                    -0.58778525229247312917, -0.95105651629515357212};
};
template <>
struct Roots<7> {
    static constexpr double c[7] = {1.0, 0.62348980185873353053, -0.22252093395631440429,
                                    -0.90096886790241912624, -0.90096886790241912624,
                                    -0.22252093395631440429, 0.62348980185873353053};
    static constexpr double s[7] = {0.0, 0.78183148246802980871, 0.97492791218182360702,
                                    0.43388373911755812048, -0.43388373911755812048,
                                    -0.97492791218182360702, -0.78183148246802980871};
};

template <>
struct Roots<9> {  // up to the product 2 * 2 of the 3 x 3 split
    static constexpr double c[5] = {1.0, 0.76604444311897803520, 0.17364817766693034885, -0.5,
                                    -0.93969262078590838405};
    static constexpr double s[5] = {0.0, 0.64278760968653932632, 0.98480775301220805937, 0.86602540378443864676,
                                    0.34202014332566873304};
};
template <>
struct Roots<16> {  // up to the product 3 * 3 of the 4 x 4 split
    static constexpr double c[10] = {1.0, 0.92387953251128675613, 0.70710678118654752440, 0.38268343236508977173, 0.0,
                                     -0.38268343236508977173, -0.70710678118654752440, -0.92387953251128675613, -1.0,
                                     -0.92387953251128675613};
    static constexpr double s[10] = {0.0, 0.38268343236508977173, 0.70710678118654752440, 0.92387953251128675613, 1.0,
                                     0.92387953251128675613, 0.70710678118654752440, 0.38268343236508977173, 0.0,
                                     -0.38268343236508977173};
};

// XCD-aware mapping: workgroups are dispatched round-robin over the 8 XCDs;
// give each XCD one contiguous range of tiles so neighbouring tiles share an L2.
__device__ __forceinline__ int xcd_remap(int g, int n) {
    int x = g & 7, l = g >> 3;
    int per = n >> 3, rem = n & 7;
    return x * per + min(x, rem) + l;
}

// DFT of length R of v[0..R-1] in place, forward sign e^{-2 pi i rs/R}.
// Radices 2, 4 and 8 use their closed-form roots; odd radices read the roots
// tw[(r s mod R) m / R] from the twiddle table.
template <int R, typename TW>
__device__ __forceinline__ void dft(double2* v, const TW& tw, int m) {
    if constexpr (R == 2) {
        const double2 a = v[0], b = v[1];
        v[0] = make_double2(a.x + b.x, a.y + b.y);
        v[1] = make_double2(a.x - b.x, a.y - b.y);
    } else if constexpr (R == 4) {
        const double2 s02 = make_double2(v[0].x + v[2].x, v[0].y + v[2].y);
        const double2 d02 = make_double2(v[0].x - v[2].x, v[0].y - v[2].y);
        const double2 s13 = make_double2(v[1].x + v[3].x, v[1].y + v[3].y);
        const double2 d13 = make_double2(v[1].x - v[3].x, v[1].y - v[3].y);
        v[0] = make_double2(s02.x + s13.x, s02.y + s13.y);
        v[2] = make_double2(s02.x - s13.x, s02.y - s13.y);
        v[1] = make_double2(d02.x + d13.y, d02.y - d13.x);  // d02 - i d13
        v[3] = make_double2(d02.x - d13.y, d02.y + d13.x);  // d02 + i d13
    } else if constexpr (R == 8) {
        // two length-4 DFTs of the even / odd samples, then the radix-2 step
        // with the eighth roots e^{-i pi s / 4}
        double2 e[4] = {v[0], v[2], v[4], v[6]};
        double2 o[4] = {v[1], v[3], v[5], v[7]};
        dft<4>(e, tw, m);
        dft<4>(o, tw, m);
        const double h = 0.70710678118654752440;
        const double2 w1 = make_double2(h * (o[1].x + o[1].y), h * (o[1].y - o[1].x));   // e^{-i pi/4} o1
        const double2 w2 = make_double2(o[2].y, -o[2].x);                                // -i o2
        const double2 w3 = make_double2(h * (o[3].y - o[3].x), -h * (o[3].x + o[3].y));  // e^{-3i pi/4} o3
        v[0] = make_double2(e[0].x + o[0].x, e[0].y + o[0].y);
        v[4] = make_double2(e[0].x - o[0].x, e[0].y - o[0].y);
        v[1] = make_double2(e[1].x + w1.x, e[1].y + w1.y);
        v[5] = make_double2(e[1].x - w1.x, e[1].y - w1.y);
        v[2] = make_double2(e[2].x + w2.x, e[2].y + w2.y);
        v[6] = make_double2(e[2].x - w2.x, e[2].y - w2.y);
        v[3] = make_double2(e[3].x + w3.x, e[3].y + w3.y);
        v[7] = make_double2(e[3].x - w3.x, e[3].y - w3.y);
    } else if constexpr (R == 3 || R == 5 || R == 7) {
        // pairs r, R - r: v_r w^{rs} + v_{R-r} w^{-rs} = a_r cos - i b_r sin
        // with a_r = v_r + v_{R-r}, b_r = v_r - v_{R-r}, w = e^{-2 pi i / R}
        constexpr int H = (R - 1) / 2;
        double2 a[H], b[H];
        double2 y0 = v[0];
#pragma unroll
        for (int r = 1; r <= H; ++r) {
            a[r - 1] = make_double2(v[r].x + v[R - r].x, v[r].y + v[R - r].y);
            b[r - 1] = make_double2(v[r].x - v[R - r].x, v[r].y - v[R - r].y);
            y0.x += a[r - 1].x;
            y0.y += a[r - 1].y;
        }
        double2 y[R];
        y[0] = y0;
#pragma unroll
        for (int s = 1; s <= H; ++s) {
            double2 re = v[0], im = make_double2(0.0, 0.0);
#pragma unroll
            for (int r = 1; r <= H; ++r) {
                const double c = Roots<R>::c[(r * s) % R], sn = Roots<R>::s[(r * s) % R];
                re.x += c * a[r - 1].x;
                re.y += c * a[r - 1].y;
                im.x += sn * b[r - 1].x;
                im.y += sn * b[r - 1].y;
            }
            y[s] = make_double2(re.x + im.y, re.y - im.x);      // re - i im
            y[R - s] = make_double2(re.x - im.y, re.y + im.x);  // re + i im
        }
#pragma unroll
        for (int s = 0; s < R; ++s) v[s] = y[s];
    } else if constexpr (R == 6 || R == 10 || R == 12 || R == 15) {
        // coprime factors A B: sample (B r1 + A r2) mod R and output s with
        // (s mod A, s mod B) make it an A x B transform without roots between
        constexpr int A = R == 6 || R == 10 ? 2 : 3, B = R / A;
        double2 y[A][B];
#pragma unroll
        for (int r2 = 0; r2 < B; ++r2) {
            double2 u[A];
#pragma unroll
            for (int r1 = 0; r1 < A; ++r1) u[r1] = v[(B * r1 + A * r2) % R];
            dft<A>(u, tw, m);
#pragma unroll
            for (int r1 = 0; r1 < A; ++r1) y[r1][r2] = u[r1];
        }
#pragma unroll
        for (int s1 = 0; s1 < A; ++s1) dft<B>(y[s1], tw, m);
#pragma unroll
        for (int s = 0; s < R; ++s) v[s] = y[s % A][s % B];
    } else if constexpr (R == 9 || R == 16) {
        // A x A with the roots e^{-2 pi i r s / R} between
        constexpr int A = R == 9 ? 3 : 4;
        double2 y[A][A];
#pragma unroll
        for (int r2 = 0; r2 < A; ++r2) {
            double2 u[A];
#pragma unroll
            for (int r1 = 0; r1 < A; ++r1) u[r1] = v[r1 * A + r2];
            dft<A>(u, tw, m);
#pragma unroll
            for (int s1 = 0; s1 < A; ++s1)
                y[s1][r2] = r2 * s1 ? cmul(u[s1], make_double2(Roots<R>::c[r2 * s1], -Roots<R>::s[r2 * s1])) : u[s1];
        }
#pragma unroll
        for (int s1 = 0; s1 < A; ++s1) {
            dft<A>(y[s1], tw, m);
#pragma unroll
            for (int s2 = 0; s2 < A; ++s2) v[s1 + A * s2] = y[s1][s2];
        }
    } else {
        double2 y[R];
#pragma unroll
        for (int s = 0; s < R; ++s) {
            double2 acc = v[0];
#pragma unroll
            for (int r = 1; r < R; ++r) {
                const double2 rt = tw(((r * s) % R) * (m / R));
                const double2 pr = cmul(v[r], rt);
                acc.x += pr.x;
                acc.y += pr.y;
            }
            y[s] = acc;
        }
#pragma unroll
        for (int s = 0; s < R; ++s) v[s] = y[s];
    }
}

// One Stockham stage of radix R over W columns held column-major in LDS
// (column stride cs complex values).  Reads all inputs into registers before
// a barrier, then writes the outputs, so the stage runs in place.
template <int R, int BPT, typename TW>
__device__ void stage(double2* z, int cs, int m, int W, int Ns, const TW& tw, int tid, int nthr) {
    const int nbf = m / R;
    const int total = W * nbf;
    const int step = m / (Ns * R);  // twiddle index stride
    const float r_nbf = 1.0f / float(nbf), r_ns = 1.0f / float(Ns);
    double2 v[BPT][R];
    int dst[BPT];
#pragma unroll
    for (int t = 0; t < BPT; ++t) {
        const int b = tid + t * nthr;
        dst[t] = -1;
        if (b < total) {
            const int w = div_small(b, nbf, r_nbf), j = b - w * nbf;
            const int jn = div_small(j, Ns, r_ns), k = j - jn * Ns;
            const double2* col = z + w * cs;
            // every twiddle is read unconditionally (k = 0 reads the exact
            // root 1), so all of the loads are in flight together;
            // k r step < Ns R step = m: the index needs no wrap
            double2 rt[R];
#pragma unroll
            for (int r = 1; r < R; ++r) rt[r] = tw(k * r * step);
            v[t][0] = col[j];
#pragma unroll
            for (int r = 1; r < R; ++r) v[t][r] = cmul(col[j + r * nbf], rt[r]);
            dft<R>(v[t], tw, m);
            dst[t] = w * cs + jn * Ns * R + k;
        }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < BPT; ++t) {
        if (dst[t] < 0) continue;
#pragma unroll
        for (int r = 0; r < R; ++r) z[dst[t] + r * Ns] = v[t][r];
    }
    __syncthreads();
}

// One Stockham stage of any radix R (a prime above 31, for which no
// unrolled butterfly exists): each output of butterfly (j = jn Ns + k) is
// y_s = sum_r z[j + r m/R] w^{r (k + s Ns) m / (Ns R)}, w = e^{-2 pi i / m},
// computed straight from LDS (R complex products per output).  The host
// keeps W m <= MAXOUT * blockDim.x.
template <int MAXOUT, typename TW>
__device__ void stage_generic(double2* z, int cs, int m, int W, int Ns, int R, const TW& tw) {
    const int nbf = m / R;
    const int step = m / (Ns * R);
    const int total = W * m;
    double2 y[MAXOUT];
    int dst[MAXOUT];
#pragma unroll
    for (int t = 0; t < MAXOUT; ++t) {
        const int o = threadIdx.x + t * blockDim.x;
        dst[t] = -1;
        if (o >= total) continue;
        const int w = o / m, rest = o - w * m;
        const int s = rest / nbf, j = rest - s * nbf;
        const int jn = j / Ns, k = j - jn * Ns;
        const double2* col = z + w * cs;
        const int inc = int(((long long)(k + s * Ns) * step) % m);
        int ti = 0;
        double2 acc = make_double2(0.0, 0.0);
        for (int r = 0; r < R; ++r) {
            const double2 pr = cmul(col[j + r * nbf], tw(ti));
            acc.x += pr.x;
            acc.y += pr.y;
            ti += inc;
            if (ti >= m) ti -= m;
        }
        y[t] = acc;
        dst[t] = w * cs + jn * Ns * R + k + s * Ns;
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < MAXOUT; ++t)
        if (dst[t] >= 0) z[dst[t]] = y[t];
    __syncthreads();
}

constexpr int kGenericOut = 16;  // outputs per thread of the any-radix stage

template <int R, typename TW>
__device__ void stage_dispatch(double2* z, int cs, int m, int W, int Ns, const TW& tw) {
    const int total = W * (m / R);
    const int bpt = (total + blockDim.x - 1) / blockDim.x;
    if constexpr (R > 8) {
        stage<R, 1>(z, cs, m, W, Ns, tw, threadIdx.x, blockDim.x);  // the host keeps W * m / R <= 256 here
    } else {
        // the host keeps bpt <= 16 / R for R = 2 and 4, bpt <= 2 otherwise
        if (bpt <= 1) stage<R, 1>(z, cs, m, W, Ns, tw, threadIdx.x, blockDim.x);
        else if (bpt <= 2) stage<R, 2>(z, cs, m, W, Ns, tw, threadIdx.x, blockDim.x);
        else if constexpr (R == 2 || R == 4) {
            if (bpt <= 4) stage<R, 4>(z, cs, m, W, Ns, tw, threadIdx.x, blockDim.x);
            else if constexpr (R == 2) stage<R, 8>(z, cs, m, W, Ns, tw, threadIdx.x, blockDim.x);
        }
    }
}

// Radix classes: 0 = powers of two only, 1 = with 3 / 5 / 7, 2 = any prime
// up to 31, 3 = also primes above 31 (the any-radix stage).  Each class is
// its own kernel so the power-of-two transforms do not carry the register
// footprint of the long odd butterflies.
template <int CLASS, typename TW>
__device__ void fft_columns(double2* z, int cs, const FFTArgs& a, const TW& tw) {
    int Ns = 1;
    for (int s = 0; s < a.nstage; ++s) {
        const int R = a.radix[s];
        switch (R) {
            case 2: stage_dispatch<2>(z, cs, a.m, a.W, Ns, tw); break;
            case 4: stage_dispatch<4>(z, cs, a.m, a.W, Ns, tw); break;
            case 8: stage_dispatch<8>(z, cs, a.m, a.W, Ns, tw); break;
            default:
                if constexpr (CLASS >= 1) {
                    switch (R) {
                        case 3: stage_dispatch<3>(z, cs, a.m, a.W, Ns, tw); break;
                        case 5: stage_dispatch<5>(z, cs, a.m, a.W, Ns, tw); break;
                        case 7: stage_dispatch<7>(z, cs, a.m, a.W, Ns, tw); break;
                        default:
                            if constexpr (CLASS >= 2) {
                                switch (R) {
                                    case 11: stage_dispatch<11>(z, cs, a.m, a.W, Ns, tw); break;
                                    case 13: stage_dispatch<13>(z, cs, a.m, a.W, Ns, tw); break;
                                    case 17: stage_dispatch<17>(z, cs, a.m, a.W, Ns, tw); break;
                                    case 19: stage_dispatch<19>(z, cs, a.m, a.W, Ns, tw); break;
                                    case 23: stage_dispatch<23>(z, cs, a.m, a.W, Ns, tw); break;
                                    case 29: stage_dispatch<29>(z, cs, a.m, a.W, Ns, tw); break;
                                    case 31: stage_dispatch<31>(z, cs, a.m, a.W, Ns, tw); break;
                                    default:
                                        if constexpr (CLASS >= 3)
                                            stage_generic<kGenericOut>(z, cs, a.m, a.W, Ns, R, tw);
                                        break;
                                }
                            }
                            break;
                    }
                }
                break;
        }
        Ns *= R;
    }
}

constexpr int kLoadBatch = 8;   // input elements per thread in flight together
constexpr int kStoreBatch = 4;  // output elements per thread whose table reads go together
constexpr int kInvBatch = 2;    // inverse cosine kinds: elements per thread read together

// Forward (dir = 0) or inverse (dir = 1) transform of W columns per workgroup.
template <int CLASS>
__global__ void __launch_bounds__(256) k_r2r(FFTArgs a, const FTile* __restrict__ tiles, int ntiles,
                                             int dir, const double* __restrict__ in,
                                             double* __restrict__ out, int* nonfinite, const int* gate) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    double2* z = reinterpret_cast<double2*>(lds_raw);
    if (gate && *gate) return;  // out is left alone
    const int tix = xcd_remap(blockIdx.x, ntiles);
    const FTile T = tiles[tix];
    const int n = a.n, m = a.m, W = a.W, cs = a.cs;
    const int lw = __ffs(W) - 1;  // W is a power of two
    const int kind = a.kind;
    const double sc2 = sqrt(2.0 / n), sc1 = sqrt(1.0 / n);
    // which algorithm runs: forward kinds, and the inverse of N-N / D-D
    const bool inv_cos = dir == 1 && (kind == Z_NN || kind == Z_DD);

    // ---------------- load + pre-processing ----------------
    if (!inv_cos) {
        bool bad = false;
        // kLoadBatch elements per thread are loaded before any is used, so
        // their loads are in flight together.  Every load is unconditional:
        // elements past the end repeat the last one, columns past the tile's
        // last read that one and are zeroed.
        for (int base = 0; base < n * W; base += kLoadBatch * blockDim.x) {
            double xs[kLoadBatch];
#pragma unroll
            for (int b = 0; b < kLoadBatch; ++b) {
                const int idx = min(base + b * int(blockDim.x) + int(threadIdx.x), n * W - 1);
                const int k = idx >> lw, w = idx & (W - 1);
                xs[b] = in[T.in_base + (long long)k * T.in_stride + min(w, T.ncol - 1)];
            }
#pragma unroll
            for (int b = 0; b < kLoadBatch; ++b) {
            const int idx = min(base + b * int(blockDim.x) + int(threadIdx.x), n * W - 1);
            const int k = idx >> lw, w = idx & (W - 1);
            double x = w >= T.ncol ? 0.0 : xs[b];
            if (!isfinite(x)) bad = true;
            double* zc = reinterpret_cast<double*>(z + w * cs);
            // position u in the length-n real sequence fed to the FFT, chosen
            // without branches: PP keeps k; NN / DD take Makhoul's even / odd
            // reordering (DD with alternating signs); ND packs for the DCT-IV,
            // DN packs the reversed input j = n - 1 - k the same way
            const int uc = (k & 1) ? n - 1 - (k >> 1) : (k >> 1);
            const int kk = kind == Z_DN ? n - 1 - k : k;
            const int u4 = (kk & 1) ? ((n - 1 - kk) >> 1) * 2 + 1 : (kk >> 1) * 2;
            const int u = kind == Z_PP ? k : (kind == Z_NN || kind == Z_DD) ? uc : u4;
            x = (kind == Z_DD && (k & 1)) ? -x : x;
            zc[u] = x;  // real part at even u, imaginary part at odd u
            }
        }
        if (bad && nonfinite) atomicOr(nonfinite, 1);
        __syncthreads();
        if (kind == Z_ND || kind == Z_DN) {
            const float rm = 1.0f / float(m);
            for (int idx = threadIdx.x; idx < m * W; idx += blockDim.x) {
                int w = div_small(idx, m, rm), k = idx - w * m;
                z[w * cs + k] = cmul(z[w * cs + k], ld2(a.pre4, k));
            }
            __syncthreads();
        }
    } else {
        // inverse of the cosine kinds: V_q = e^{i pi q/(2n)} (y'_q - i y'_{n-q}),
        // Z_k = (V_k + conj V_{m-k}) + i (V_k - conj V_{m-k}) e^{2 pi i k/n};
        // the FFT below then computes conj(IFFT) of conj(Z).
        const int half = m / 2;
        for (int base = 0; base < (half + 1) * W; base += kInvBatch * blockDim.x) {
            // y'_q = y_q / c_q at q = k, n-k, m-k, m+k (y'_n = 0), and the
            // table values, read for kInvBatch elements before any is used
            double yv[kInvBatch][4];
            double2 pk[kInvBatch], pmk[kInvBatch], tk[kInvBatch], tmk[kInvBatch];
#pragma unroll
            for (int b = 0; b < kInvBatch; ++b) {
                const int idx = min(base + b * int(blockDim.x) + int(threadIdx.x), (half + 1) * W - 1);
                const int k = idx >> lw, w = idx & (W - 1);
                const int qs[4] = {k, n - k, m - k, m + k};
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int qc = min(qs[v], n - 1);
                    const int row = kind == Z_DD ? n - 1 - qc : qc;
                    yv[b][v] = in[T.in_base + (long long)row * T.in_stride + min(w, T.ncol - 1)];
                }
                pk[b] = ld2(a.post, k);
                pmk[b] = ld2(a.post, m - k);
                tk[b] = ld2(a.twn, k);
                tmk[b] = ld2(a.twn, m - k);
            }
#pragma unroll
            for (int b = 0; b < kInvBatch; ++b) {
                const int idx = min(base + b * int(blockDim.x) + int(threadIdx.x), (half + 1) * W - 1);
                const int k = idx >> lw, w = idx & (W - 1);
                const bool colok = w < T.ncol;
                const int qs[4] = {k, n - k, m - k, m + k};
                double y[4];
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    y[v] = (qs[v] < n && colok) ? yv[b][v] / (qs[v] == 0 ? sc1 : sc2) : 0.0;
                // V_q = e^{i pi q/(2n)} (y'_q - i y'_{n-q}) for q = k and m - k
                const double2 Vk = cmul(cconj(pk[b]), make_double2(y[0], -y[1]));
                const double2 Vmk = cmul(cconj(pmk[b]), make_double2(y[2], -y[3]));
                // Z_kk = (A + conj B) + i (A - conj B) e^{2 pi i kk / n}
                {
                    const double2 Bc = cconj(Vmk);
                    const double2 s = make_double2(Vk.x + Bc.x, Vk.y + Bc.y);
                    const double2 d = make_double2(Vk.x - Bc.x, Vk.y - Bc.y);
                    const double2 id = cmul(make_double2(-d.y, d.x), cconj(tk[b]));
                    if (k < m) z[w * cs + k] = cconj(make_double2(s.x + id.x, s.y + id.y));
                }
                if (k > 0 && m - k != k && m - k < m) {
                    const double2 Bc = cconj(Vk);
                    const double2 s = make_double2(Vmk.x + Bc.x, Vmk.y + Bc.y);
                    const double2 d = make_double2(Vmk.x - Bc.x, Vmk.y - Bc.y);
                    const double2 id = cmul(make_double2(-d.y, d.x), cconj(tmk[b]));
                    z[w * cs + (m - k)] = cconj(make_double2(s.x + id.x, s.y + id.y));
                }
            }
        }
        __syncthreads();
    }

    // ---------------- complex FFT of length m ----------------
    fft_columns<CLASS>(z, cs, a, GlobalTab{a.tw});

    // ---------------- post-processing + store ----------------
    if (inv_cos) {
        const double inv_n = 1.0 / n;
#pragma unroll 8
        for (int base = 0; base < n * W; base += blockDim.x) {
            const int idx = min(base + int(threadIdx.x), n * W - 1);
            // lanes past the tile's last column redo that column and store
            // the same value to the same place: no branch around the store
            int j = idx >> lw, w = min(idx & (W - 1), T.ncol - 1);
            int u = (j & 1) ? n - 1 - (j >> 1) : (j >> 1);
            double2 Fz = z[w * cs + (u >> 1)];
            double v = (u & 1) ? -Fz.y * inv_n : Fz.x * inv_n;
            if (kind == Z_DD && (j & 1)) v = -v;
            out[T.out_base + (long long)j * T.out_stride + w] = v;
        }
        return;
    }
    if (kind == Z_ND || kind == Z_DN) {
        for (int base = 0; base < m * W; base += kStoreBatch * blockDim.x) {
            double2 zv[kStoreBatch], tv[kStoreBatch];
#pragma unroll
            for (int b = 0; b < kStoreBatch; ++b) {
                const int idx = min(base + b * int(blockDim.x) + int(threadIdx.x), m * W - 1);
                const int k = idx >> lw, w = min(idx & (W - 1), T.ncol - 1);
                zv[b] = z[w * cs + k];
                tv[b] = ld2(a.post4, k);
            }
#pragma unroll
            for (int b = 0; b < kStoreBatch; ++b) {
            const int idx = min(base + b * int(blockDim.x) + int(threadIdx.x), m * W - 1);
            const int k = idx >> lw, w = min(idx & (W - 1), T.ncol - 1);
            double2 u = cmul(zv[b], tv[b]);
            int q0 = 2 * k, q1 = n - 1 - 2 * k;
            double y0 = sc2 * u.x, y1 = -sc2 * u.y;
            if (kind == Z_DN) {
                if (q0 & 1) y0 = -y0;
                if (q1 & 1) y1 = -y1;
            }
            out[T.out_base + (long long)q0 * T.out_stride + w] = y0;
            out[T.out_base + (long long)q1 * T.out_stride + w] = y1;
            }
        }
        return;
    }
    // PP / NN / DD: real DFT X_k (k = 0..m) from the half-length FFT
    for (int base = 0; base < (m + 1) * W; base += kStoreBatch * blockDim.x) {
        double2 tks[kStoreBatch], pks[kStoreBatch], pns[kStoreBatch];
#pragma unroll
        for (int b = 0; b < kStoreBatch; ++b) {
            const int k = min(base + b * int(blockDim.x) + int(threadIdx.x), (m + 1) * W - 1) >> lw;
            tks[b] = ld2(a.twn, k);
            pks[b] = ld2(a.post, k);
            pns[b] = ld2(a.post, n - k);
        }
#pragma unroll
        for (int b = 0; b < kStoreBatch; ++b) {
        const int idx = min(base + b * int(blockDim.x) + int(threadIdx.x), (m + 1) * W - 1);
        int k = idx >> lw, w = min(idx & (W - 1), T.ncol - 1);
        const double2 tk = tks[b], pk = pks[b], pn = pns[b];
        double2 Zk = z[w * cs + (k == m ? 0 : k)];
        double2 Zc = cconj(z[w * cs + (k == 0 ? 0 : m - k)]);
        double2 s = make_double2(0.5 * (Zk.x + Zc.x), 0.5 * (Zk.y + Zc.y));
        double2 d = make_double2(0.5 * (Zk.x - Zc.x), 0.5 * (Zk.y - Zc.y));
        double2 t = cmul(tk, d);  // e^{-2 pi i k/n} (Zk - Zc) / 2
        double2 X = make_double2(s.x + t.y, s.y - t.x);  // s - i t
        // PP: Hartley values at k and n - k; NN / DD: DCT-II
        // y_q = c_q Re(e^{-i pi q/(2n)} X_q) at q = k and n - k (X_{n-k} = conj X_k),
        // DD written in reversed order.  k = 0 and k = m have no partner: the
        // second store repeats the first.  Selects, not branches, so that the
        // loop body is one block.
        const bool pp = kind == Z_PP, dd = kind == Z_DD, pair = k > 0 && k < m;
        const double yk = pp ? sc1 * (X.x - X.y) : (k == 0 ? sc1 : sc2) * (pk.x * X.x - pk.y * X.y);
        const double yn = pp ? sc1 * (X.x + X.y) : sc2 * (pn.x * X.x + pn.y * X.y);
        const int rk = dd ? n - 1 - k : k;
        const int rn = pp ? n - k : dd ? k - 1 : n - k;
        double* o = out + T.out_base + w;
        const long long st = T.out_stride;
        o[rk * st] = yk;
        o[(pair ? rn : rk) * st] = pair ? yn : yk;
        }
    }
}

// ---------------------------------------------------------------------------
// Wide form of the same transforms, for half lengths of factors 2, 3, 5 and 7.
// A workgroup loops over tiles of W columns (z rows are segments of 8 W bytes); the
// next tile's input, 16 values a thread, is loaded into registers while the
// current tile is transformed and stored.  All tables the loop reads are in LDS: a
// load from device memory issued after the prefetch would wait for it.
//
// Bound by memory where two workgroups share a CU, by the LDS round trips of the
// stages (barriers, index arithmetic, 48 B of LDS traffic a complex value) where n
// is long.  Hence few stages of large radices (180 = 15 x 12, both in registers),
// lanes along the columns (indices and roots are the same for W lanes, and an odd
// column stride in complex values spreads a wave over the banks), division by the
// stage's stride through a high product, bins k and m - k from one pair of values,
// and for power-of-two lengths the first stage on the loaded values.  The finite
// check is a running product with zero: a flag kept across the stages spilled.
//
// TB/s, forward and inverse alike, 32 million cells, N-N / periodic z, against one
// pass per tile of short row segments with stages of radix 2 to 8:
//   n         64   96  128  200  300  360  420  600  768 1024 1200 2048
//   before   2.9  2.4  2.8  2.4  1.9  2.0  1.7  1.7  1.9  3.4  1.5  1.9
//   now      4.4  4.2  4.2  4.0  3.6  3.7  3.6  3.2  3.1  3.3  2.6  2.9
// ---------------------------------------------------------------------------

// v, hidden from the optimiser: index arithmetic built on it is redone in
// each phase of the tile loop instead of being hoisted out of the loop or
// shared between phases, which would hold it in registers throughout.
__device__ __forceinline__ int fresh(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

struct SArgs {
    int n, m, kind, lw, cs, nstage, groups;
    int radix[8], ns[8], step[8];
    unsigned magic[8];     // ceil(2^32 / ns): j / ns by the high product, j < 2^16
    const double *tw, *t1, *t2;
    int n1, n2;            // entries of t1 and t2
    int first8;            // 1: the first stage, of radix 8, runs on the loaded values
};

enum { F_PAIRS, F_COS, F_ICOS, F_QUARTER };

// One Stockham stage over the tile, in place.
template <int R>
__device__ void wide_stage(double2* z, const SArgs& a, int s, const double2* __restrict__ tw, int nthr) {
    constexpr int BPT = R >= 8 ? 1 : (8 + R - 1) / R;
    const int nbf = a.m / R, Ns = a.ns[s], step = a.step[s];
    const int total = nbf << a.lw;
    const unsigned magic = a.magic[s];
    const int tid = fresh(threadIdx.x);
    double2 v[BPT][R];
    int dst[BPT];
#pragma unroll
    for (int t = 0; t < BPT; ++t) {
        const int b = tid + t * nthr;
        dst[t] = -1;
        if (b < total) {
            const int w = b & ((1 << a.lw) - 1), j = b >> a.lw;
            const double2* col = z + w * a.cs + j;
#pragma unroll
            for (int r = 0; r < R; ++r) v[t][r] = col[r * nbf];
            int k = 0;
            if (s > 0) {
                k = j - int(__umulhi(unsigned(j), magic)) * Ns;
#pragma unroll
                for (int r = 1; r < R; ++r) v[t][r] = cmul(v[t][r], tw[k * step * r]);
            }
            dft<R>(v[t], GlobalTab{nullptr}, a.m);
            dst[t] = w * a.cs + (j - k) * R + k;
        }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < BPT; ++t) {
        if (dst[t] < 0) continue;
#pragma unroll
        for (int r = 0; r < R; ++r) z[dst[t] + r * Ns] = v[t][r];
    }
    __syncthreads();
}

// The thread's 16 inputs of a tile; lanes run over the columns first, so a wave
// reads whole row segments.  With r0 = tid / W and a pass of NT / W rows:
//   F_COS: rows r0 + e passes;
//   F_PAIRS, F_QUARTER: the two real inputs of the FFT's complex input
//     t = r0 + e passes: rows 2t and 2t + 1, or 2t and n - 1 - 2t (D-N: reversed);
//   F_ICOS: for k = r0 + g passes the rows that Z_k and Z_{m-k} need, y at k, n - k,
//     m - k, m + k (k = 0: 0, m, m / 2, 3 m / 2 for Z_0 and Z_{m/2}), reversed for D-D.
// Lanes past the end repeat the last row, columns past the tile's last read that
// one: all are discarded later.  Nothing here may use a loaded value, or the wave
// would wait for it.
template <int FORM>
__device__ __forceinline__ void wide_load(double (&r)[kWidePer], const double* __restrict__ in, const FTile& T,
                                          const SArgs& a, int nthr) {
    const int tid = fresh(threadIdx.x);
    const int W = 1 << a.lw, n = a.n, m = a.m, rpp = nthr >> a.lw;
    const int col = min(tid & (W - 1), T.ncol - 1), r0 = tid >> a.lw;
    const double* base = in + T.in_base + col;
    if (FORM == F_COS) {
#pragma unroll
        for (int e = 0; e < kWidePer; ++e) r[e] = base[(long long)min(r0 + e * rpp, n - 1) * T.in_stride];
    } else if (FORM == F_PAIRS || FORM == F_QUARTER) {
#pragma unroll
        for (int e = 0; e < kWidePer / 2; ++e) {
            const int t = min(r0 + e * rpp, m - 1);
            const int p = 2 * t, q = FORM == F_PAIRS ? 2 * t + 1 : n - 1 - 2 * t;
            r[2 * e] = base[(long long)(a.kind == Z_DN ? q : p) * T.in_stride];
            r[2 * e + 1] = base[(long long)(a.kind == Z_DN ? p : q) * T.in_stride];
        }
    } else {
        const bool rev = a.kind == Z_DD;
#pragma unroll
        for (int g = 0; g < kWidePer / 4; ++g) {
            const int k = min(r0 + g * rpp, a.groups - 1);
            const int q[4] = {k, k == 0 ? m : n - k, k == 0 ? m / 2 : m - k, k == 0 ? m + m / 2 : m + k};
#pragma unroll
            for (int v = 0; v < 4; ++v) r[4 * g + v] = base[(long long)(rev ? n - 1 - q[v] : q[v]) * T.in_stride];
        }
    }
}

template <int FORM>
__global__ void __launch_bounds__(1024) k_wide(SArgs a, const FTile* __restrict__ tiles, int ntiles,
                                                const double* __restrict__ in, double* __restrict__ out,
                                                int* nonfinite, const int* gate) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    double2* z = reinterpret_cast<double2*>(lds_raw);
    if (gate && *gate) return;  // out is left alone
    const int n = a.n, m = a.m, lw = a.lw, W = 1 << lw, cs = a.cs, nthr = blockDim.x, rpp = nthr >> lw;
    const double sc2 = sqrt(2.0 / n), sc1 = sqrt(1.0 / n);
    double2* tw = z + W * cs;
    double2* t1 = tw + m;
    double2* t2 = t1 + a.n1;
    for (int i = threadIdx.x; i < m; i += nthr) tw[i] = ld2(a.tw, i);
    for (int i = threadIdx.x; i < a.n1; i += nthr) t1[i] = ld2(a.t1, i);
    for (int i = threadIdx.x; i < a.n2; i += nthr) t2[i] = ld2(a.t2, i);
    __syncthreads();
    const int G = gridDim.x;
    int v = blockIdx.x;
    FTile T = tiles[xcd_remap(v, ntiles)];
    double r[kWidePer];
    wide_load<FORM>(r, in, T, a, nthr);
    for (;;) {
        int tid = fresh(threadIdx.x);
        {
            double chk = 0.0;  // NaN once a value is not finite
            const int w = tid & (W - 1), r0 = tid >> lw;
            const bool colok = w < T.ncol;
            double2* zc = z + w * cs;
            if (FORM == F_COS) {
#pragma unroll
                for (int e = 0; e < kWidePer; ++e) {
                    const int k = r0 + e * rpp;
                    const double x = colok ? r[e] : 0.0;
                    chk = fma(x, 0.0, chk);
                    const int u = (k & 1) ? n - 1 - (k >> 1) : (k >> 1);
                    if (k < n) reinterpret_cast<double*>(zc)[u] = (a.kind == Z_DD && (k & 1)) ? -x : x;
                }
            } else if (FORM == F_PAIRS || FORM == F_QUARTER) {
                double2 x[kWidePer / 2];
#pragma unroll
                for (int e = 0; e < kWidePer / 2; ++e) {
                    x[e] = make_double2(colok ? r[2 * e] : 0.0, colok ? r[2 * e + 1] : 0.0);
                    chk = fma(x[e].y, 0.0, fma(x[e].x, 0.0, chk));
                }
                if (a.first8) {  // rpp = m / 8: the thread holds a butterfly of the first stage
                    if (FORM == F_QUARTER)
#pragma unroll
                        for (int e = 0; e < 8; ++e) x[e] = cmul(x[e], t1[r0 + e * rpp]);
                    dft<8>(x, GlobalTab{nullptr}, m);
#pragma unroll
                    for (int e = 0; e < 8; ++e) zc[8 * r0 + e] = x[e];
                } else {
#pragma unroll
                    for (int e = 0; e < kWidePer / 2; ++e)
                        if (r0 + e * rpp < m)
                            zc[r0 + e * rpp] = FORM == F_QUARTER ? cmul(x[e], t1[r0 + e * rpp]) : x[e];
                }
            } else {
#pragma unroll
                for (int g = 0; g < kWidePer / 4; ++g) {
                    const int k = r0 + g * rpp;
                    if (k >= a.groups) continue;
                    const double y0 = colok ? r[4 * g] * (k == 0 ? 1.41421356237309504880 : 1.0) : 0.0;
                    const double y1 = colok ? r[4 * g + 1] : 0.0;
                    const double y2 = colok ? r[4 * g + 2] : 0.0;
                    const double y3 = colok ? r[4 * g + 3] : 0.0;
                    // V_q = e^{i pi q/(2n)} (y'_q - i y'_{n-q}), y'_0 = sqrt(2) y_0 (the common
                    // factor waits for the store); with A = V_k, B = V_{m-k},
                    // s = A + conj B and t = i (A - conj B) e^{2 pi i k/n}:
                    // Z_k = conj(s + t), Z_{m-k} = s - t
                    const double2 A = cmul(cconj(t2[k]), make_double2(y0, k == 0 ? 0.0 : -y1));
                    const double2 B = k == 0 ? cmul(cconj(t2[m]), make_double2(y1, -y1))
                                             : cmul(cconj(t2[m - k]), make_double2(y2, -y3));
                    const double2 sm = make_double2(A.x + B.x, A.y - B.y), d = make_double2(A.x - B.x, A.y + B.y);
                    const double2 t = cmul(make_double2(-d.y, d.x), cconj(t1[k]));
                    zc[k] = make_double2(sm.x + t.x, -(sm.y + t.y));
                    if (k > 0) {
                        zc[m - k] = make_double2(sm.x - t.x, sm.y - t.y);
                    } else if ((m & 1) == 0) {  // Z_{m/2} of A = B
                        const double2 H = cmul(cconj(t2[m / 2]), make_double2(y2, -y3));
                        const double2 th = cmul(make_double2(-2.0 * H.y, 0.0), cconj(t1[m / 2]));
                        zc[m / 2] = make_double2(2.0 * H.x + th.x, -th.y);
                    }
                }
            }
            if (FORM != F_ICOS && chk != 0.0 && nonfinite) atomicOr(nonfinite, 1);
        }
        const int vn = v + G;
        FTile Tn = T;
        if (vn < ntiles) {
            Tn = tiles[xcd_remap(vn, ntiles)];
            wide_load<FORM>(r, in, Tn, a, nthr);
        }
        __syncthreads();
        for (int s = a.first8; s < a.nstage; ++s) {
            switch (a.radix[s]) {
                case 2: wide_stage<2>(z, a, s, tw, nthr); break;
                case 3: wide_stage<3>(z, a, s, tw, nthr); break;
                case 4: wide_stage<4>(z, a, s, tw, nthr); break;
                case 5: wide_stage<5>(z, a, s, tw, nthr); break;
                case 6: wide_stage<6>(z, a, s, tw, nthr); break;
                case 7: wide_stage<7>(z, a, s, tw, nthr); break;
                case 8: wide_stage<8>(z, a, s, tw, nthr); break;
                case 9: wide_stage<9>(z, a, s, tw, nthr); break;
                case 10: wide_stage<10>(z, a, s, tw, nthr); break;
                case 12: wide_stage<12>(z, a, s, tw, nthr); break;
                case 15: wide_stage<15>(z, a, s, tw, nthr); break;
                default: wide_stage<16>(z, a, s, tw, nthr); break;
            }
        }
        tid = fresh(threadIdx.x);
        const int w = tid & (W - 1), r0 = tid >> lw;
        const double2* zc = z + w * cs;
        double* o = out + T.out_base + w;
        const long long st = T.out_stride;
        if (w < T.ncol) {
            if (FORM == F_ICOS) {
                const double scale = sqrt(0.5 / n);
#pragma unroll
                for (int e = 0; e < kWidePer; ++e) {
                    const int j = r0 + e * rpp;
                    if (j >= n) continue;
                    const int u = (j & 1) ? n - 1 - (j >> 1) : (j >> 1);
                    const double y = reinterpret_cast<const double*>(zc)[u] * scale;
                    const bool neg = ((u & 1) != 0) != (a.kind == Z_DD && (j & 1));  // conjugate; (-1)^j of D-D
                    o[j * st] = neg ? -y : y;
                }
            } else if (FORM == F_QUARTER) {
#pragma unroll
                for (int e = 0; e < kWidePer / 2; ++e) {
                    const int k = r0 + e * rpp;
                    if (k >= m) continue;
                    const double2 u = cmul(zc[k], t2[k]);
                    const int q0 = 2 * k, q1 = n - 1 - 2 * k;  // even and odd
                    o[q0 * st] = sc2 * u.x;
                    o[q1 * st] = a.kind == Z_DN ? sc2 * u.y : -sc2 * u.y;
                }
            } else {
                const bool dd = a.kind == Z_DD;
#pragma unroll
                for (int g = 0; g < kWidePer / 4; ++g) {
                    const int k = r0 + g * rpp;
                    if (k >= a.groups) continue;
                    auto put = [&](int row, double y) { o[(dd ? n - 1 - row : row) * st] = y; };
                    // outputs q and n - q of the real DFT value X_q
                    auto both = [&](int q, double2 X) {
                        if (FORM == F_PAIRS) {
                            put(q, sc1 * (X.x - X.y));
                            put(n - q, sc1 * (X.x + X.y));
                        } else {
                            const double2 p = t2[q];  // post[n - q] = -i conj(post[q])
                            put(q, sc2 * (p.x * X.x - p.y * X.y));
                            put(n - q, -sc2 * (p.y * X.x + p.x * X.y));
                        }
                    };
                    const double2 Z = zc[k];
                    if (k > 0) {
                        const double2 Y = zc[m - k];
                        const double2 s = make_double2(0.5 * (Z.x + Y.x), 0.5 * (Z.y - Y.y));
                        const double2 d = make_double2(0.5 * (Z.x - Y.x), 0.5 * (Z.y + Y.y));
                        const double2 t = cmul(t1[k], d);
                        both(k, make_double2(s.x + t.y, s.y - t.x));
                        both(m - k, make_double2(s.x - t.y, -s.y - t.x));
                    } else {
                        const double x0 = Z.x + Z.y, xm = Z.x - Z.y;
                        put(0, sc1 * x0);
                        put(m, FORM == F_PAIRS ? sc1 * xm : sc2 * t2[m].x * xm);
                        if ((m & 1) == 0) {
                            const double2 H = zc[m / 2];
                            both(m / 2, make_double2(H.x, -H.y));
                        }
                    }
                }
            }
        }
        if (vn >= ntiles) break;
        __syncthreads();
        T = Tn;
        v = vn;
    }
}

int fft_col_stride(const mbp_plan* P);

// Columns per workgroup, a power of two up to 64: wide tiles read long row
// segments and amortise the stage barriers.  Each stage gives a thread at
// most 16 complex values (4 butterflies of radix 4, 8 of radix 2, 2 of the
// radices 3 to 8, 1 of the larger ones).  The LDS image W * cs complex
// values is held to 40 KB (four workgroups per CU) unless that leaves fewer
// than 8 columns, then to 80 KB (two per CU).
constexpr int64_t kFFTLdsSmall = 40 * 1024;
constexpr int64_t kFFTLds = 80 * 1024;

static int fft_width_for(const mbp_plan* P, int64_t lds) {
    const int m = P->fft.m;
    int W = 64;
    while (W > 1 && int64_t(W) * fft_col_stride(P) * 16 > std::min<int64_t>(lds, P->lds_limit)) W >>= 1;
    for (int R : P->fft.radices) {
        const int per = R > 8 ? 1 : (R == 2 ? 8 : R == 4 ? 4 : 2);  // butterflies per thread
        while (W > 1 && W * (m / R) > per * 256) W >>= 1;
        if (R > 31)  // the any-radix stage holds W m / 256 outputs per thread
            while (W > 1 && W * m > kGenericOut * 256) W >>= 1;
    }
    return W;
}

int fft_columns_per_wg(const mbp_plan* P) {
    if (P->fft.W) return P->fft.W;
    const int W = fft_width_for(P, kFFTLdsSmall);
    return W >= 8 ? W : fft_width_for(P, kFFTLds);
}

// Column stride in complex values: one padding slot breaks the power-of-two
// bank pattern when the padded image still fits.
int fft_col_stride(const mbp_plan* P) {
    const int m = P->fft.m;
    return (int64_t(8) * (m + 1) * 16 <= std::min<int64_t>(kFFTLds, P->lds_limit)) ? m + 1 : m;
}

void fft_build_tiles(const mbp_plan* P, std::vector<unsigned char>& fwd, std::vector<unsigned char>& inv,
                     int* ntiles) {
    const int W = fft_columns_per_wg(P);
    std::vector<FTile> f, iv;
    for (int b = 0; b < P->g.nb; ++b) {
        long long cols = (long long)P->g.nx[b] * P->g.ny[b];
        long long off2 = P->levels[0].off[b];
        for (long long c0 = 0; c0 < cols; c0 += W) {
            FTile t{};
            t.ncol = int(std::min<long long>(W, cols - c0));
            t.in_base = P->block_off[b] + c0;
            t.in_stride = int(cols);
            t.out_base = off2 + c0;
            t.out_stride = int(P->plane0);
            f.push_back(t);
            FTile u{};
            u.ncol = t.ncol;
            u.in_base = off2 + c0;
            u.in_stride = int(P->plane0);
            u.out_base = P->block_off[b] + c0;
            u.out_stride = int(cols);
            iv.push_back(u);
        }
    }
    *ntiles = int(f.size());
    fwd.assign(reinterpret_cast<unsigned char*>(f.data()),
               reinterpret_cast<unsigned char*>(f.data()) + f.size() * sizeof(FTile));
    inv.assign(reinterpret_cast<unsigned char*>(iv.data()),
               reinterpret_cast<unsigned char*>(iv.data()) + iv.size() * sizeof(FTile));
}

static FFTArgs make_args(const mbp_plan* P) {
    FFTArgs a{};
    a.n = P->fft.n;
    a.m = P->fft.m;
    a.kind = P->g.zkind;
    a.W = fft_columns_per_wg(P);
    a.cs = fft_col_stride(P);
    a.nstage = int(P->fft.radices.size());
    for (int s = 0; s < a.nstage && s < 16; ++s) a.radix[s] = P->fft.radices[s];
    a.tw = P->d_dbl + P->fft_tw;
    a.twn = P->d_dbl + P->fft_twn;
    a.post = P->d_dbl + P->fft_post;
    a.pre4 = P->d_dbl + P->fft_pre4;
    a.post4 = P->d_dbl + P->fft_post4;
    return a;
}

static size_t lds_bytes(const mbp_plan* P) {
    const size_t img = size_t(fft_columns_per_wg(P)) * fft_col_stride(P);
    return img * sizeof(double2);
}

static int radix_class(const mbp_plan* P) {
    int c = 0;
    for (int R : P->fft.radices) {
        if (R == 3 || R == 5 || R == 7) c = std::max(c, 1);
        else if (R > 31) c = 3;
        else if (R > 8) c = std::max(c, 2);
    }
    return c;
}

template <int CLASS>
static void launch_r2r(const mbp_plan* P, const FFTArgs& a, const void* tiles, int dir, const double* in,
                       double* out, int* nonfinite, const int* gate, hipStream_t s) {
    const size_t bytes = lds_bytes(P);
    if (bytes > 64 * 1024)
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k_r2r<CLASS>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
    hipLaunchKernelGGL(k_r2r<CLASS>, dim3(P->fft_ntiles), dim3(256), bytes, s, a,
                       reinterpret_cast<const FTile*>(tiles), P->fft_ntiles, dir, in, out, nonfinite, gate);
}

static const void* wide_fn(int form) {
    return form == F_PAIRS    ? reinterpret_cast<const void*>(k_wide<F_PAIRS>)
           : form == F_COS    ? reinterpret_cast<const void*>(k_wide<F_COS>)
           : form == F_ICOS   ? reinterpret_cast<const void*>(k_wide<F_ICOS>)
                              : reinterpret_cast<const void*>(k_wide<F_QUARTER>);
}
static int wide_form(int kind, int dir) {
    return kind == Z_PP ? F_PAIRS : kind == Z_ND || kind == Z_DN ? F_QUARTER : dir ? F_ICOS : F_COS;
}

// A grid of as many workgroups as fit on the current device at once (a multiple of
// 8, so each keeps its XCD's share of tiles), at most one per tile.
int fft_setup_grid(mbp_plan* P) {
    FFTPlan& F = P->fft;
    if (!F.W) return MBP_OK;
    int dev = 0, ncu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return MBP_ERR_HIP;
    for (int dir = 0; dir < 2; ++dir) {
        const void* fn = wide_fn(wide_form(P->g.zkind, dir));
        const size_t bytes = F.bytes;
        int per = 0;
        if (bytes > 64 * 1024 &&
            hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes)) != hipSuccess)
            return MBP_ERR_HIP;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, F.nt, bytes) != hipSuccess) return MBP_ERR_HIP;
        int g = std::min<int64_t>(P->fft_ntiles, int64_t(std::max(per, 1)) * std::max(ncu, 1));
        if (g >= 8) g -= g % 8;
        F.grid[dir] = std::max(g, 1);
    }
    return MBP_OK;
}

static void run_wide(const mbp_plan* P, const void* tiles, int dir, const double* in, double* out, int* nonfinite,
                     const int* gate, hipStream_t s) {
    const FFTPlan& F = P->fft;
    SArgs a{};
    a.n = F.n;
    a.m = F.m;
    a.kind = P->g.zkind;
    a.lw = __builtin_ctz(unsigned(F.W));
    a.cs = F.m | 1;
    a.nstage = int(F.wide.size());
    a.first8 = F.first8;
    for (int i = 0, Ns = 1; i < a.nstage; ++i) {
        a.radix[i] = F.wide[i];
        a.ns[i] = Ns;
        a.step[i] = a.m / (Ns * F.wide[i]);
        a.magic[i] = unsigned(((1ull << 32) + Ns - 1) / Ns);
        Ns *= F.wide[i];
    }
    const bool quarter = a.kind == Z_ND || a.kind == Z_DN;
    a.groups = (a.m + 1) / 2;
    a.tw = P->d_dbl + P->fft_tw;
    a.t1 = P->d_dbl + (quarter ? P->fft_pre4 : P->fft_twn);
    a.n1 = quarter ? a.m : a.m / 2 + 1;
    a.t2 = P->d_dbl + (quarter ? P->fft_post4 : P->fft_post);
    a.n2 = quarter ? a.m : a.kind == Z_PP ? 0 : a.m + 1;
    const size_t bytes = F.bytes;
    const void* fn = wide_fn(wide_form(a.kind, dir));
    if (bytes > 64 * 1024)
        (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
    const FTile* tl = reinterpret_cast<const FTile*>(tiles);
    int ntiles = P->fft_ntiles;
    void* args[] = {&a, &tl, &ntiles, &in, &out, &nonfinite, &gate};
    (void)hipLaunchKernel(fn, dim3(F.grid[dir]), dim3(F.nt), args, bytes, s);
}

static void run_r2r(const mbp_plan* P, const void* tiles, int dir, const double* in, double* out,
                    int* nonfinite, const int* gate, hipStream_t s) {
    if (P->fft.W) return run_wide(P, tiles, dir, in, out, nonfinite, gate, s);
    const FFTArgs a = make_args(P);
    switch (radix_class(P)) {
        case 0: launch_r2r<0>(P, a, tiles, dir, in, out, nonfinite, gate, s); break;
        case 1: launch_r2r<1>(P, a, tiles, dir, in, out, nonfinite, gate, s); break;
        case 2: launch_r2r<2>(P, a, tiles, dir, in, out, nonfinite, gate, s); break;
        default: launch_r2r<3>(P, a, tiles, dir, in, out, nonfinite, gate, s); break;
    }
}

void launch_forward(const mbp_plan* P, const double* f, double* fhat, int* nonfinite, hipStream_t s) {
    run_r2r(P, P->d_ftiles_fwd, 0, f, fhat, nonfinite, nullptr, s);
}

void launch_inverse(const mbp_plan* P, const double* phat, double* p, hipStream_t s, const int* gate) {
    run_r2r(P, P->d_ftiles_inv, 1, phat, p, nullptr, gate, s);
}

}  // namespace mbp
