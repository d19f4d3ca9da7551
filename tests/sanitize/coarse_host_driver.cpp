// Host check of the LDS-resident levels (coarse.hip): every cell of every level has a
// thread, and the LDS image fits, over layouts whose colours are uneven or whose blocks
// are many and small, and over seeded random grids of blocks.  Runs no HIP call.
#include <cstdio>
#include <random>
#include <string>
#include <vector>

#include "internal.h"

namespace {

const int D = MBP_DIRICHLET, N = MBP_NEUMANN, C = MBP_CONNECT;
constexpr int kLevInts = 12;  // ints a level descriptor: cells, cells of colours 0..3, ..., the last: odd rings
int failures = 0, formed = 0;

struct Layout {
    std::vector<std::vector<double>> xf, yf;
    std::vector<mbp_block_desc> b;
    void add(int x0, int y0, int nx, int ny, int bxm, int bxp, int bym, int byp) {
        std::vector<double> x(nx + 1), y(ny + 1);
        for (int i = 0; i <= nx; ++i) x[i] = (x0 - 1 + i) / 32.0;
        for (int j = 0; j <= ny; ++j) y[j] = (y0 - 1 + j) / 32.0;
        xf.push_back(x);
        yf.push_back(y);
        mbp_block_desc d{};
        d.lo[0] = x0;
        d.lo[1] = y0;
        d.hi[0] = x0 + nx - 1;
        d.hi[1] = y0 + ny - 1;
        d.bc[0] = bxm;
        d.bc[1] = bxp;
        d.bc[2] = bym;
        d.bc[3] = byp;
        b.push_back(d);
    }
};

// columns w x rows h of joined blocks, some missing
Layout grid(const std::vector<int>& w, const std::vector<int>& h, const std::vector<char>& gone) {
    Layout L;
    auto have = [&](int i, int j) {
        return i >= 0 && j >= 0 && i < int(w.size()) && j < int(h.size()) && !gone[size_t(j) * w.size() + i];
    };
    int y = 1;
    for (int j = 0; j < int(h.size()); y += h[j++]) {
        int x = 1;
        for (int i = 0; i < int(w.size()); x += w[i++])
            if (have(i, j))
                L.add(x, y, w[i], h[j], have(i - 1, j) ? C : D, have(i + 1, j) ? C : N, have(i, j - 1) ? C : N,
                      have(i, j + 1) ? C : D);
    }
    return L;
}

// -1: refused; 0: the generic kernels run; 1: coarse.hip does, and everything fits
int check(const char* name, Layout& L, int precision, bool must_plan = true) {
    std::vector<mbp_block_desc> d = L.b;
    for (size_t i = 0; i < d.size(); ++i) {
        d[i].xf = L.xf[i].data();
        d[i].yf = L.yf[i].data();
    }
    mbp_synth_desc z{8, 0.25, N, N};
    mbp_options o;
    mbp::options_default(&o);
    o.precision = precision;
    mbp_plan P;
    std::string err;
    const int64_t limit = 160 * 1024;
    const int st = mbp::build_plan_host_limits(d.data(), int(d.size()), &z, &o, limit, &P, &err);
    auto fail = [&](const char* what, long long a, long long b) {
        std::fprintf(stderr, "FAIL %s precision %d: %s (%lld, %lld)\n", name, precision, what, a, b);
        ++failures;
    };
    if (st != MBP_OK) {
        if (must_plan) fail(err.c_str(), st, 0);
        return -1;
    }
    (void)mbp::plan_device_bytes(&P);
    const mbp::CoarseInfo& ci = P.coarse;
    const int top = precision == MBP_MIXED ? P.lds_level32 : P.lds_level;
    if (!ci.ok) {
        const int64_t bytes = precision == MBP_MIXED ? P.lds_bytes32 : P.lds_bytes64;
        if (bytes > limit) fail("generic kernels: LDS", bytes, limit);
        return 0;
    }
    ++formed;
    if (ci.bytes > limit) fail("LDS", ci.bytes, limit);
    if (ci.nthr < 64 || ci.nthr > 512) fail("threads", ci.nthr, 512);
    for (int k = 0; k < ci.nl; ++k) {
        const int* v = &P.hint[ci.lev + kLevInts * k];
        if (v[0] != P.levels[top + k].plane || v[1] + v[2] + v[3] + v[4] != v[0]) fail("cells of a level", v[0], k);
        const bool odd = v[kLevInts - 1] != 0;  // (looped over, whatever their count)
        const int most = std::max(v[1], v[2]);
        if (odd || k + 1 == ci.nl) continue;
        if (v[3] || v[4]) fail("extra colours on an even level", k, v[3] + v[4]);
        if (k == 0 && most > ci.per * ci.nthr) fail("cells of a colour on the top level", most, ci.per * ci.nthr);
        if (k > 0 && most > ci.nthr) fail("cells of a colour on a lower level", most, ci.nthr);
        if (k >= ci.ls && most > 64) fail("cells of a colour in the single wave", most, 64);
    }
    return 1;
}

}  // namespace

int main() {
    for (int precision : {MBP_FP64, MBP_MIXED}) {
        // a T of 4096 cells whose second level has 511 and 513 cells of the two
        // colours; and the same one level up
        for (int s : {1, 2}) {
            Layout t;
            t.add(34 * s + 1, 30 * s + 1, 30 * s, 34 * s, C, C, C, D);
            t.add(1, 30 * s + 1, 34 * s, 34 * s, D, C, N, N);
            t.add(64 * s + 1, 30 * s + 1, 30 * s, 34 * s, C, N, D, N);
            t.add(34 * s + 1, 1, 30 * s, 30 * s, N, D, N, C);
            check(s == 1 ? "T" : "T of twice the size", t, precision);
        }
        // many small blocks: their tables fill the LDS
        for (int n : {6, 8})
            for (int c : {8, 16}) {
                Layout g = grid(std::vector<int>(n, c), std::vector<int>(n, c), std::vector<char>(n * n, 0));
                check("grid of small blocks", g, precision);
            }
        // planes of odd blocks, all of one colour's majority
        for (int n : {3, 5, 7}) {
            Layout g = grid(std::vector<int>(n, 9), std::vector<int>(n, 9), std::vector<char>(n * n, 0));
            check("grid of odd blocks", g, precision);
        }
        // ordinary planes keep the form
        for (int n : {16, 33, 64}) {
            Layout b;
            b.add(1, 1, n, n, D, N, N, D);
            if (check("box", b, precision) != 1) {
                std::fprintf(stderr, "FAIL box %d precision %d: the form is not taken\n", n, precision);
                ++failures;
            }
        }
    }
    std::mt19937 rng(64);
    auto uni = [&](int a, int b) { return std::uniform_int_distribution<int>(a, b)(rng); };
    for (int s = 0; s < 400; ++s) {
        const int nx = uni(1, 6), ny = uni(1, 6), even = uni(0, 2), most = uni(8, 40);
        auto size = [&]() {
            const int n = uni(4, most);
            return even ? n & ~1 : n;
        };
        std::vector<int> w(nx), h(ny);
        for (int& v : w) v = size();
        for (int& v : h) v = size();
        std::vector<char> gone(size_t(nx) * ny, 0);
        for (char& v : gone) v = uni(0, 4) == 0;
        gone[uni(0, nx * ny - 1)] = 0;
        Layout g = grid(w, h, gone);
        check("random grid", g, s & 1 ? MBP_MIXED : MBP_FP64, false);
    }
    std::printf("%s (%d failures, %d plans in the form)\n", failures ? "FAILED" : "OK", failures, formed);
    return failures ? 1 : 0;
}
