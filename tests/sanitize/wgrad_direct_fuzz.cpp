// Host-only fuzz of the direct filter gradient's planning (wd_setup in setup.cpp), built with -fsanitize=address,undefined by
// tests/test_direct_planning.py: for random layers what the kernel (wgrad_direct.hip) reads and writes is replayed from the
// tables -- every output pixel of every image once in each tile, the tap's own pixel of x beside it, nothing outside the tensors,
// LDS or the workspace, every filter and column of dw once.  Nothing here touches a GPU.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../../paper_2002_00552_amd/csrc/plan.hpp"
using namespace dwm;
static uint64_t g = 0x9E3779B97F4A7C15ull;
static uint32_t rnd() { g ^= g << 13; g ^= g >> 7; g ^= g << 17; return (uint32_t)(g >> 32); }
static int pick(int lo, int hi) { return lo + (int)(rnd() % (uint32_t)(hi - lo + 1)); }
#define CHECK(c)                                                              \
    do {                                                                      \
        if (!(c)) {                                                           \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #c); \
            std::exit(2);                                                     \
        }                                                                     \
    } while (0)
static int dv(const FastDiv& f, int n) { return (int)(((((unsigned long long)(unsigned)n * f.mul) >> 32) + (unsigned)n) >> f.shift); }

static void replay(const WdArgs& A)
{
    const int KT = 32 * A.mb, CT = 32 * A.nb, RS = A.R * A.S, plane = A.rows * A.pcols, PW = 1 << A.lgw, PH = 16 >> A.lgw, mask = PW - 1;
    const size_t pitch = KT * 48 + 16;
    CHECK(A.cols == A.C * RS && A.lds_bytes <= 80 * 1024 && A.lds_bytes >= 16 * 1024);
    CHECK(A.ntiles % A.nkt == 0);
    std::vector<char> units((size_t)A.nunits, 0);
    CHECK(A.stride % 64 == 0 && A.stride >= A.K * A.cols);
    std::vector<int> tiles((size_t)A.pieces * A.ntiles, 0);
    for (int b = 0; b < A.pieces * A.ntiles; ++b) {
        const int ranges = A.nunits < 8 ? A.nunits : 8, range = b % ranges, r0 = b / ranges, tile = r0 % A.ntiles, piece = r0 / A.ntiles * ranges + range;
        CHECK(piece < A.pieces);
        ++tiles[(size_t)piece * A.ntiles + tile];
        const int first = range * A.xunits, end = std::min(first + A.xunits, A.nunits);
        if (tile == 0)
            for (int u = first + r0 / A.ntiles; u < end; u += A.ustep) CHECK(u < A.nunits && !units[u]++);
    }
    for (int v : tiles) CHECK(v == 1);
    for (char v : units) CHECK(v == 1);
    CHECK(A.ntiles / A.nkt * CT >= A.cols && A.nkt * KT >= A.K);
    std::vector<char> seen((size_t)A.N * A.OH * A.OW, 0);
    for (int ct = 0; ct < A.ntiles / A.nkt; ++ct) {
        const int clo = dv(A.div_rs, ct * CT), chi = dv(A.div_rs, std::min(ct * CT + CT, A.cols) - 1), npix = (chi - clo + 1) * plane;
        CHECK(clo == ct * CT / RS && chi < A.C);
        CHECK(16 * pitch + (size_t)npix * 48 <= A.lds_bytes);
        if (ct > 1 && ct + 1 < A.ntiles / A.nkt && rnd() % 4) continue;
        for (int u = 0; u < A.nunits; ++u) {
            const int t = dv(A.div_npx, u), px = u - t * A.npx, gr = dv(A.div_npy, t), py0 = (t - gr * A.npy) * PH, ow0 = px << A.lgw;
            CHECK(px >= 0 && px < A.npx && py0 < A.npy * PH);
            if (ct > 0 && u > 2 && rnd() % 8) continue;
            for (int e = 0; e < 8; ++e) {
                const int vi = gr * 8 + e, n = dv(A.div_nb, vi), oh0 = (vi - n * A.NB) * A.BH;
                CHECK(n == vi / A.NB);
                std::vector<long long> sx((size_t)npix, -2);
                for (int i = 0; i < npix; ++i) {
                    const int c = dv(A.div_plane, i), r = i - c * plane, row = dv(A.div_pcols, r), iw = A.s * ow0 - A.P + r - row * A.pcols;
                    const int ih = A.s * py0 - A.P + A.s * oh0 + row;
                    CHECK(c <= chi - clo && row < A.rows);
                    const bool in = n < A.N && (unsigned)iw < (unsigned)A.W && (unsigned)ih < (unsigned)A.H;
                    const long long at = in ? (long long)(clo + c) * A.H * A.W + iw + (long long)ih * A.W : -1;
                    if (in) CHECK(at >= 0 && at < (long long)A.C * A.H * A.W && at * 4 < (1LL << 31));
                    // (the offset the kernel forms, from the image's row `top`, without a sign)
                    if (in) CHECK((long long)(uint32_t)(((clo + c) * A.H + row) * A.W + iw) * 4 < 0x7ffffff0LL);
                    sx[i] = at;
                }
                for (int p = 0; p < 16; ++p) {
                    const int ol = py0 + (p >> A.lgw), oh = oh0 + ol, ow = ow0 + (p & mask);
                    const bool in = ol < A.BH && ow < A.OW && n < A.N && oh < A.OH;
                    if (in) CHECK(((long long)(A.nkt * KT) * A.OH * A.OW + (long long)ol * A.OW + ow) * 4 < 0x80000000LL && ow0 + (p & mask) >= 0);
                    if (in && ct == 0) CHECK(!seen[((size_t)n * A.OH + oh) * A.OW + ow]++);
                    for (int j = 0; j < CT; j += (ct || u > 4 ? 7 : 1)) {
                        const int col = std::min(ct * CT + j, A.cols - 1), c = col / RS, tap = col - c * RS, r = tap / A.S, q = tap - r * A.S;
                        const int at = (c - clo) * plane + r * A.pcols + q + (p >> A.lgw) * A.s * A.pcols + (p & mask) * A.s;
                        CHECK(at >= 0 && at < npix && sx[at] != -2);
                        if (!in) continue;
                        const int ih = A.s * oh + r - A.P, iw = A.s * ow + q - A.P;
                        const long long want = (unsigned)ih < (unsigned)A.H && (unsigned)iw < (unsigned)A.W ? ((long long)c * A.H + ih) * A.W + iw : -1;
                        CHECK(sx[at] == want);
                    }
                }
            }
        }
    }
    for (char v : seen) CHECK(v == 1);
}

int main(int argc, char** argv)
{
    const int iters = argc > 1 ? std::atoi(argv[1]) : 100;
    int n = 0, took = 0, shapes[3][6] = {};
    for (int it = 0; it < iters; ++it) {
        const int R = pick(1, 11), S = rnd() % 2 ? R : pick(1, 11), s = pick(1, 4), P = pick(0, 5), N = rnd() % 2 ? pick(1, 9) : pick(1, 70);
        const int C = rnd() % 2 ? pick(1, 5) : pick(6, 60), K = rnd() % 2 ? pick(1, 40) : pick(41, 200);
        const int H = pick(1, rnd() % 4 ? 14 : 30), W = pick(1, rnd() % 4 ? 20 : 60);
        if (H + 2 * P < R || W + 2 * P < S) continue;
        const int OH = (H + 2 * P - R) / s + 1, OW = (W + 2 * P - S) / s + 1;
        WdArgs a;
        ++n;
        if (!wd_setup(N, C, H, W, K, R, S, s, P, OH, OW, &a)) continue;
        ++took;
        ++shapes[a.mb][a.nb];
        if ((long long)a.nunits * a.ntiles < 4000) replay(a);
    }
    CHECK(took * 4 > n * 3);
    std::printf("wgrad direct fuzz: %d of %d layers planned and replayed; tiles", took, n);
    for (int m = 1; m <= 2; ++m)
        for (int b = 1; b <= 5; ++b) std::printf(" %dx%d:%d", 32 * m, 32 * b, shapes[m][b]);
    std::printf("\n");
}
