// Host-only fuzz of the direct convolution's planning (setup.cpp), built with -fsanitize=address,undefined by
// tests/test_direct_planning.py: for random layers, forward and data gradient, every shape of the workgroup, what the kernel
// (direct.hip) and its filter transform read and write is replayed from the tables -- every tap and channel once, staged pixels where the
// taps look for them, every output once, nothing outside the tensors, the filter's copies or LDS.  Nothing here touches a GPU.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>
#include <algorithm>
#include "../../paper_2002_00552_amd/csrc/plan.hpp"
namespace dwm {
dwm_status_t launch_filter_transform(const dwm_plan&, const float*, float*, void*) { return DWM_OK; }
dwm_status_t launch_input_transform(const dwm_plan&, const float*, float*, void*) { return DWM_OK; }
dwm_status_t launch_contract_output(const dwm_plan&, const float*, float*, float*, void*) { return DWM_OK; }
dwm_status_t launch_fused_forward(const dwm_plan&, const float*, const float*, float*, void*) { return DWM_OK; }
dwm_status_t launch_direct(const dwm_plan&, const float*, const float*, float*, float*, void*) { return DWM_OK; }
}
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

static int dv(const FastDiv& f, int n) { int q = (int)(((((unsigned long long)(unsigned)n * f.mul) >> 32) + (unsigned)n) >> f.shift); return q; }

// Every tap that the filter transform reads from `F` for these problems: the one meant (tap r, s of problem i is tap
// (oy_i + step*r, ox_i + step*s) of the R x S filter whose element strides are ks, cs), and so inside w
struct Taps { int oh, ow, step; };
static void reads(const DirectArgs& A, const FilterSource& F, const std::vector<Taps>& taps, long long ks, long long cs, int R, int S) {
    for (int i = 0; i < A.nprob; ++i) for (int r = 0; r < A.p[i].R; ++r) for (int s = 0; s < A.p[i].S; ++s) {
        const int wr = taps[i].oh + taps[i].step * r, ws = taps[i].ow + taps[i].step * s;
        CHECK(wr >= 0 && wr < R && ws >= 0 && ws < S);
        for (int k : {0, A.K - 1}) for (int c : {0, A.C - 1}) CHECK(A.p[i].at(F, k, c, r, s) == k * ks + c * cs + (long long)wr * S + ws);
    }
}

static void replay(const DirectArgs& A, bool full) {
    const DirectShape& sh = kDirectShapes[A.shape];
    const int NT = sh.threads(), NPX = A.npx;
    CHECK(A.P <= A.ns * NT && A.ns <= kDirectSlots && A.lds_bytes <= (NT <= 256 ? 80 : 160) * 1024u);
    CHECK(A.groups[1] <= A.groups[0] && A.groups[1] >= 1);
    // the pieces take every chunk once, none is without one, and their outputs lie apart
    CHECK(A.pieces >= 1 && A.pieces <= kDirectMaxPieces && (A.pieces - 1) * A.cpp < A.nchunks && A.pieces * A.cpp >= A.nchunks);
    CHECK(A.pieces == 1 ? A.piece_floats == 0 && A.cpp == A.nchunks : A.nprob == 1 && A.piece_floats >= (size_t)A.N * A.K * A.YH * A.YW);
    CHECK((A.nchunks - 1) * A.groups[0] + A.groups[1] == (A.C + 7) / 8);
    const size_t total = (size_t)A.N * A.C * A.H * A.W, image = (size_t)A.C * A.H * A.W;
    const int per = A.nkt * A.nprob;
    std::vector<char> tiles(A.ntiles, 0);
    // filter: every tap and channel of every problem once; Wd and W32 inside their sizes
    int steps = 0, longest = 0; long long w32 = 0;
    for (int i = 0; i < A.nprob; ++i) {
        const DirectProb& q = A.p[i];
        CHECK(q.step0 == steps && q.w32 == w32);
        const int taps = q.R * q.S;
        std::vector<int> seen((size_t)taps * A.C, 0);
        const int n = (A.nchunks - 1) * q.steps[0] + q.steps[1];
        for (int rel = 0; rel < n; ++rel) for (int h = 0; h < 2; ++h) {
            const int chunk = std::min(rel / q.steps[0], A.nchunks - 1), st = rel - chunk * q.steps[0];
            const int G = chunk == A.nchunks - 1 ? A.groups[1] : A.groups[0], unit = 2 * st + h, tap = unit / G;
            const int c0 = (chunk * A.groups[0] + unit - tap * G) * 8, r = tap / q.S;
            for (int e = 0; e < 8; ++e) if (r < q.R && c0 + e < A.C) seen[(size_t)tap * A.C + c0 + e]++;
        }
        for (int v : seen) CHECK(v == 1);
        steps += n; w32 += (long long)taps * A.C * A.Kpad;
        // the longest of a wave's sums: its share of every chunk of its piece (of the longest piece)
        for (int first = 0; first < A.nchunks; first += A.cpp) {
            int sum = 0;
            for (int c = first; c < std::min(first + A.cpp, A.nchunks); ++c)
                for (int st = 0; st < q.steps[c == A.nchunks - 1]; st += sh.wk) ++sum;
            longest = std::max(longest, sum);
        }
    }
    CHECK(longest <= A.longest && (A.pieces > 1 || longest == A.longest) && A.two_level == (A.longest > (sh.wk > 1 ? 112 : 80)));
    CHECK(steps == A.all_steps && (size_t)w32 == A.w32_floats && A.wd_bytes == (unsigned)steps * 96u * A.Kpad);
    std::vector<std::vector<char>> outs(A.nprob);
    for (int i = 0; i < A.nprob; ++i) outs[i].assign(full ? (size_t)A.N * A.p[i].OH * A.p[i].OW : 0, 0);
    for (int t = 0; t < A.ntiles; ++t) {
        const bool low = t < A.full8; const int r0 = low ? t >> 3 : t - A.full8;
        const int place = r0 % per, tt = low ? (r0 / per) * 8 + (t & 7) : (A.ntt / 8) * 8 + r0 / per;
        const int inner = (r0 - place) / 32 % 2 == 0 ? place : per - 1 - place, pi = inner / A.nkt, kt = inner - pi * A.nkt;
        CHECK(kt < A.nkt && tt < A.ntt && pi < A.nprob);
        CHECK(!tiles[tt * per + inner]); tiles[tt * per + inner] = 1;
        if (kt != 0 || (!full && t > 0 && rnd() % 8)) continue;
        const DirectProb& q = A.p[pi];
        const int p0 = tt * NPX, g0 = dv(A.div_bw, p0), v0 = dv(A.div_oh, g0), oh0 = g0 - v0 * A.OH, n0 = dv(A.div_strips, v0);
        CHECK(g0 == p0 / A.bw && v0 == g0 / A.OH && n0 == v0 / A.nstrips && n0 < A.N);
        const int nr0 = A.rstep * (A.OH - 1 - oh0) + A.run;
        const size_t left = ((size_t)(A.N - n0) * image + A.bias) * 4;
        const uint32_t nrec = (uint32_t)std::min<size_t>(left, 0x7ffffff0u);
        auto load = [&](uint32_t vo, uint32_t so) -> long long {
            if (vo & 0x80000000u) return -1;
            const uint64_t at = (uint64_t)vo + so;
            CHECK(at < nrec);
            const long long idx = (long long)n0 * (long long)image - A.bias + (long long)(at / 4);
            CHECK(idx >= 0 && (size_t)idx < total);
            return idx;
        };
        for (int chunk = 0; chunk < A.nchunks; ++chunk) {
            if (chunk > 0 && chunk < A.nchunks - 1 && rnd() % 4) continue;
            const bool last = chunk == A.nchunks - 1;
            const int G = last ? A.groups[1] : A.groups[0];
            std::vector<long long> lds((size_t)A.groups[0] * A.P * 8, -2);
            for (int gg = 0; gg < G; ++gg) for (int px = 0; px < A.P; ++px) {
                const int j = dv(A.div_row, px), pc = px - j * A.row_px, ph = dv(A.div_lwp, pc), jc = pc - ph * A.lwp;
                int v = v0, jj = j, base = oh0;
                if (j >= nr0) { const int d = dv(A.div_rows, j - nr0); v = v0 + 1 + d; jj = j - nr0 - d * A.rows_full; base = 0; }
                const int k = dv(A.div_rstep, jj), n = dv(A.div_strips, v), strip = v - n * A.nstrips;
                const int ih = A.s * (base + k) + (jj - k * A.rstep) - q.Ph, iw = A.s * (strip * A.bw + jc) + ph - q.Pw;
                const bool in = n < A.N && (unsigned)ih < (unsigned)A.H && (unsigned)iw < (unsigned)A.W;
                const uint32_t off = in ? (uint32_t)((n - n0) * (int)image + ih * A.W + iw + A.bias) * 4u : 0x80000000u;
                const int c0 = (chunk * A.groups[0] + gg) * 8;
                for (int e = 0; e < 8; ++e) lds[((size_t)gg * A.P + px) * 8 + e] = load(off, (uint32_t)std::min(c0 + e, A.C - 1) * (uint32_t)(A.H * A.W) * 4u);
            }
            const int nst = last ? q.steps[1] : q.steps[0];
            CHECK(2 * nst <= kDirectMaxUnits);
            for (int l = 0; l < NPX; ++l) {
                const int pp = std::min(p0 + l, A.total_px - 1), gr = dv(A.div_bw, pp), ow = pp - gr * A.bw, v = dv(A.div_oh, gr), oh = gr - v * A.OH;
                const int j = v == v0 ? A.rstep * (oh - oh0) : nr0 + (v - v0 - 1) * A.rows_full + A.rstep * oh;
                const uint32_t lb = (uint32_t)(j * A.row_px + ow) * 48u;
                const int n = dv(A.div_strips, v), owf = (v - n * A.nstrips) * A.bw + ow;
                const bool in = p0 + l < A.total_px && oh < q.OH && owf < q.OW;
                if (in && chunk == 0 && full) outs[pi][((size_t)n * q.OH + oh) * q.OW + owf]++;
                const long long plane = (long long)A.YH * A.YW;
                CHECK(((n - n0) * (long long)A.K + 4) * plane + plane + 64 * plane < (1LL << 29));
                if (in) CHECK(A.sy * oh + q.oy < A.YH && A.sx * owf + q.ox < A.YW && q.oy >= 0 && q.ox >= 0);
                for (int st = 0; st < nst; ++st) for (int h = 0; h < 2; ++h) {
                    const int u = std::min(2 * st + h, G * q.R * q.S - 1), tap = u / G, r = tap / q.S, s = tap - r * q.S, sq = s / A.s;
                    const uint32_t at = lb + (uint32_t)(u - tap * G) * (uint32_t)A.P * 48u + (uint32_t)(r * A.row_px + (s - sq * A.s) * A.lwp + sq) * 48u;
                    CHECK(at % 48 == 0 && at / 48 < (uint32_t)A.groups[0] * A.P);
                    for (int e = 0; e < 8; ++e) {
                        const long long got = lds[(size_t)(at / 48) * 8 + e];
                        CHECK(got != -2);
                        const int c = (chunk * A.groups[0] + u - tap * G) * 8 + e;
                        if (2 * st + h != u || c >= A.C || !in) continue;
                        const int ih = A.s * oh - q.Ph + r, iw = A.s * owf - q.Pw + s;
                        const long long want = ih < 0 || iw < 0 || ih >= A.H || iw >= A.W ? -1 : (((long long)n * A.C + c) * A.H + ih) * A.W + iw;
                        CHECK(got == want);
                    }
                }
            }
        }
    }
    for (char v : tiles) CHECK(v == 1);
    for (auto& o : outs) for (char v : o) CHECK(v == 1);
}
static int cdiv(int x, int d) { return x >= 0 ? (x + d - 1) / d : -((-x) / d); }
int main(int argc, char** argv)
{
    const int iters = argc > 1 ? std::atoi(argv[1]) : 60;
    int n = 0, took = 0, cut = 0;
    const int fixed[][9] = {{5, 67, 35, 29, 93, 5, 5, 2, 2}, {4, 76, 8, 8, 18, 3, 3, 3, 0}, {1, 300, 2, 2, 40, 3, 3, 1, 1},
                            {70, 9, 1, 1, 17, 1, 1, 1, 0}, {2, 16, 60, 230, 20, 3, 5, 1, 2}};
    for (int it = 0; it < iters + 5; ++it) {
        int s[9];
        if (it < 5) std::copy(fixed[it], fixed[it] + 9, s);
        else {
            s[5] = pick(1, 11); s[6] = rnd() % 2 ? s[5] : pick(1, 11); s[7] = pick(1, 4); s[8] = pick(0, 5);
            s[0] = pick(1, 6); s[1] = rnd() % 2 ? pick(1, 15) : pick(16, 50); s[4] = pick(1, 300);
            s[2] = pick(1, rnd() % 4 ? 20 : 60); s[3] = pick(1, rnd() % 4 ? 20 : 150);
        }
        const int N = s[0], C = s[1], H = s[2], W = s[3], K = s[4], R = s[5], S = s[6], st = s[7], P = s[8];
        if (H + 2 * P < R || W + 2 * P < S) continue;
        const int OH = (H + 2 * P - R) / st + 1, OW = (W + 2 * P - S) / st + 1;
        for (int v = 0; v < kNumDirectShapes; ++v) {
            DirectArgs A;
            DirectProb q{}; q.R = R; q.S = S; q.Ph = q.Pw = P; q.OH = OH; q.OW = OW;
            ++n;
            if (direct_setup(N, C, H, W, K, st, OH, OW, 1, 1, &q, 1, v, &A)) {
                ++took; replay(A, it != 4);
                reads(A, FilterSource{0, (long long)C * R * S, R * S, S, 1}, {{0, 0, 1}}, (long long)C * R * S, R * S, R, S);
            }
            // a tile's chunks shared by several workgroups
            const int pieces = pick(2, rnd() % 4 ? 4 : kDirectMaxPieces);
            if (direct_setup(N, C, H, W, K, st, OH, OW, 1, 1, &q, 1, v, &A, pieces)) {
                ++cut; CHECK(A.pieces == pieces); replay(A, it != 4);
            }
            // data gradient: all phases
            std::vector<DirectProb> ps;
            std::vector<Taps> tp;
            for (int a = 0; a < st; ++a) for (int b = 0; b < st; ++b) {
                DirectProb q{};
                const int na = a < R ? (R - a + st - 1) / st : 0, nb = b < S ? (S - b + st - 1) / st : 0;
                const int u0 = cdiv(P - a, st), v0 = cdiv(P - b, st);
                const int u1 = H + P - 1 - a >= 0 ? (H + P - 1 - a) / st : -1, v1 = W + P - 1 - b >= 0 ? (W + P - 1 - b) / st : -1;
                q.R = na; q.S = nb; q.OH = u1 - u0 + 1; q.OW = v1 - v0 + 1; q.Ph = na - 1 - u0; q.Pw = nb - 1 - v0;
                q.oy = st * u0 + a - P; q.ox = st * v0 + b - P;
                q.base = (long long)(st * (na - 1) + a) * S + st * (nb - 1) + b;
                if (na > 0 && nb > 0 && q.OH > 0 && q.OW > 0) { ps.push_back(q); tp.push_back({st * (na - 1) + a, st * (nb - 1) + b, -st}); }
            }
            ++n;
            if (!ps.empty() && direct_setup(N, K, OH, OW, C, 1, H, W, st, st, ps.data(), (int)ps.size(), v, &A)) {
                ++took; replay(A, it != 4);
                FilterSource F{0, R * S, (long long)R * S * C, -st * S, -st};
                reads(A, F, tp, R * S, (long long)R * S * C, R, S);
                if (st == 1) {  // (a plan of its own: the base is the source's)
                    std::swap(F.base, A.p[0].base);
                    reads(A, F, tp, R * S, (long long)R * S * C, R, S);
                }
            }
        }
    }
    // the most pixels that a call may have: no launch of 2^32 threads or more
    const int large[][7] = {{107374182, 1, 5, 4, 6, 3, 2}, {238609294, 1, 3, 3, 4, 2, 2}, {429496729, 1, 1, 5, 5, 4, 2}};  // N, C, H, W, R, stride, pad; one filter
    for (const auto& l : large)
        for (int v = 0; v < kNumDirectShapes; ++v) {
            const int OH = (l[2] + 2 * l[6] - l[4]) / l[5] + 1, OW = (l[3] + 2 * l[6] - l[4]) / l[5] + 1;
            std::vector<DirectProb> ps;
            for (int a = 0; a < l[5]; ++a) for (int b = 0; b < l[5]; ++b) {
                DirectProb q{};
                const int u0 = cdiv(l[6] - a, l[5]), v0 = cdiv(l[6] - b, l[5]);
                q.R = (l[4] - a + l[5] - 1) / l[5]; q.S = (l[4] - b + l[5] - 1) / l[5];
                q.OH = (l[2] + l[6] - 1 - a) / l[5] - u0 + 1; q.OW = (l[3] + l[6] - 1 - b) / l[5] - v0 + 1;
                q.Ph = q.R - 1 - u0; q.Pw = q.S - 1 - v0;
                if (l[2] + l[6] - 1 >= a && l[3] + l[6] - 1 >= b && q.OH > 0 && q.OW > 0) ps.push_back(q);
            }
            DirectArgs A;
            CHECK(!ps.empty());
            if (direct_setup(l[0], 1, OH, OW, l[1], 1, l[2], l[3], l[5], l[5], ps.data(), (int)ps.size(), v, &A))
                CHECK((long long)A.ntiles * kDirectShapes[v].threads() < 1LL << 32);
        }
    CHECK(took * 2 > n && cut > 0);
    std::printf("direct fuzz: %d of %d (layer, shape) pairs planned and replayed, %d more in pieces\n", took, n, cut);
}
