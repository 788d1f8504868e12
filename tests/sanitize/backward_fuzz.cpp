// Host-only fuzz of the data gradient's planning (backward.hip's host code), built with -fsanitize=address,undefined by
// tests/test_sanitize.py: sub-convolutions contracted in one launch, their tiles cut into pieces, one input transform and one
// filter transform for all of them.  What the kernels read from these tables is replayed against the definition of the
// gradient and the sizes of the buffers.  Nothing here touches a GPU.
#include <cstdio>
#include <cstdlib>

#include "../../paper_2002_00552_amd/csrc/backward.hip"

namespace dwm {
dwm_status_t launch_filter_transform(const dwm_plan&, const float*, float*, void*) { return DWM_OK; }
dwm_status_t launch_filter_transform_from(const dwm_plan&, const FilterSource&, const float*, float*, void*) { return DWM_OK; }
dwm_status_t launch_filter_batch(const FilterBatchArgs&, const float*, float*, void*) { return DWM_OK; }
dwm_status_t launch_input_transform(const dwm_plan&, const float*, float*, void*) { return DWM_OK; }
dwm_status_t launch_contract_output(const dwm_plan&, const float*, float*, float*, void*) { return DWM_OK; }
dwm_status_t launch_contract_batch(const BatchArgs&, const PlaneTable&, int, const float*, const float*, float*, float*, void*) { return DWM_OK; }
dwm_status_t launch_fused_forward(const dwm_plan&, const float*, const float*, float*, void*) { return DWM_OK; }
dwm_status_t launch_direct(const dwm_plan&, const float*, const float*, float*, float*, void*) { return DWM_OK; }
dwm_status_t launch_bwd_small_filter(const BwdSmallArgs&, int, int, const float*, float*, void*) { return DWM_OK; }
dwm_status_t launch_bwd_small(const BwdSmallArgs&, const float*, const float*, float*, void*) { return DWM_OK; }
}  // namespace dwm

static uint64_t g_state = 0x9E3779B97F4A7C15ull;
static uint32_t rnd()
{
    g_state ^= g_state << 13;
    g_state ^= g_state >> 7;
    g_state ^= g_state << 17;
    return (uint32_t)(g_state >> 32);
}
static int pick(int lo, int hi) { return lo + (int)(rnd() % (uint32_t)(hi - lo + 1)); }

#define CHECK(c)                                                              \
    do {                                                                      \
        if (!(c)) {                                                           \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #c); \
            std::exit(2);                                                     \
        }                                                                     \
    } while (0)

// counts: layers contracted in one launch, with one input transform, of these with unequal tile grids, cut into pieces, with
// one filter transform
static int n_batched, n_merged, n_unequal, n_pieces, n_filter;

static void walk(int N, int C, int H, int W, int K, int R, int S, int s, int P)
{
    using namespace dwm;
    dwm_bwd_data_plan_t* bp = nullptr;
    if (dwm_bwd_data_plan_create(&bp, N, C, H, W, K, R, S, s, P) != DWM_OK) {
        CHECK(bp == nullptr);
        return;
    }
    if (!bp->batched) {
        CHECK(!bp->merged && !bp->filter_batched);
        dwm_bwd_data_plan_destroy(bp);
        return;
    }
    ++n_batched;
    const BatchArgs& A = bp->batch;
    CHECK(A.nprob >= 2 && A.nprob <= kMaxBatch && bp->batch_planes.n <= kMaxPlanes);
    const size_t partials = A.ipw > 0 ? (size_t)A.nblocks * 65536 : 0;
    CHECK(A.ipw == 0 || (bp->partial_off % 256 == 0 && bp->partial_off + partials <= bp->ws_bytes));
    const size_t v_end = A.ipw > 0 ? bp->partial_off : bp->ws_bytes;  // bytes that V may take
    int tiles = 0, blocks = 0, merged_class = 0, max_rows = 0;
    bool unequal = false;
    // the sub-convolutions in the launch's order: by their output maps
    for (int q = 0; q < A.nprob; ++q) {
        const BatchProb& Q = A.p[q];
        const dwm_bwd_data_plan::Phase* ph = nullptr;
        for (const auto& f : bp->phases)
            if (f.sub && f.oy == Q.om.oy && f.ox == Q.om.ox) ph = &f;
        CHECK(ph && Q.om.YH == H && Q.om.YW == W && Q.om.sy == s && Q.om.sx == s);
        const dwm_plan_t& sub = *ph->sub;
        const DevPlan& sd = sub.d;
        // tiles and workgroups, end to end; the pieces cover a tile's chunks, none empty
        CHECK(Q.tile0 == tiles && Q.block0 == blocks);
        const int ntt = (Q.T + 63) / 64;
        tiles += A.nkt * ntt;
        blocks += A.nkt * ntt * Q.pieces;
        CHECK(A.ipw > 0 ? Q.pieces >= 1 && Q.pieces * A.ipw >= Q.n_iter && (Q.pieces - 1) * A.ipw < Q.n_iter : Q.pieces == 1);
        // the tile grid reaches every pixel of the phase
        CHECK(2 * Q.TH >= Q.OH && 2 * Q.TW >= Q.OW && Q.OH == ph->UH && Q.OW == ph->UW && Q.T == N * Q.TH * Q.TW);
        unequal |= Q.TH != sd.TH || Q.TW != sd.TW;
        // planes: where their chunks lie in U and V
        int chunks = 0;
        for (int e = 0; e < sub.planes.n; ++e) {
            const DevPlaneEntry& b = bp->batch_planes.e[Q.plane0 + e];
            CHECK(b.Lpad == sub.planes.e[e].Lpad && b.coef == sub.planes.e[e].coef && b.Lpad % bp->batch_lc == 0);
            CHECK((size_t)b.u_off64 * 64 == (size_t)sub.planes.e[e].u_off64 * 64 + ph->u_off);
            CHECK((size_t)b.u_off64 * 64 + (size_t)A.nkt * 64 * b.Lpad <= bp->filter_floats);
            CHECK(((size_t)b.v_off64 + b.Lpad) * 64 <= (size_t)Q.vblock);
            chunks += b.Lpad / bp->batch_lc;
        }
        CHECK(chunks == Q.n_iter);
        CHECK(((size_t)Q.v_base + (size_t)ntt * Q.vblock) * 4 <= v_end);
        // one input transform: its classes are the sub-convolutions', in the launch's order; a part's rows and columns of dy
        // are those of the sub-convolution; its planes lie where the launch's table says
        if (bp->merged) {
            const DevPlan& d = bp->merged->d;
            CHECK(Q.v_base == 0 && Q.vblock == d.vblock_rows * 64 && Q.TH == d.TH && Q.TW == d.TW && Q.T == d.T);
            CHECK(d.nh <= kMaxPieces && d.nw <= kMaxPieces && d.ncls <= kMaxClasses && d.Tpad % 64 == 0 && d.Tpad >= d.T);
            CHECK((size_t)d.vblock_rows * d.Tpad * 4 <= v_end && d.C == K && d.H == bp->OH && d.W == bp->OW && d.s == 1);
            for (int c = 0; c < sd.ncls; ++c, ++merged_class) {
                const DevClass &a = sd.cls[c], &m = d.cls[merged_class];
                CHECK(m.lh == a.lh && m.lw == a.lw && m.hn == a.hn && m.wn == a.wn && m.L == a.L && m.Lpad == a.Lpad);
                CHECK(m.h0 + m.hn <= d.nh && m.w0 + m.wn <= d.nw);
                for (int i = 0; i < a.hn; ++i)
                    CHECK(d.ph[m.h0 + i].j - d.Ph == sd.ph[a.h0 + i].j - sd.Ph && d.ph[m.h0 + i].l == a.lh && d.ph[m.h0 + i].p == 0);
                for (int i = 0; i < a.wn; ++i)
                    CHECK(d.pw[m.w0 + i].j - d.Pw == sd.pw[a.w0 + i].j - sd.Pw && d.pw[m.w0 + i].l == a.lw && d.pw[m.w0 + i].p == 0);
                for (int pl = 0; pl < (a.lh + 1) * (a.lw + 1); ++pl)
                    CHECK(bp->batch_planes.e[Q.plane0 + a.plane0 + pl].v_off64 == (uint32_t)(m.v_row0 + pl * m.Lpad));
            }
        }
        // one filter transform: tap (i, j) of a part is the gradient's tap of w
        if (bp->filter_batched) {
            const FilterBatchArgs& F = bp->filter_batch;
            CHECK(F.nprob == A.nprob && F.K == C && F.C == K && F.Kpad == sd.Kpad);
            const FilterBatchProb& B = F.p[q];
            CHECK(B.ncls == sd.ncls && B.rows_total == sd.rows_total);
            max_rows = B.rows_total > max_rows ? B.rows_total : max_rows;
            for (int c = 0; c < sd.ncls; ++c) {
                const DevClass& a = sd.cls[c];
                const FilterBatchClass& b = B.cls[c];
                CHECK(b.lh == a.lh && b.lw == a.lw && b.wn == a.wn && b.L == a.L && b.Lpad == a.Lpad && b.row0 == a.row0);
                CHECK(b.L == a.hn * a.wn * K && b.u_off == a.u_off + (long long)ph->u_off);
                CHECK((size_t)b.u_off + (size_t)(a.lh + 1) * (a.lw + 1) * F.Kpad * a.Lpad <= bp->filter_floats);
                for (int x = 0; x < a.hn; ++x)
                    for (int y = 0; y < a.wn; ++y)
                        for (int i = 0; i < a.lh; ++i)
                            for (int j = 0; j < a.lw; ++j) {
                                const int k = pick(0, K - 1), ch = pick(0, C - 1);
                                // taps of the phase, flipped: row ti of the sub-convolution's filter
                                const int ti = sd.ph[a.h0 + x].j + i, tj = sd.pw[a.w0 + y].j + j;
                                if (i >= sd.ph[a.h0 + x].lr || j >= sd.pw[a.w0 + y].lr) continue;
                                CHECK(ti >= 0 && ti < ph->na && tj >= 0 && tj < ph->nb);
                                const long long want = (((long long)k * C + ch) * R + s * (ph->na - 1 - ti) + ph->a) * S + s * (ph->nb - 1 - tj) + ph->b;
                                const long long got = B.base + ch * F.sk + k * F.sc + (long long)(B.jh[b.h0 + x] + i) * F.sr + (long long)(B.jw[b.w0 + y] + j) * F.ss;
                                CHECK(got == want && got >= 0 && got < (long long)K * C * R * S);
                            }
            }
            CHECK(max_rows <= F.max_rows);
        }
    }
    CHECK(tiles == A.ntiles && blocks == A.nblocks);
    CHECK(!bp->merged || merged_class == bp->merged->d.ncls);
    n_merged += bp->merged != nullptr;
    n_unequal += bp->merged && unequal;
    n_pieces += A.ipw > 0;
    n_filter += bp->filter_batched;
    dwm_bwd_data_plan_destroy(bp);
}

int main(int argc, char** argv)
{
    const int iters = argc > 1 ? std::atoi(argv[1]) : 2000;
    // the layers of tests/test_gpu_backward_pieces.py
    const int fixed[][9] = {
        {5, 67, 35, 29, 93, 5, 5, 2, 2}, {1, 17, 9, 8, 200, 3, 3, 2, 1}, {2, 20, 21, 21, 40, 7, 7, 2, 3},
        {2, 33, 20, 20, 64, 4, 4, 3, 1}, {1, 18, 23, 19, 70, 5, 5, 4, 2}, {1, 65, 31, 30, 130, 6, 3, 2, 0},
        {32, 128, 56, 56, 256, 3, 3, 2, 1},
    };
    for (const auto& f : fixed) walk(f[0], f[1], f[2], f[3], f[4], f[5], f[6], f[7], f[8]);
    for (int i = 0; i < iters; ++i) {
        const int R = pick(1, 13), S = rnd() % 4 ? R : pick(1, 13), s = pick(2, 4), P = rnd() % 2 ? R / 2 : pick(0, R);
        walk(pick(1, 9), pick(1, 200), pick(1, 70), pick(1, 70), pick(1, 300), R, S, s, P);
    }
    CHECK(n_batched > iters / 4 && n_merged > iters / 8 && n_unequal > iters / 30 && n_pieces > iters / 20 && n_filter > iters / 8);
    std::printf("backward fuzz: %d layers in one launch, %d with one input transform (%d over unequal grids), %d in pieces, %d with one "
                "filter transform\n", n_batched, n_merged, n_unequal, n_pieces, n_filter);
    return 0;
}
