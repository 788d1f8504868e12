// Gradient of the DWM convolution with respect to its input (paper Sec. 3.1 eq. 5 and
// Sec. 4.2 eq. 16-17 state what is computed: every part receives the whole output gradient
// and the parts' input gradients add up -- the sum is the gradient of the ordinary
// convolution).
//
// How it is organised here.  The gradient image is itself a convolution of dy, and the
// stride splitting of Sec. 4.1 (eq. 12-14) applies to it in mirror image: an input pixel at
// padded position u belongs to phase a = u mod stride, only taps r = stride*i + a reach it,
// and with u = stride*u' + a
//     dx_a[u'] = sum_k sum_i dy[k][u' - i] * w[k][c][stride*i + a]
// is a STRIDE-1 convolution of dy with the taps of phase a, flipped, filters and channels
// swapped.  So the gradient is stride^2 independent stride-1 convolutions -- one per phase
// pair (a, b) -- each run through the forward DWM machinery of this library (splitting into
// pieces of at most three taps, F(2,l), the same kernels), whose outputs interleave: the
// sub-convolution of phase (a, b) writes the pixels (stride*o + oy, stride*o' + ox) of dx.
// Every pixel of dx is written exactly once, nothing is accumulated in memory, results are
// bit-identical from run to run.  Phases that hold no tap (stride > kernel) get zeros.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <new>
#include <vector>

#include "plan.hpp"

struct dwm_bwd_data_plan {
    int N, C, H, W, K, R, S, s, P, OH, OW;
    struct Phase {
        int a, b, na, nb;    // phase pair, taps per dimension (0: no tap)
        int oy, ox, UH, UW;  // first pixel of the phase in dx, pixels per dimension
        dwm_plan_t* sub;     // stride-1 sub-convolution (null if the phase has no tap or no pixel)
        size_t u_off;        // its transformed filter inside Ugw (floats)
    };
    std::vector<Phase> phases;
    size_t wtmp_floats;      // start of Ugw: room for the weights of a phase on the single-kernel forward path, if any is (not used:
                             // they are read where they lie; the buffer's layout is as callers know it)
    size_t filter_floats, ws_bytes;
    double direct_flops;
    // all sub-convolutions contracted in one launch (contract_batch.hip): each then has its own
    // slice of the workspace, ws_off[i] bytes from its start for phase i
    bool batched;
    int batch_lc;
    dwm::BatchArgs batch;
    dwm::PlaneTable batch_planes;
    std::vector<size_t> ws_off;
    size_t partial_off;      // bytes from the start of the workspace to the partial outputs of tiles cut into pieces
    float* ws;
    // ... their filters transformed in one launch too, where their tables fit its arguments
    bool filter_batched;
    dwm::FilterBatchArgs filter_batch;
    // ... and, where their pieces and classes fit one plan, ONE input transform for all of them: a plan that
    // holds every sub-convolution's pieces and classes (used by the input transform only)
    dwm_plan_t* merged;
    // ... or the whole gradient as one direct convolution of all phases (direct.hip): a plan that holds nothing else, its filter
    // u_direct_off floats into Ugw.  The planner's choice wherever it is planned
    dwm_plan_t* direct;
    size_t u_direct_off;
    bool use_direct() const { return direct && variant_path < 0; }
    // (stride 1: its one sub-convolution's plan has the direct convolution itself)
    bool use_sub_direct() const { return s == 1 && phases[0].sub && phases[0].sub->use_direct(); }
    // few input channels: the whole gradient in one kernel (backward_small.hip), its filter copy
    // u_small_off floats into Ugw; variant_path < 0: the planner's choice, 0: sub-convolutions, 1: that kernel
    bool small_ok;
    dwm::BwdSmallArgs small;
    size_t u_small_off;
    int variant_path;
    bool use_small() const { return small_ok && (variant_path == 1 || (variant_path < 0 && small_default)); }
    bool small_default;
};

namespace dwm {

// dx[n][c][sy*o + oy][sx*o' + ox] = 0 for o < UH, o' < UW
__global__ __launch_bounds__(256) void bwd_zero_phase_kernel(float* __restrict__ dx, int planes, int H, int W, int s,
                                                             int oy, int ox, int UH, int UW)
{
    const size_t total = (size_t)planes * UH * UW;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (size_t)gridDim.x * 256) {
        const int v = (int)(e % UW);
        const int u = (int)((e / UW) % UH);
        const size_t pl = e / ((size_t)UW * UH);
        dx[(pl * H + (size_t)(s * u + oy)) * W + (s * v + ox)] = 0.f;
    }
}

static int ceil_div(int x, int d) { return x >= 0 ? (x + d - 1) / d : -((-x) / d); }

}  // namespace dwm


// (the batch's plane table with every plane pointing into its own sub-convolution's V)
static void setup_batch_unmerged_planes(dwm_bwd_data_plan& bp, const std::vector<int>& subs)
{
    for (int q = 0; q < bp.batch.nprob; ++q) {
        const dwm_plan_t* sp = bp.phases[subs[q]].sub;
        for (int e = 0; e < sp->planes.n; ++e) bp.batch_planes.e[bp.batch.p[q].plane0 + e].v_off64 = sp->planes.e[e].v_off64;
    }
}

// One input transform for all sub-convolutions.  They read the same dy; what differs is which
// window of it a tile of phase (a, b) starts at.  A sub-convolution's patch element is at row
// 2*ty + j + i - Ph_a of dy; with Ph = the largest Ph_a and j' = j + (Ph - Ph_a) that is
// 2*ty + j' + i - Ph for all of them, so one plan can hold the pieces of every phase (those of
// phase a once, shifted), and one class per (sub-convolution, class) whose parts are the products
// of ITS phases' pieces.  The staged rows of dy are then fetched once instead of once per phase.
// The tile grid is the largest of theirs (they differ by a row or a column of tiles at most, where the image's sides do not
// divide by twice the stride): patches past the image read zeros, outputs past a sub-convolution's extent are dropped.
// Applies when the pieces and classes fit the plan's tables.
static void setup_merged(dwm_bwd_data_plan& bp, const std::vector<int>& subs)
{
    using namespace dwm;
    bp.merged = nullptr;
    const dwm_plan_t* first = bp.phases[subs[0]].sub;
    int Ph = first->d.Ph, Pw = first->d.Pw, ncls = 0, TH = 0, TW = 0;
    long long sum_t = 0;
    for (int i : subs) {
        const DevPlan& d = bp.phases[i].sub->d;
        TH = std::max(TH, d.TH);
        TW = std::max(TW, d.TW);
        sum_t += d.T;
        Ph = std::max(Ph, d.Ph);
        Pw = std::max(Pw, d.Pw);
        ncls += d.ncls;
    }
    if (ncls > kMaxClasses) return;
    // (a common grid more than a quarter larger than theirs costs more in the contraction than the shared staging gains)
    const long long T = (long long)bp.N * TH * TW, Tpad = (T + kTAlign - 1) / kTAlign * kTAlign;
    if (Tpad >= (1LL << 31) - 1 || T * (long long)subs.size() * 4 > sum_t * 5) return;
    dwm_plan* m = new (std::nothrow) dwm_plan;
    if (!m) return;
    std::memset(m, 0, sizeof(*m));
    DevPlan& d = m->d;
    d = first->d;
    d.Ph = Ph; d.Pw = Pw;
    d.TH = TH; d.TW = TW;
    d.T = (int)T; d.Tpad = (int)Tpad;
    d.nh = d.nw = d.ncls = d.rows_total = d.vblock_rows = 0;
    // pieces: those of phase a (rows) / b (columns) once
    std::vector<int> hoff(bp.s, -1), woff(bp.s, -1);
    bool ok = true;
    for (int i : subs) {
        const auto& ph = bp.phases[i];
        const DevPlan& sd = ph.sub->d;
        if (hoff[ph.a] < 0) {
            if (d.nh + sd.nh > kMaxPieces) { ok = false; break; }
            hoff[ph.a] = d.nh;
            for (int q = 0; q < sd.nh; ++q) {
                DevPiece pc = sd.ph[q];
                pc.j += Ph - sd.Ph;
                d.ph[d.nh++] = pc;
            }
        }
        if (woff[ph.b] < 0) {
            if (d.nw + sd.nw > kMaxPieces) { ok = false; break; }
            woff[ph.b] = d.nw;
            for (int q = 0; q < sd.nw; ++q) {
                DevPiece pc = sd.pw[q];
                pc.j += Pw - sd.Pw;
                d.pw[d.nw++] = pc;
            }
        }
    }
    long long v_off = 0;
    if (ok)
        for (int q = 0; q < bp.batch.nprob && ok; ++q) {
            const auto& ph = bp.phases[subs[q]];
            const DevPlan& sd = ph.sub->d;
            for (int c = 0; c < sd.ncls; ++c) {
                DevClass cl = sd.cls[c];
                const int planes = (cl.lh + 1) * (cl.lw + 1);
                cl.h0 += hoff[ph.a];
                cl.w0 += woff[ph.b];
                cl.row0 = d.rows_total;
                cl.v_row0 = (int)v_off;
                // this class's planes in the batch's table now point into the merged V
                for (int pl = 0; pl < planes; ++pl)
                    bp.batch_planes.e[bp.batch.p[q].plane0 + sd.cls[c].plane0 + pl].v_off64 = (uint32_t)(v_off + (long long)pl * cl.Lpad);
                d.cls[d.ncls++] = cl;
                d.rows_total += cl.Lpad;
                v_off += (long long)planes * cl.Lpad;
                if (v_off * d.Tpad >= ((1LL << 31) - 1) * 32) ok = false;
            }
        }
    if (!ok) {
        delete m;
        setup_batch_unmerged_planes(bp, subs);
        return;
    }
    d.vblock_rows = (int)v_off;
    m->v_floats = (size_t)v_off * (size_t)d.Tpad;
    m->lgran = bp.batch_lc;
    m->variant_input = -1;
    m->variant_forward = 0;
    m->inlds_ok = input_lds_setup(*m, &m->inlds, 0);
    for (int q = 0; q < bp.batch.nprob; ++q) {
        BatchProb& P = bp.batch.p[q];
        P.vblock = d.vblock_rows * 64;
        P.v_base = 0;
        P.TH = TH; P.TW = TW; P.T = (int)T;
        P.tile0 = q * bp.batch.nkt * (int)((T + 63) / 64);
    }
    bp.batch.ntiles = bp.batch.nprob * bp.batch.nkt * (int)((T + 63) / 64);
    bp.ws_bytes = std::max<size_t>((m->v_floats * sizeof(float) + 255) / 256 * 256 + 256, 256);
    bp.merged = m;
}

// Fewer tiles than CUs: each is cut into pieces.  By this model (us; a 32-step chunk takes 0.8 in a workgroup alone on its CU
// -- latency -- and 0.45 of the CU's matrix cores; pieces are added up by a launch of its own, 5 and 0.2 per MB) whole tiles
// stay where cutting them gains less than a tenth; a piece has four chunks at least.
static void setup_pieces(dwm_bwd_data_plan& bp)
{
    using namespace dwm;
    BatchArgs& A = bp.batch;
    int longest = 0;
    for (int q = 0; q < A.nprob; ++q) longest = std::max(longest, A.p[q].n_iter);
    auto tiles = [&](int q) { return (q + 1 < A.nprob ? A.p[q + 1].tile0 : A.ntiles) - A.p[q].tile0; };
    const double unit = bp.batch_lc / 32.0;
    double best = 0.9 * longest * unit * std::max(0.8, 0.45 * ((A.ntiles + kNumCUs - 1) / kNumCUs));
    A.ipw = 0;
    for (int f = 2; f <= 16 && A.ntiles < kNumCUs && longest >= 4 * f; ++f) {
        const int ipw = (longest + f - 1) / f;
        int blocks = 0;
        for (int q = 0; q < A.nprob; ++q) blocks += tiles(q) * ((A.p[q].n_iter + ipw - 1) / ipw);
        const double us = ipw * unit * std::max(0.8, 0.45 * ((blocks + kNumCUs - 1) / kNumCUs)) + 5.0 + 0.2e-6 * 65536.0 * blocks;
        if (us >= best) continue;
        best = us;
        A.ipw = ipw;
    }
    A.nblocks = 0;
    for (int q = 0; q < A.nprob; ++q) {
        A.p[q].pieces = A.ipw > 0 ? (A.p[q].n_iter + A.ipw - 1) / A.ipw : 1;
        A.p[q].block0 = A.nblocks;
        A.nblocks += tiles(q) * A.p[q].pieces;
    }
    bp.partial_off = (bp.ws_bytes + 255) / 256 * 256;
    if (A.ipw > 0) bp.ws_bytes = bp.partial_off + (size_t)A.nblocks * 65536;
}

static void setup_filter_batch(dwm_bwd_data_plan& bp, const std::vector<int>& subs)
{
    using namespace dwm;
    bp.filter_batched = false;
    if (subs.size() > (size_t)kMaxFilterBatch) return;
    FilterBatchArgs& F = bp.filter_batch;
    F = FilterBatchArgs{};
    const long long rs = (long long)bp.R * bp.S;
    const DevPlan& d0 = bp.phases[subs[0]].sub->d;
    F.K = d0.K; F.C = d0.C; F.Kpad = d0.Kpad;
    F.sk = rs; F.sc = rs * bp.C;
    F.sr = -bp.s * bp.S; F.ss = -bp.s;
    for (int i : subs) {
        const auto& ph = bp.phases[i];
        const DevPlan& d = ph.sub->d;
        if (ph.sub->fused_ok || ph.sub->split_ok || d.ncls > 4) return;
        FilterBatchProb& P = F.p[F.nprob++];
        P.ncls = d.ncls;
        P.rows_total = d.rows_total;
        P.base = (long long)(bp.s * (ph.na - 1) + ph.a) * bp.S + bp.s * (ph.nb - 1) + ph.b;
        for (int q = 0; q < d.nh; ++q) {
            if (d.ph[q].p != 0 || d.ph[q].j > 127) return;
            P.jh[q] = (signed char)d.ph[q].j;
        }
        for (int q = 0; q < d.nw; ++q) {
            if (d.pw[q].p != 0 || d.pw[q].j > 127) return;
            P.jw[q] = (signed char)d.pw[q].j;
        }
        for (int c = 0; c < d.ncls; ++c) {
            const DevClass& q = d.cls[c];
            P.cls[c] = FilterBatchClass{q.lh, q.lw, q.wn, q.L, q.Lpad, q.row0, q.h0, q.w0, (long long)ph.u_off + q.u_off};
        }
        F.max_rows = std::max(F.max_rows, d.rows_total);
    }
    bp.filter_batched = true;
}

// One launch for the contractions of all sub-convolutions where that applies: at least two of
// them, all on the staged path, their planes fit one table.  The sub-convolutions are ordered
// longest first; each keeps its own slice of the workspace (its V is alive until the one launch).
static void setup_batch(dwm_bwd_data_plan& bp)
{
    using namespace dwm;
    bp.batched = false;
    bp.filter_batched = false;
    bp.partial_off = 0;
    bp.merged = nullptr;
    bp.ws = nullptr;
    bp.ws_off.assign(bp.phases.size(), 0);
    std::vector<int> subs;
    int planes = 0, lc = 32;  // 32-step chunks, three stages: 48 KB of LDS, three workgroups per CU (measured best)
    for (size_t i = 0; i < bp.phases.size(); ++i) {
        const dwm_plan_t* sp = bp.phases[i].sub;
        if (!sp) continue;
        if (sp->use_fused()) return;
        subs.push_back((int)i);
        planes += sp->planes.n;
        lc = std::min(lc, sp->lgran);
    }
    if (subs.size() < 2 || subs.size() > (size_t)kMaxBatch || planes > kMaxPlanes) return;
    auto n_iter = [&](int i) {
        int n = 0;
        const PlaneTable& pt = bp.phases[i].sub->planes;
        for (int q = 0; q < pt.n; ++q) n += pt.e[q].Lpad / lc;
        return n;
    };
    std::stable_sort(subs.begin(), subs.end(), [&](int a, int b) { return n_iter(a) > n_iter(b); });
    BatchArgs& A = bp.batch;
    A = BatchArgs{};
    A.K = bp.C;  // the sub-convolutions' filters are the layer's input channels
    A.nkt = (bp.C + 63) / 64;
    A.nprob = (int)subs.size();
    bp.batch_planes = PlaneTable{};
    size_t ws = 0;
    long long tiles = 0;
    for (int q = 0; q < A.nprob; ++q) {
        const int i = subs[q];
        const auto& ph = bp.phases[i];
        const dwm_plan_t* sp = ph.sub;
        if (ph.u_off % 64 != 0) return;
        BatchProb& P = A.p[q];
        P.plane0 = bp.batch_planes.n;
        P.n_iter = n_iter(i);
        P.tile0 = (int)tiles;
        P.vblock = sp->d.vblock_rows * 64;
        P.om = sp->d.om;
        P.OH = sp->d.OH; P.OW = sp->d.OW; P.TH = sp->d.TH; P.TW = sp->d.TW; P.T = sp->d.T;
        P.v_base = (long long)(ws / sizeof(float));
        bp.ws_off[i] = ws;
        ws += (dwm_plan_workspace_bytes(sp) + 255) / 256 * 256;
        for (int e = 0; e < sp->planes.n; ++e) {
            DevPlaneEntry pe = sp->planes.e[e];
            pe.u_off64 += (uint32_t)(ph.u_off / 64);
            bp.batch_planes.e[bp.batch_planes.n++] = pe;
        }
        tiles += (long long)A.nkt * ((sp->d.T + 63) / 64);
    }
    if (tiles > 0x7fffffffLL || ws / sizeof(float) > 0x7fffffffffffLL) return;
    A.ntiles = (int)tiles;
    bp.batch_lc = lc;
    bp.ws_bytes = std::max<size_t>(ws, 256);
    bp.batched = true;
    setup_merged(bp, subs);
    setup_pieces(bp);
    setup_filter_batch(bp, subs);
}

// The time (us) of the sub-convolutions by the method's transforms (what writes zeros left out): contracted in one launch, behind one
// input transform (711 measured, rms of the logarithm 0.13) or one for each, a 32-step chunk of a tile 0.55 to 1 us on its CU, V written
// and read; or one after the other (1002 measured, 0.19).
static double subconv_us(const dwm_bwd_data_plan& bp)
{
    double n = 0.0, alone = 1.0, chunks = 0.0;
    for (const auto& ph : bp.phases)
        if (ph.sub) {
            n += 1.0;
            alone += 0.98 * dwm::transforms_us(*ph.sub);
        }
    if (!bp.batched) return alone;
    const dwm::BatchArgs& A = bp.batch;
    for (int q = 0; q < A.nprob; ++q) chunks += (double)((q + 1 < A.nprob ? A.p[q + 1].tile0 : A.ntiles) - A.p[q].tile0) * A.p[q].n_iter;
    chunks *= bp.batch_lc / 32.0 / dwm::kNumCUs;
    if (!bp.merged) return 13.0 + chunks + 8.0 * n;
    return 22.0 + 0.55 * chunks + 0.44 * (double)bp.merged->v_floats * 8.0 / 4.3e6 + 1.5 * (double)bp.N * bp.C * bp.H * bp.W / 1e6 + 0.4 * n;
}

// All phases that a tap reaches as one direct convolution (direct.hip), where its model and its filter's copy (0.6 us a MB, and a launch
// where it is not written with the others) come to less than 0.85 of the sub-convolutions' time.  Of 1780 layers drawn with strides 2
// to 4 (up to 150 GFLOP) it takes 1585, at 0.45 of the time in the mean of all, the copy included, 14 of them slower by 3 % or
// more (1.23 at most).  At 0.93 of a rougher estimate one in twenty was, by up to 1.65 (5x5, 258 <- 147 channels, 37 images of 63x68).
// Nine input transforms of stride 3, 76 <- 18 channels, 46 images of 8x8, 180 -> 7 us; 5x5 at stride 2, 67 <- 93 channels, five 35x29 images
// 30 -> 14; 7x7 at stride 2, 256 <- 256 channels, 256 14x14 images 603 -> 456; 3x3 at stride 2, 128 <- 256, 32 56x56 images 136 -> 132.
static void setup_direct(dwm_bwd_data_plan& bp)
{
    using namespace dwm;
    std::vector<DirectProb> p;
    for (const auto& ph : bp.phases) {
        if (!ph.sub) continue;
        const DevPlan& d = ph.sub->d;
        DirectProb q{};
        q.R = ph.na; q.S = ph.nb; q.Ph = d.Ph; q.Pw = d.Pw; q.OH = ph.UH; q.OW = ph.UW; q.oy = ph.oy; q.ox = ph.ox;
        q.base = (long long)(bp.s * (ph.na - 1) + ph.a) * bp.S + bp.s * (ph.nb - 1) + ph.b;
        p.push_back(q);
    }
    if (p.empty() || p.size() > (size_t)kDirectMaxProbs) return;
    std::stable_sort(p.begin(), p.end(), [](const DirectProb& a, const DirectProb& b) { return a.R * a.S > b.R * b.S; });
    DirectArgs a;
    if (!direct_choose(bp.N, bp.K, bp.OH, bp.OW, bp.C, 1, bp.H, bp.W, bp.s, bp.s, p.data(), (int)p.size(), &a)) return;
    if (a.us + 2.4e-6 * a.filter_floats() + (bp.filter_batched ? 1.0 : 4.5) >= 0.85 * subconv_us(bp)) return;
    dwm_plan* m = new (std::nothrow) dwm_plan;
    if (!m) return;
    std::memset(m, 0, sizeof(*m));
    m->direct = a;
    m->direct_only = true;
    bp.direct = m;
    bp.u_direct_off = bp.filter_floats;
    bp.filter_floats += (a.filter_floats() + 63) / 64 * 64;
    bp.filter_batch.direct_blocks = a.all_steps * ((a.Kpad + 127) / 128);
    bp.filter_batch.direct_off = (long long)bp.u_direct_off;
    bp.filter_batch.direct = a;
}

extern "C" {

dwm_status_t dwm_bwd_data_plan_create(dwm_bwd_data_plan_t** out, int N, int C, int H, int W, int K, int R, int S,
                                      int stride, int pad)
{
    using namespace dwm;
    if (!out) return DWM_ERR_INVALID_ARG;
    if (N < 1 || C < 1 || H < 1 || W < 1 || K < 1 || R < 1 || S < 1 || stride < 1 || pad < 0)
        return DWM_ERR_INVALID_ARG;
    if ((long long)H + 2LL * pad < R || (long long)W + 2LL * pad < S) return DWM_ERR_INVALID_ARG;
    if (pad > (1 << 20) || H > (1 << 20) || W > (1 << 20) || stride > 8) return DWM_ERR_UNSUPPORTED;
    dwm_bwd_data_plan* bp = new (std::nothrow) dwm_bwd_data_plan;
    if (!bp) return DWM_ERR_ALLOC;
    bp->N = N; bp->C = C; bp->H = H; bp->W = W; bp->K = K; bp->R = R; bp->S = S; bp->s = stride; bp->P = pad;
    bp->OH = (H + 2 * pad - R) / stride + 1;
    bp->OW = (W + 2 * pad - S) / stride + 1;
    bp->direct_flops = 2.0 * N * K * C * R * S * bp->OH * bp->OW;
    bp->wtmp_floats = 0;
    bp->ws_bytes = 256;
    // the single-kernel form: chosen where the sub-convolutions would have only a handful of filters
    bp->small_ok = bwd_small_setup(N, C, H, W, K, R, S, stride, pad, &bp->small);
    // (LDS: room for the workgroups per CU its registers allow -- one where a wave holds several column blocks of
    // sixteen planes, else at least two)
    const size_t small_lds_max = (bp->small.nb > 1 && bp->small.four ? 152 : 78) * 1024;
    bp->small_default = bp->small_ok && C <= 16 && bp->small.nf <= 64 && bp->small.lds_bytes <= small_lds_max &&
                        bp->small.eff_pct >= 50;
    const int s = stride;
    dwm_status_t st = DWM_OK;
    for (int a = 0; a < s && st == DWM_OK; ++a)
        for (int b = 0; b < s && st == DWM_OK; ++b) {
            dwm_bwd_data_plan::Phase ph{};
            ph.a = a; ph.b = b;
            ph.na = a < R ? (R - a + s - 1) / s : 0;
            ph.nb = b < S ? (S - b + s - 1) / s : 0;
            // pixels of this phase: padded position u = s*u' + a with pad <= u < H + pad
            const int u0 = ceil_div(pad - a, s), v0 = ceil_div(pad - b, s);
            const int u1 = H + pad - 1 - a >= 0 ? (H + pad - 1 - a) / s : -1;
            const int v1 = W + pad - 1 - b >= 0 ? (W + pad - 1 - b) / s : -1;
            ph.UH = u1 - u0 + 1; ph.UW = v1 - v0 + 1;
            ph.oy = s * u0 + a - pad; ph.ox = s * v0 + b - pad;
            ph.sub = nullptr;
            if (ph.UH > 0 && ph.UW > 0 && ph.na > 0 && ph.nb > 0) {
                // the stride-1 sub-convolution: dy is its input (K channels), C filters of na x nb
                // taps; output o stands for u' = o + u0, whose window starts at dy row u' - (na-1)
                PlanSpec sp{};
                sp.N = N; sp.C = K; sp.H = bp->OH; sp.W = bp->OW; sp.K = C; sp.R = ph.na; sp.S = ph.nb; sp.stride = 1;
                sp.pad_h = ph.na - 1 - u0; sp.pad_w = ph.nb - 1 - v0;
                sp.OH = ph.UH; sp.OW = ph.UW;
                sp.om = OutMap{H, W, s, ph.oy, s, ph.ox};
                sp.direct = sp.over_split = s == 1 && !bp->small_default;
                sp.no_split = s > 1;  // (several sub-convolutions are contracted together, on fp32 MFMAs)
                st = plan_from_spec(&ph.sub, sp);
                if (st == DWM_OK) {
                    if (ph.sub->fused_ok) bp->wtmp_floats = std::max(bp->wtmp_floats, (size_t)C * K * ph.na * ph.nb);
                    bp->ws_bytes = std::max(bp->ws_bytes, dwm_plan_workspace_bytes(ph.sub));
                }
            }
            bp->phases.push_back(ph);
        }
    if (st != DWM_OK) {
        for (auto& ph : bp->phases)
            if (ph.sub) dwm_plan_destroy(ph.sub);
        delete bp;
        return st;
    }
    size_t off = (bp->wtmp_floats + 63) / 64 * 64;
    bp->wtmp_floats = off;
    for (auto& ph : bp->phases)
        if (ph.sub) {
            ph.u_off = off;
            off += (dwm_plan_filter_bytes(ph.sub) / sizeof(float) + 63) / 64 * 64;
        }
    bp->variant_path = -1;
    bp->u_small_off = off;
    if (bp->small_ok) off += (bp->small.u_floats + 63) / 64 * 64;
    bp->filter_floats = off;
    setup_batch(*bp);
    bp->direct = nullptr;
    if (stride > 1 && !bp->small_default) setup_direct(*bp);
    *out = bp;
    return DWM_OK;
}

dwm_status_t dwm_bwd_data_plan_destroy(dwm_bwd_data_plan_t* plan)
{
    if (!plan) return DWM_ERR_INVALID_ARG;
    for (auto& ph : plan->phases)
        if (ph.sub) dwm_plan_destroy(ph.sub);
    delete plan->merged;
    delete plan->direct;
    delete plan;
    return DWM_OK;
}

dwm_status_t dwm_bwd_data_plan_info(const dwm_bwd_data_plan_t* plan, dwm_bwd_data_info_t* info)
{
    if (!plan || !info) return DWM_ERR_INVALID_ARG;
    info->n_phases = (int)plan->phases.size();
    info->n_subconvs = 0;
    info->winograd_flops = 0.0;
    info->mults_per_input_block = 0;
    for (const auto& ph : plan->phases)
        if (ph.sub) {
            dwm_plan_info_t si;
            dwm_plan_info(ph.sub, &si);
            ++info->n_subconvs;
            info->winograd_flops += si.winograd_flops;
            info->mults_per_input_block += si.mults_per_tile;
        }
    info->direct_flops = plan->direct_flops;
    info->single_kernel = plan->use_small() ? 1 : 0;
    return DWM_OK;
}

dwm_status_t dwm_bwd_data_plan_phase(const dwm_bwd_data_plan_t* plan, int i, dwm_bwd_phase_t* out)
{
    if (!plan || !out || i < 0 || i >= (int)plan->phases.size()) return DWM_ERR_INVALID_ARG;
    const auto& ph = plan->phases[i];
    out->phase_h = ph.a; out->phase_w = ph.b; out->taps_h = ph.na; out->taps_w = ph.nb;
    out->first_h = ph.oy; out->first_w = ph.ox; out->count_h = ph.UH; out->count_w = ph.UW;
    out->has_subconv = ph.sub != nullptr;
    return DWM_OK;
}

int dwm_bwd_data_kernel(const dwm_bwd_data_plan_t* plan) { return !plan ? -1 : plan->use_small() ? 1 : plan->use_direct() || plan->use_sub_direct() ? 2 : 0; }

dwm_status_t dwm_bwd_data_set_variant(dwm_bwd_data_plan_t* plan, const char* stage, int variant)
{
    if (!plan || !stage) return DWM_ERR_INVALID_ARG;
    if (std::strcmp(stage, "path") != 0) return DWM_ERR_INVALID_ARG;
    if (variant < -1 || variant > 1) return DWM_ERR_INVALID_ARG;
    if (variant == 1 && !plan->small_ok) return DWM_ERR_UNSUPPORTED;
    plan->variant_path = variant;
    if (plan->s == 1 && plan->phases[0].sub) plan->phases[0].sub->no_direct = variant >= 0;
    return DWM_OK;
}

size_t dwm_bwd_data_filter_bytes(const dwm_bwd_data_plan_t* plan) { return plan ? plan->filter_floats * sizeof(float) : 0; }
size_t dwm_bwd_data_workspace_bytes(const dwm_bwd_data_plan_t* plan) { return plan ? plan->ws_bytes : 0; }

dwm_status_t dwm_bwd_data_set_workspace(dwm_bwd_data_plan_t* plan, void* ws_dev, size_t bytes)
{
    if (!plan) return DWM_ERR_INVALID_ARG;
    if (bytes < plan->ws_bytes) return DWM_ERR_WORKSPACE;
    if (plan->merged) {
        if (!ws_dev || ((uintptr_t)ws_dev & 255u)) return DWM_ERR_WORKSPACE;
        plan->merged->ws = static_cast<float*>(ws_dev);
        plan->merged->ws_bytes = bytes;
        plan->ws = static_cast<float*>(ws_dev);
        return DWM_OK;
    }
    for (size_t i = 0; i < plan->phases.size(); ++i) {
        auto& ph = plan->phases[i];
        if (!ph.sub) continue;
        const size_t off = plan->batched ? plan->ws_off[i] : 0;
        const dwm_status_t st = dwm_plan_set_workspace(ph.sub, ws_dev ? static_cast<char*>(ws_dev) + off : nullptr,
                                                       plan->batched ? dwm_plan_workspace_bytes(ph.sub) : bytes);
        if (st != DWM_OK) return st;
    }
    plan->ws = static_cast<float*>(ws_dev);
    return DWM_OK;
}

dwm_status_t dwm_bwd_data_filter_transform(const dwm_bwd_data_plan_t* plan, const float* w_dev, float* Ugw_dev,
                                           void* stream)
{
    // (a layer in which no tap reaches any pixel of dx -- stride above the kernel size on a narrow image -- has no
    // transformed filter at all: zero bytes, and no buffer to ask for)
    if (!plan || !w_dev || (!Ugw_dev && plan->filter_floats > 0)) return DWM_ERR_INVALID_ARG;
    if (plan->direct && !plan->filter_batched) {
        const long long rs = (long long)plan->R * plan->S;
        const dwm::FilterSource src{0, rs, rs * plan->C, -plan->s * plan->S, -plan->s};
        const dwm_status_t st = dwm::launch_filter_transform_from(*plan->direct, src, w_dev, Ugw_dev + plan->u_direct_off, stream);
        if (st != DWM_OK) return st;
    }
    if (plan->filter_batched) {
        const dwm_status_t st = dwm::launch_filter_batch(plan->filter_batch, w_dev, Ugw_dev, stream);
        if (st != DWM_OK) return st;
    }
    for (const auto& ph : plan->phases) {
        if (!ph.sub || plan->filter_batched) continue;
        // straight from w: flipped taps of the phase, filters and channels swapped (gathering them first took 17 us of
        // 58 for 256x256 filters of 7x7)
        const int s = plan->s;
        const long long rs = (long long)plan->R * plan->S;
        const dwm::FilterSource src{(long long)(s * (ph.na - 1) + ph.a) * plan->S + s * (ph.nb - 1) + ph.b, rs,
                                    rs * plan->C, -s * plan->S, -s};
        const dwm_status_t st = dwm::launch_filter_transform_from(*ph.sub, src, w_dev, Ugw_dev + ph.u_off, stream);
        if (st != DWM_OK) return st;
    }
    if (plan->small_ok)
        return dwm::launch_bwd_small_filter(plan->small, plan->R, plan->S, w_dev, Ugw_dev + plan->u_small_off, stream);
    return DWM_OK;
}

dwm_status_t dwm_conv_backward_data(const dwm_bwd_data_plan_t* plan, const float* dy_dev, const float* Ugw_dev,
                                    float* dx_dev, void* stream)
{
    if (!plan || !dy_dev || (!Ugw_dev && plan->filter_floats > 0) || !dx_dev) return DWM_ERR_INVALID_ARG;
    if (plan->use_small()) return dwm::launch_bwd_small(plan->small, dy_dev, Ugw_dev + plan->u_small_off, dx_dev, stream);
    const bool direct = plan->use_direct();
    if (direct && !plan->ws) return DWM_ERR_WORKSPACE;  // (it needs none; the other paths do)
    for (const auto& ph : plan->phases) {
        if (ph.UH <= 0 || ph.UW <= 0 || (direct && ph.sub)) continue;
        if (!ph.sub) {  // no tap reaches these pixels
            const size_t total = (size_t)plan->N * plan->C * ph.UH * ph.UW;
            const unsigned blocks = (unsigned)std::min<size_t>((total + 255) / 256, 8192);
            hipLaunchKernelGGL(dwm::bwd_zero_phase_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)stream, dx_dev,
                               plan->N * plan->C, plan->H, plan->W, plan->s, ph.oy, ph.ox, ph.UH, ph.UW);
            if (hipGetLastError() != hipSuccess) return DWM_ERR_HIP;
            continue;
        }
        if (plan->merged) continue;  // one input transform for all of them, below
        if (plan->batched) {  // its input transform now, its contraction with all the others below
            if (!plan->ws) return DWM_ERR_WORKSPACE;
            const dwm_status_t st = dwm::launch_input_transform(*ph.sub, dy_dev, ph.sub->ws, stream);
            if (st != DWM_OK) return st;
            continue;
        }
        const dwm_status_t st = dwm_conv_forward(ph.sub, dy_dev, Ugw_dev + ph.u_off, dx_dev, stream);
        if (st != DWM_OK) return st;
    }
    if (direct) return dwm::launch_direct(*plan->direct, dy_dev, Ugw_dev + plan->u_direct_off, dx_dev, nullptr, stream);
    if (plan->merged) {
        if (!plan->ws) return DWM_ERR_WORKSPACE;
        const dwm_status_t st = dwm::launch_input_transform(*plan->merged, dy_dev, plan->ws, stream);
        if (st != DWM_OK) return st;
    }
    if (plan->batched)
        return dwm::launch_contract_batch(plan->batch, plan->batch_planes, plan->batch_lc, Ugw_dev, plan->ws,
                                          plan->ws + plan->partial_off / sizeof(float), dx_dev, stream);
    return DWM_OK;
}

}  // extern "C"
