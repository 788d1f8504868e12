// Host-side geometry of two kernels of libdwm: which block of tiles a workgroup of the
// single-kernel forward path owns and how its input region is staged in LDS (fused.hip), and how
// the LDS-staged input transform stages its rows (transforms.hip).  Pure integer logic, no GPU
// call: this file and plan.cpp also build with a plain host compiler (sanitizer builds).
#include <algorithm>
#include <cmath>

#include "plan.hpp"

namespace dwm {

// ---------------------------------------------------------------------------------
// Single-kernel forward path: does it apply, and with which block of tiles
// ---------------------------------------------------------------------------------
bool fused_setup(const dwm_plan& p, FusedArgs* out)
{
    const DevPlan& d = p.d;
    FusedArgs f{};
    if (d.C > 127 || d.nh > 15 || d.nw > 15) return false;
    // classes = pairs of families; inside a class the rows (part, channel) follow each other sorted by
    // (len_h, len_w), longest first, and only the class's end is padded to a multiple of four.  A step
    // whose four rows mix piece lengths runs the planes of the longest: the shorter pieces' rows hold
    // zeros in the filter copy for the frequencies they lack.
    int rows = 0, steps = 0;
    int row_lh[kFusedMaxRows], row_lw[kFusedMaxRows];
    for (int wh = 1; wh >= 0; --wh)
        for (int ww = 1; ww >= 0; --ww) {
            FusedClass fc{};
            fc.wide_h = wh; fc.wide_w = ww;
            fc.nfh = wh ? 4 : 2; fc.nfw = ww ? 4 : 2;
            fc.step0 = steps; fc.row0 = rows;
            for (int lh = 3; lh >= 1; --lh)
                for (int lw = 3; lw >= 1; --lw) {
                    if ((lh >= 2) != (wh == 1) || (lw >= 2) != (ww == 1)) continue;
                    for (int a = 0; a < d.nh; ++a)
                        for (int b = 0; b < d.nw; ++b) {
                            if (d.ph[a].l != lh || d.pw[b].l != lw) continue;
                            for (int c = 0; c < d.C; ++c) {
                                if (rows >= kFusedMaxRows) return false;
                                f.rowdesc[rows] = (unsigned short)(a | b << 4 | c << 8 | 1 << 15);
                                row_lh[rows] = lh; row_lw[rows] = lw;
                                ++rows;
                            }
                        }
                }
            if (rows == fc.row0) continue;
            while ((rows - fc.row0) & 3) {  // padding rows: a real row's offsets, zero filter rows
                if (rows >= kFusedMaxRows) return false;
                f.rowdesc[rows] = (unsigned short)(f.rowdesc[rows - 1] & 0x7fff);
                row_lh[rows] = row_lh[rows - 1]; row_lw[rows] = row_lw[rows - 1];
                ++rows;
            }
            for (int r0 = fc.row0; r0 < rows; r0 += 4) {
                if (steps >= kFusedMaxSteps) return false;
                int mh = 0, mw = 0;
                for (int r = r0; r < r0 + 4; ++r) { mh = std::max(mh, row_lh[r]); mw = std::max(mw, row_lw[r]); }
                f.step_type[steps++] = mh * 4 + mw;
            }
            fc.nsteps = steps - fc.step0;
            fc.rows = rows - fc.row0;
            f.fc[f.nfc++] = fc;
        }
    f.rows_total = rows;

    // One class of two- and three-tap pieces only: the kernel then reads a patch row
    // as two pairs of adjacent LDS words (columns 0,2 and 1,3 of the patch lie 2*stride input columns
    // apart, i.e. one word apart in the de-interleaved row), also for two-tap pieces, whose fourth
    // column is then the input's real next element (it only meets zeros of the filter copy): the
    // staged region is as wide as if every piece had three taps.
    f.wide = f.nfc == 1 && f.fc[0].wide_h && f.fc[0].wide_w;
    int max_oh = 0, max_ow = 0;
    for (int i = 0; i < d.nh; ++i) max_oh = std::max(max_oh, d.s * (d.ph[i].j + d.ph[i].l) + d.ph[i].p);
    for (int i = 0; i < d.nw; ++i) max_ow = std::max(max_ow, d.s * (d.pw[i].j + (f.wide ? 3 : d.pw[i].l)) + d.pw[i].p);
    f.nphase = 2 * d.s;
    const size_t table_bytes = (size_t)rows * 64;
    const size_t budget = 72 * 1024;  // two workgroups per CU

    // block of `lanes` tiles: most useful lanes first, then the smallest staged region
    double best_eff = 0.0;
    size_t best_x = 0;
    auto choose_block = [&](int lanes, size_t limit) {
        best_eff = 0.0;
        best_x = 0;
        for (int bw = 1; bw <= lanes && bw <= d.TW; ++bw) {
            int bh = lanes / bw;
            if (bh > d.TH) bh = d.TH;
            if (bh < 1) continue;
            const int nbh = (d.TH + bh - 1) / bh, nbw = (d.TW + bw - 1) / bw;
            const double eff = (double)d.TH * d.TW / ((double)nbh * nbw * lanes);
            const long long nrows = 2LL * d.s * (bh - 1) + max_oh + 1;
            const long long lw_in = 2LL * d.s * (bw - 1) + max_ow + 1;
            const long long lwp = ((lw_in + f.nphase - 1) / f.nphase) | 1;
            const long long x_bytes = (long long)d.C * nrows * f.nphase * lwp * (long long)sizeof(float);
            if (x_bytes + (long long)table_bytes > (long long)limit) continue;
            if (eff > best_eff + 1e-9 || (eff > best_eff - 1e-9 && (size_t)x_bytes < best_x)) {
                best_eff = eff; best_x = (size_t)x_bytes;
                f.BH = bh; f.BW = bw; f.nbh = nbh; f.nbw = nbw;
                f.nrows = (int)nrows; f.lw_in = (int)lw_in; f.lwp = (int)lwp;
            }
        }
    };
    choose_block(64, budget);
    if (best_eff < 0.5) return false;
    long long blocks = (long long)d.N * f.nbh * f.nbw;
    if (blocks > 0x7fffffffLL) return false;
    f.nslices = (d.K + 31) / 32;
    // A handful of blocks: the time is one wave's walk through all the steps, on an idle chip.  Up to half a workgroup per
    // CU a block is 16 tiles instead of 64, and the workgroup's four waves take a quarter of the steps each and add up
    // their outputs in LDS (5x5 over 16 channels, one 32x32 image: 4 workgroups of 16 steps a wave 20.8 us, 16 of 4 steps 12.1;
    // 9x9 over 12 channels, 19x17: 30.5 -> 14.3; 7x7 stride 2 over 3 channels, 224x224: 12.0 -> 11.3).
    size_t sum_bytes = 0;
    if (blocks * f.nslices * 2 <= kNumCUs && steps >= 4) {
        const FusedArgs whole = f;
        const size_t whole_x = best_x;
        choose_block(16, budget - kFusedShareBytes);
        f.share = best_eff > 0.0;
        if (!f.share) {
            f = whole;
            best_x = whole_x;
        } else {
            blocks = (long long)d.N * f.nbh * f.nbw;
            sum_bytes = kFusedShareBytes;
        }
    }
    f.row_floats = f.nphase * f.lwp;
    f.chan_floats = f.nrows * f.row_floats;
    f.tile_row_step = 2 * d.s * f.row_floats;
    // with few blocks the filter slices are spread over workgroups as well
    f.slices_per_wg = blocks >= 2 * kNumCUs && !f.share ? f.nslices : 1;
    f.nkw = (f.nslices + f.slices_per_wg - 1) / f.slices_per_wg;
    if (f.nkw > 65535) return false;
    f.div_bw.init((unsigned)f.BW);
    f.div_nphase.init((unsigned)f.nphase);
    for (int i = 0; i < kMaxPieces; ++i)
        for (int k = 0; k < 4; ++k) {
            // offsets past a piece's own patch (k > its length) repeat its last element: they are read
            // (the patch is always read 4 wide) and only ever multiplied by zeros, but must be finite
            // (with a single class of two- and three-tap pieces the real fourth column is read instead: see above)
            const int kh = i < d.nh ? std::min(k, d.ph[i].l) : 0, kw = i < d.nw ? (f.wide ? k : std::min(k, d.pw[i].l)) : 0;
            const int oh = i < d.nh ? d.s * (d.ph[i].j + kh) + d.ph[i].p : 0;
            const int ow = i < d.nw ? d.s * (d.pw[i].j + kw) + d.pw[i].p : 0;
            f.roff[i][k] = oh * f.row_floats;
            f.coff[i][k] = (ow % f.nphase) * f.lwp + ow / f.nphase;
        }
    for (int i = 0; i < d.nw; ++i)  // columns two apart are one word apart in a de-interleaved row
        if (f.wide && (f.coff[i][2] != f.coff[i][0] + 1 || f.coff[i][3] != f.coff[i][1] + 1)) return false;
    f.lds_bytes = table_bytes + sum_bytes + best_x;
    *out = f;
    return true;
}

// Steps that a wave adds up of a problem's tile (of a piece of it)
static int direct_sum_steps(const DirectArgs& a, const DirectShape& sh, const DirectProb& q)
{
    auto share = [&](int steps) { return (steps + sh.wk - 1) / sh.wk; };
    return a.pieces > 1 ? a.cpp * share(q.steps[0]) : (a.nchunks - 1) * share(q.steps[0]) + share(q.steps[1]);
}

// What a workgroup of a direct convolution moves (shared: problems and pieces), in bytes of the 64-byte pieces of lines that memory
// gives and takes: a strip one pixel wide loads and stores sixteen times what it needs (the tiles beside it run on other XCDs).  x is
// read by a pixel tile's workgroups, all filters and problems, at about the same time on one XCD.
static double direct_bytes(int C, int K, int kt, int npx, int shared, int bw, int P, int row_px, int lwp, int s, int sx)
{
    auto pieces = [](int pixels, int step) { return 64.0 + 4.0 * (pixels - 1) * step; };
    const int nkt = (K + kt - 1) / kt, wide = (lwp - 1) * s + row_px / lwp;
    const double load = (double)C * P / row_px * std::min(pieces(wide, 1), 64.0 * row_px) / ((double)nkt * shared);
    const double store = (double)K / nkt * npx / bw * std::min(pieces(bw, sx), 64.0 * bw);
    return load + store;
}

// The time (us) of a direct convolution, fitted to 1700 (layer, shape) pairs drawn from the timed cases' ranges (forward and
// strided data gradients): cycles at 2.1 GHz of a workgroup -- its MFMAs, 340 a staged pixel and wave of a SIMD, 5400 a chunk (first
// loads, barriers), stores --, shared by the workgroups on a CU (registers allow two of 64-row wave tiles, three of 32), the address unit's
// 19 for each load and store, and 1.19 PFLOP/s as the most (long runs have reached 1.4: it errs on the side of the other paths); and
// what all tiles move, at 8 TB/s, as the other side of a right angle.  Over 3015 plans that the planner chose (rms of the logarithm of
// measured to modelled time) 0.16, 1.8 at worst; without the last term 0.22, and strips of one to three pixels up to 3.5 times as long as
// modelled: 1x1, 179 -> 218 channels, 49 37x37 images 74 by the model, 215 measured, 107 the contraction.
static double direct_us(const DirectArgs& a, const DirectShape& sh)
{
    const double w = sh.threads() / 256.0, waves = sh.threads() / 64.0, groups = std::min((a.C + 7) / 8, a.cpp * a.groups[0]);
    double mean = 0.0;
    for (int i = 0; i < a.nprob; ++i) mean += (double)direct_sum_steps(a, sh, a.p[i]) / a.nprob;
    const int fits = (int)(160 * 1024 / a.lds_bytes);
    const double on_cu = sh.threads() > 256 ? 1 : std::max(1, std::min(fits, sh.mb == 2 ? 2 : 3));
    const double slots = groups * a.ns, store = 1180.0 * sh.mb * w / sh.wk;
    const double lone = a.longest * 368.0 * sh.mb * w + slots * 340.0 * w + a.cpp * 5400.0 + store;
    auto shared = [&](double steps) {  // a workgroup's part of a CU's time
        const double simd = steps * 368.0 * sh.mb * w + slots * 340.0 * w + store;
        return std::max(simd, 19.0 * (slots * waves * 8 + steps * waves * 3 * sh.mb + sh.mb * 32 * waves / sh.wk * (a.sx > 1 ? 2 : 1)));
    };
    const double wgs = (double)a.ntiles * a.pieces, per_cu = wgs / kNumCUs, full = per_cu / on_cu, beside = std::min(on_cu, std::ceil(per_cu));
    const double rounds = std::max(1.0, full < 3 ? std::ceil(full) : full + 0.5);
    // (problems of several lengths: some of the longest tiles are among the last to start)
    const double together = a.nprob == 1 ? rounds * shared(mean) : full <= 1 ? shared(a.longest) : full * shared(mean) + 0.5 * shared(a.longest);
    const double cycles = std::max(rounds * lone, beside * together);
    const double flops = wgs * mean * waves * sh.mb * 2 * 6 * 32768.0;
    const double sum = a.pieces > 1 ? 3.0 + (2.0 * a.pieces + 1.0) * 4.0 * a.piece_floats / 5e6 : 0.0;
    const double alone = std::max(cycles / 2100.0, flops / 1.19e9) + 4.3 + sum, moved = wgs * direct_bytes(a.C, a.K, a.kt, a.npx, a.nprob * a.pieces, a.bw, a.P, a.row_px, a.lwp, a.s, a.sx) / 8e6;
    return std::sqrt(alone * alone + moved * moved);
}

// The direct convolution with one of its shapes, a tile's chunks shared by `pieces` workgroups.
bool direct_setup(int N, int C, int H, int W, int K, int s, int YH, int YW, int sy, int sx, const DirectProb* p, int n, int shape,
                  DirectArgs* out, int pieces)
{
    const DirectShape& sh = kDirectShapes[shape];
    DirectArgs a{};
    if (n < 1 || n > kDirectMaxProbs || s > 64) return false;
    if (pieces < 1 || pieces > kDirectMaxPieces || (pieces > 1 && (n > 1 || sy != 1 || sx != 1))) return false;  // (a piece's outputs lie as all of y)
    a.pieces = pieces;
    a.shape = shape; a.kt = sh.kt(); a.npx = sh.px();
    a.N = N; a.C = C; a.H = H; a.W = W; a.K = K; a.s = s;
    a.YH = YH; a.YW = YW; a.sy = sy; a.sx = sx;
    a.nprob = n;
    int R = 0, S = 0, Ph = 0, Pw = 0, OH = 0, OW = 0;
    for (int i = 0; i < n; ++i) {
        if (p[i].R > 64 || p[i].S > 64) return false;
        R = std::max(R, p[i].R); S = std::max(S, p[i].S);
        Ph = std::max(Ph, p[i].Ph); Pw = std::max(Pw, p[i].Pw);
        OH = std::max(OH, p[i].OH); OW = std::max(OW, p[i].OW);
        a.p[i] = p[i];
    }
    int taps = 0;
    for (int i = 0; i < n; ++i) taps = std::max(taps, p[i].R * p[i].S);
    a.OH = OH;
    const long long image = (long long)C * H * W, oplane = (long long)YH * YW, bias = (long long)Ph * W + Pw;
    if (image > (1LL << 29) || bias > (1LL << 28)) return false;
    a.bias = (int)bias;
    const int threads = sh.threads(), nph = std::min(s, S), ngroups = (C + 7) / 8;
    const long long rstep = std::min(s, R), rows_full = rstep * (long long)(OH - 1) + R;
    if (rows_full > (1 << 24)) return false;
    a.rstep = (int)rstep; a.run = R; a.rows_full = (int)rows_full;
    const size_t tables = 2 * kDirectMaxUnits * sizeof(int), reduce = sh.wk > 1 ? (size_t)threads * sh.mb * 128 : 0;
    const size_t lds_max = (threads <= 256 ? 80 : 160) * 1024 - tables;
    double best = 0.0;
    for (int nstrips = 1; nstrips <= 64 && nstrips <= OW; ++nstrips) {
        const int bw = (OW + nstrips - 1) / nstrips;
        const long long total_rows = (long long)N * nstrips * OH, total = total_rows * bw;
        if (total >= (1LL << 31) - 65536) continue;
        const long long nr = std::min<long long>(total_rows, a.npx % bw == 0 ? a.npx / bw : (a.npx + bw - 2) / bw + 1);
        const long long cross = nr <= 1 ? 0 : std::min<long long>((nr - 2) / OH + 1, (long long)N * nstrips - 1);
        const long long rows = rstep * nr + (cross + 1) * (R - rstep);
        const int lwp = bw + (S + s - 1) / s - 1;
        const long long row_px = (long long)lwp * nph, P = rows * row_px;
        if (P > (long long)kDirectSlots * threads || P < 1) continue;
        if ((cross + 1) * image * 4 + bias * 4 >= 0x7fff0000LL || ((cross + 1) * K + 256) * oplane * 4 >= 0x7fff0000LL) continue;
        const int ns = (int)((P + threads - 1) / threads);
        const double moved = direct_bytes(C, K, a.kt, a.npx, n * pieces, bw, (int)P, (int)row_px, lwp, s, sx) * (kNumCUs * 2100.0 / 8e6);
        // (no number of groups is below this)
        const double own = (double)ngroups / pieces;
        const double least = 0.5 * own * taps / sh.wk * sh.mb * 2 * 6 * 32 * (threads / 256.0) + own * ns * 400 * (threads / 256.0) + 3000.0;
        if (best > 0.0 && best <= std::sqrt(least * least + moved * moved) * bw * nstrips / OW) continue;
        for (int G = 1; G <= ngroups; ++G) {
            if ((size_t)G * P * 48 > lds_max || G * taps + 1 > kDirectMaxUnits) break;
            const int nchunks = (ngroups + G - 1) / G, gl = ngroups - (nchunks - 1) * G, cpp = (nchunks + pieces - 1) / pieces;
            if ((pieces - 1) * cpp >= nchunks) continue;  // a piece without a chunk
            // cycles of a tile of the longest problem, as in direct_us
            const double steps = (double)(cpp - 1) * ((G * taps + 1) / 2 + sh.wk - 1) + ((pieces > 1 ? G : gl) * taps + 1) / 2 + sh.wk - 1;
            const double busy = steps / sh.wk * sh.mb * 2 * 6 * 32 * (threads / 256.0) + (pieces > 1 ? cpp * G : ngroups) * (double)ns * 400 * (threads / 256.0) + cpp * 3000.0;
            const double cost = std::sqrt(busy * busy + moved * moved) * bw * nstrips / OW;
            if (best > 0.0 && cost >= best) continue;
            best = cost;
            a.bw = bw; a.nstrips = nstrips; a.total_px = (int)total;
            a.lwp = lwp; a.row_px = (int)row_px; a.P = (int)P; a.ns = ns;
            a.nchunks = nchunks; a.cpp = cpp;
            a.groups[0] = nchunks > 1 ? G : gl; a.groups[1] = gl;
            a.lds_bytes = std::max<size_t>((size_t)a.groups[0] * P * 48, reduce) + tables;
        }
    }
    if (best == 0.0) return false;
    a.ntt = (int)(((long long)a.total_px + a.npx - 1) / a.npx);
    a.nkt = (K + a.kt - 1) / a.kt;
    const long long per = (long long)a.nkt * n;
    if (a.ntt * per > 0x3fffffffLL || a.ntt * per * threads > 0xffffffffLL) return false;  // (a launch counts threads in 32 bits)
    a.piece_floats = pieces > 1 ? ((size_t)N * K * YH * YW + 63) / 64 * 64 : 0;
    a.ntiles = (int)(a.ntt * per);
    a.full8 = (int)(8 * per * (a.ntt / 8));
    a.Kpad = a.nkt * a.kt;
    long long steps = 0, w32 = 0;
    for (int i = 0; i < n; ++i) {
        DirectProb& q = a.p[i];
        const int t = q.R * q.S;
        q.steps[0] = (a.groups[0] * t + 1) / 2;
        q.steps[1] = (a.groups[1] * t + 1) / 2;
        q.step0 = (int)steps;
        q.w32 = w32;
        steps += (long long)(a.nchunks - 1) * q.steps[0] + q.steps[1];
        w32 += (long long)t * C * a.Kpad;
        if (steps * 96 * a.Kpad >= 0x7fff0000LL) return false;
    }
    a.all_steps = (int)steps;
    a.wd_bytes = (unsigned)(steps * 96 * a.Kpad);
    a.w32_floats = (size_t)w32;
    a.div_bw.init((unsigned)a.bw);
    a.div_oh.init((unsigned)OH);
    a.div_strips.init((unsigned)a.nstrips);
    a.div_row.init((unsigned)a.row_px);
    a.div_lwp.init((unsigned)a.lwp);
    a.div_rows.init((unsigned)a.rows_full);
    a.div_rstep.init((unsigned)a.rstep);
    for (int i = 0; i < n; ++i) a.longest = std::max(a.longest, direct_sum_steps(a, sh, a.p[i]));
    // (Measured where the other form begins to be further from 64 bits, with operands of zero mean and with positive ones: a tile's sum
    // in one wave from 88 steps on, shared by four waves from 117; at 82 to 97 steps of four waves one level is as good or better.)
    a.two_level = a.longest > (sh.wk > 1 ? 112 : 80);
    a.us = direct_us(a, sh);
    *out = a;
    return true;
}

bool direct_choose(int N, int C, int H, int W, int K, int s, int YH, int YW, int sy, int sx, const DirectProb* p, int n, DirectArgs* out,
                   size_t partial_floats)
{
    bool found = false;
    for (int shape = 0; shape < kNumDirectShapes; ++shape)
        for (int pieces : {1, 2, 3, 4, 6, 8, 12, 16}) {
            DirectArgs a;
            if (pieces > 1 && pieces * ((size_t)N * K * YH * YW + 63) > partial_floats) break;
            if (!direct_setup(N, C, H, W, K, s, YH, YW, sy, sx, p, n, shape, &a, pieces)) {
                if (pieces == 1) break;
                continue;
            }
            if (!found || a.us < out->us) *out = a;
            found = true;
            if ((long long)a.ntiles * pieces >= 2 * kNumCUs) break;  // (the chip is full)
        }
    return found;
}

// The direct filter gradient with the tile, patch, bands and pieces that take the least time by this model (fitted to 150 drawn
// layers, rms of the logarithm 0.22): cycles at 2 GHz of a workgroup's unit -- its MFMAs, 480 a wave's 64 staged pixels,
// 1.5 for each 128-byte line that dy's and x's rows touch, 2000 of latency --, of two workgroups on a CU their sum or the largest
// of what they share, a tile's sums at the end, and the pieces' trip through memory.
bool wd_setup(int N, int C, int H, int W, int K, int R, int S, int s, int P, int OH, int OW, WdArgs* out)
{
    const long long lim = 1LL << 29;  // (elements: byte offsets within an image are 32 bits, signed)
    if (((long long)C * H + R + P + 16LL * s) * W >= lim || (K + 64LL) * OH * OW >= lim || (long long)K * C * R * S >= (1LL << 31) - 64 || R > 64 || S > 64 || s > 64) return false;
    const long long cols = (long long)C * R * S;
    const int rs = R * S;
    if (cols >= (1LL << 30) || K > (1 << 24)) return false;
    bool found = false;
    for (int mb = K > 32 ? 2 : 1; mb >= 1; --mb)
        for (int nb : {5, 3, 2, 1})
            for (int lgw = 0; lgw <= 4; ++lgw) {
                const int kt = 32 * mb, ct = 32 * nb, PW = 1 << lgw, PH = 16 >> lgw;
                const long long ncol = (cols + ct - 1) / ct, nkt = (K + kt - 1) / kt, ntiles = ncol * nkt;
                const int nch = ncol == 1 ? C : std::min(C, ct % rs == 0 ? ct / rs : (ct - 2) / rs + 2);
                const int rows = s * (PH - 1) + R, pcols = s * (PW - 1) + S;
                const long long npix = (long long)nch * rows * pcols;
                const size_t lds = 16 * (size_t)(kt * 48 + 16) + (size_t)npix * 48;
                if (npix > 4096 || lds > 80 * 1024 || ntiles > (1 << 20)) continue;
                const double mfma = 439.0 * mb * nb, stage = (kt / 4 + (npix + 511) / 512 * 8) * 119.0, ends = 625.0 * mb * nb;
                const double lines = 1.5 * 8 * (kt * PH * (1 + (PW - 1) / 32.0) + nch * rows * (1 + (pcols - 1) / 32.0));
                const double lone = mfma + stage + lines + 1980.0;
                auto p4 = [](double v) { return v * v * v * v; };
                const double pair = std::sqrt(std::sqrt(p4(2 * mfma) + p4(2 * stage) + p4(2 * lines) + p4(lone)));
                for (int NB = 1; NB <= 8 && NB <= OH; ++NB) {
                    if (NB > 1 && N >= 64) break;
                    const int BH = (OH + NB - 1) / NB;
                    const long long npx = (OW + PW - 1) / PW, npy = (BH + PH - 1) / PH, groups = ((long long)N * NB + 7) / 8;
                    const long long nunits = groups * npx * npy;
                    if (nunits >= (1 << 29)) continue;
                    for (int target : {256, 512, 1024}) {
                        const long long xunits = (nunits + 7) / 8, per = std::min(std::max(1LL, target / ntiles / 8), xunits);
                        const long long upp = (xunits + per - 1) / per, pieces = nunits <= 8 ? nunits : 8 * per;
                        const long long wgs = pieces * ntiles, left = wgs % 512;
                        const double cycles = (wgs / 512) * (upp * pair + ends) + (left > 256 ? upp * pair + ends : left > 0 ? upp * lone + ends : 0.0);
                        const double bytes = (double)K * cols * 4 * pieces;
                        const double us = 3.5 + cycles / 2000.0 + (pieces > 1 ? 2.2 + 2 * bytes / 4.3e6 : 0.0);
                        if ((found && us >= out->us) || bytes > 256e6) continue;
                        found = true;
                        WdArgs a{};
                        a.N = N; a.C = C; a.H = H; a.W = W; a.K = K; a.R = R; a.S = S; a.s = s; a.P = P; a.OH = OH; a.OW = OW;
                        a.NB = NB; a.BH = BH; a.lgw = lgw;
                        a.per_image = NB > 1 || ((long long)C * H + R + P + 16LL * s) * W >= lim / 8 || (K + 64LL) * OH * OW >= lim / 8;
                        a.npx = (int)npx; a.npy = (int)npy; a.nunits = (int)nunits; a.xunits = (int)xunits; a.ustep = (int)per; a.pieces = (int)pieces;
                        a.cols = (int)cols; a.nkt = (int)nkt; a.ntiles = (int)ntiles;
                        a.rows = rows; a.pcols = pcols; a.mb = mb; a.nb = nb;
                        a.stride = (int)((K * cols + 63) / 64 * 64);
                        a.lds_bytes = lds;
                        a.us = us;
                        *out = a;
                    }
                }
            }
    if (!found) return false;
    out->div_rs.init((unsigned)rs);
    out->div_plane.init((unsigned)(out->rows * out->pcols));
    out->div_pcols.init((unsigned)out->pcols);
    out->div_nb.init((unsigned)out->NB);
    out->div_npx.init((unsigned)out->npx);
    out->div_npy.init((unsigned)out->npy);
    return true;
}

// Does the LDS-staged form apply, and with how many channels per workgroup: the rows a block
// stages must fit in LDS.  The row count depends on where a block of 64 tiles starts; the
// pattern repeats after at most TH*TW blocks, so the maximum is found by walking them.
bool input_lds_setup(const dwm_plan& p, InLdsArgs* out, int cg_wish)
{
    const DevPlan& d = p.d;
    InLdsArgs a{};
    int max_oh = 0, max_ow = 0;
    for (int i = 0; i < d.nh; ++i) max_oh = std::max(max_oh, d.s * (d.ph[i].j + d.ph[i].l) + d.ph[i].p);
    for (int i = 0; i < d.nw; ++i) max_ow = std::max(max_ow, d.s * (d.pw[i].j + d.pw[i].l) + d.pw[i].p);
    if (d.s > 4096 || max_oh > (1 << 20) || max_ow > (1 << 20)) return false;
    a.nphase = 2 * d.s;
    a.foot_h = max_oh + 1;
    const long long lw_in = 2LL * d.s * (d.TW - 1) + max_ow + 1;
    const long long rows_full = 2LL * d.s * (d.TH - 1) + a.foot_h;
    if (lw_in > (1 << 16) || rows_full > (1 << 24)) return false;
    a.lw_in = (int)lw_in;
    a.lwp = ((a.lw_in + a.nphase - 1) / a.nphase) | 1;
    a.row_floats = a.nphase * a.lwp;
    a.rows_full = (int)rows_full;
    const long long per = (long long)d.TH * d.TW;
    const long long nb = (d.T + 63) / 64, scan = std::min(nb, per);
    long long max_rows = 0;
    const int s2 = 2 * d.s;
    for (long long bt = 0; bt < scan; ++bt) {
        const long long t0 = bt * 64, t1 = std::min<long long>(t0 + 63, d.T - 1);
        const long long g0 = t0 / d.TW, g1 = t1 / d.TW, n0 = g0 / d.TH, n1 = g1 / d.TH;
        const long long ty_a0 = g0 - n0 * d.TH, ty_b1 = g1 - n1 * d.TH;
        const long long rows0 = s2 * ((n1 == n0 ? ty_b1 : d.TH - 1) - ty_a0) + a.foot_h;
        const long long total = n1 == n0 ? rows0 : rows0 + (n1 - n0 - 1) * rows_full + s2 * ty_b1 + a.foot_h;
        max_rows = std::max(max_rows, total);
        if (max_rows * a.row_floats * 4 > 64 * 1024) return false;
    }
    a.max_rows = (int)max_rows;
    a.chan_floats = a.max_rows * a.row_floats;
    const size_t chan_bytes = (size_t)a.chan_floats * sizeof(float);
    if (chan_bytes > 64 * 1024) return false;
    // channels per workgroup: one per wave (measured best: many small workgroups keep more loads
    // and stores in flight than fewer large ones)
    int cg = d.C < 4 ? d.C : 4;
    while (cg > 1 && cg * chan_bytes > 150 * 1024) --cg;  // (a channel's region fits by the check above)
    if (cg_wish > 0 && cg_wish <= d.C && cg_wish * chan_bytes <= 150 * 1024) cg = cg_wish;
    a.cg = cg;
    a.ncg = (d.C + cg - 1) / cg;
    if ((long long)a.ncg * (d.Tpad / 64) > 0x7fffffffLL) return false;
    a.div_tw.init((unsigned)d.TW);
    a.div_th.init((unsigned)d.TH);
    a.div_lw.init((unsigned)a.lw_in);
    a.div_nphase.init((unsigned)a.nphase);
    a.div_rows_full.init((unsigned)a.rows_full);
    for (int i = 0; i < kMaxPieces; ++i)
        for (int k = 0; k < 4; ++k) {
            const int oh = i < d.nh ? d.s * (d.ph[i].j + k) + d.ph[i].p : 0;
            const int ow = i < d.nw ? d.s * (d.pw[i].j + k) + d.pw[i].p : 0;
            a.roff[i][k] = oh * a.row_floats;
            a.coff[i][k] = (ow % a.nphase) * a.lwp + ow / a.nphase;
        }
    a.lds_bytes = (size_t)cg * chan_bytes;
    *out = a;
    return true;
}

// ---------------------------------------------------------------------------------
// 16-bit kernel from x to y for many input channels (half_wide.inc)
// ---------------------------------------------------------------------------------
// images that a block of 64 tiles spans beyond its first
static double more_images(const DevPlan& d)
{
    const double per = (double)d.TH * d.TW;
    return per < 64.0 ? std::min(d.N - 1.0, 64.0 / per) : 0.0;
}

// What the staged path takes (us): its input transform in one of three forms (gather; staged in LDS by groups of eight
// channels, or all channels in a workgroup; a wave stages its channels image by image), then its contraction, tiles whole or cut
// into ranges.  V past 220 MB no longer stays in the memory-side cache.  Fitted by least squares of the relative error: each
// stage timed alone on 9000 layers of 17-1024 channels, what images, a large V and parts of one tap (V is x itself) add on
// 6000 whole calls: nine in ten of those within -11 and +22 %.
static double staged16_us(const dwm_plan& p, const InLdsArgs* lds)
{
    const DevPlan& d = p.d;
    const ContractGeometry& g = p.geo;
    int planes = 0, parts = p.info.n_parts;  // planes summed over the parts
    for (int i = 0; i < d.ncls; ++i) planes += d.cls[i].hn * d.cls[i].wn * (d.cls[i].lh + 1) * (d.cls[i].lw + 1);
    const double v = 2e-6 * p.info.mults_per_tile * d.C * d.T, x = 2e-6 * d.N * d.C * d.H * d.W, y = 2e-6 * d.N * d.K * d.OH * d.OW;  // MB
    const double blocks = (double)((d.T + 63) / 64), per_part = (double)planes / parts;
    double in;
    if (!lds) {
        in = 1.6 * std::ceil(blocks * std::ceil((double)parts * d.C / 32.0) / (8 * kNumCUs)) + 0.5 * v + 1.3 * d.ncls + 0.97 * per_part;
    } else {
        const double kb = (double)lds->lds_bytes / 1024.0, per_cu = std::min(8.0, std::max(1.0, std::floor(160.0 / (kb + 1.0))));
        const double rounds = std::ceil(blocks * lds->ncg / (kNumCUs * per_cu)), items = std::ceil(lds->cg / 8.0 * parts / 4.0);
        in = d.C % 8 == 0 ? 5.0 + rounds * (2.1 + 0.0265 * kb + 0.1 * items * per_part) + 0.127 * v + 0.141 * x
                          : 4.8 + rounds * (items * (1.29 + 0.415 * per_part) + 0.084 * kb) + 0.066 * v + 1.72 * d.ncls;
        in += 0.1 * rounds * lds->cg * more_images(d);
    }
    // start, a chunk of the longest workgroup, chunks per CU of all tiles, a class, pieces per CU, a MB of y, of V
    struct Ct { double start, chunk, all, cls, piece, y, v; };
    const bool whole = g.n_full > 0;
    const Ct c = g.variant == 44   ? (whole ? Ct{1.5, 0.229, 0.144, 2.21, 30.3, 0.51, 0.057} : Ct{13.7, 0.302, 0.125, 1.41, 19.1, 0.32, 0.0})
                 : g.variant == 32 ? (whole ? Ct{3.7, 0.311, 0.0, 1.10, 3.2, 0.22, 0.047} : Ct{10.3, 0.242, 0.0, 1.17, 10.2, 0.44, 0.032})
                 : g.variant == 31 ? (whole ? Ct{7.2, 0.114, 0.0, 2.77, 7.6, 0.02, 0.083} : Ct{9.9, 0.179, 0.0, 1.53, 12.6, 0.85, 0.0})
                                   : (whole ? Ct{9.6, 0.077, 0.0, 3.42, 4.9, 0.0, 0.044} : Ct{10.1, 0.148, 0.0, 1.43, 13.6, 0.31, 0.0});
    const double longest = whole ? g.n_iter * std::ceil((double)g.n_full / kNumCUs) + (g.n_sk_tiles > 0 ? g.sk_ipw : 0) : g.sk_ipw;
    const double contract = c.start + c.chunk * longest + c.all * (double)g.ntiles * g.n_iter / kNumCUs + c.cls * d.ncls +
                            c.piece * (double)g.n_sk_tiles * std::max(g.sk_f, 1) / kNumCUs + c.y * y + c.v * v;
    return 1.02 * (in + contract) + 0.6 + 0.15 * std::max(0.0, v - 220.0) - (planes == 4 * parts ? 2.9 : 0.0);
}

bool wide16_setup(const dwm_plan& p, size_t partial_room, const InLdsArgs* staged_lds, Wide16Args* out)
{
    const DevPlan& d = p.d;
    Wide16Args f{};
    if (d.om.sy != 1 || d.om.sx != 1 || d.om.oy != 0 || d.om.ox != 0 || d.om.YH != d.OH || d.om.YW != d.OW) return false;
    if (d.Ph < 0 || d.Pw < 0 || d.C < kWideC || d.s > 64) return false;
    int max_oh = 0, max_ow = 0, planes = 0;
    for (int i = 0; i < d.nh; ++i) max_oh = std::max(max_oh, d.s * (d.ph[i].j + d.ph[i].l) + d.ph[i].p);
    for (int i = 0; i < d.nw; ++i) max_ow = std::max(max_ow, d.s * (d.pw[i].j + d.pw[i].l) + d.pw[i].p);
    for (int i = 0; i < d.ncls; ++i) planes = std::max(planes, (d.cls[i].lh + 1) * (d.cls[i].lw + 1));
    f.v_bytes = planes * kWideT * kWideC * 2;
    f.nphase = 2 * d.s;
    f.foot_h = max_oh + 1;
    const long long lw_in = 2LL * d.s * (d.TW - 1) + max_ow + 1, rows_full = 2LL * d.s * (d.TH - 1) + f.foot_h;
    if (lw_in > 4096 || rows_full > (1 << 20)) return false;
    f.lw_in = (int)lw_in;
    f.lwp = (f.lw_in + f.nphase - 1) / f.nphase;
    f.row_px = f.nphase * f.lwp;
    f.rows_full = (int)rows_full;
    f.npairs = (d.W + 1) / 2;
    const int s2 = 2 * d.s;
    const long long row_bytes = (long long)f.row_px * 2 * kWideC, px_bytes = 2 * kWideC,
                    room = 160 * 1024 - 2LL * f.v_bytes - 2 * px_bytes - 16LL * p.info.n_parts;
    const long long per = (long long)d.TH * d.TW, nb = (d.T + kWideT - 1) / kWideT;
    long long max_rows = 0;
    for (long long bt = 0; bt < std::min(nb, per); ++bt) {
        const long long t0 = bt * kWideT, t1 = std::min<long long>(t0 + kWideT - 1, d.T - 1);
        const long long g0 = t0 / d.TW, g1 = t1 / d.TW, n0 = g0 / d.TH, n1 = g1 / d.TH;
        const long long ty_a0 = g0 - n0 * d.TH, ty_b1 = g1 - n1 * d.TH;
        const long long rows0 = s2 * ((n1 == n0 ? ty_b1 : d.TH - 1) - ty_a0) + f.foot_h;
        max_rows = std::max(max_rows, n1 == n0 ? rows0 : rows0 + (n1 - n0 - 1) * rows_full + s2 * ty_b1 + f.foot_h);
        if (max_rows * (2 * row_bytes + 8LL * f.npairs) > room) return false;
    }
    f.max_rows = (int)max_rows;
    f.x_px = (int)(max_rows * f.row_px) + 1;  // (a last pixel for what is staged nowhere)
    f.x_bytes = (f.x_px * 2 * kWideC + 15) / 16 * 16;
    f.lds_bytes = std::max<size_t>((size_t)2 * (f.v_bytes + f.x_bytes) + 16 * (size_t)p.info.n_parts +
                                       8 * (size_t)f.max_rows * f.npairs, kWideExchangeBytes);
    // a block's images are addressed through a 31-bit buffer offset
    if ((kWideT / per + 2) * d.C * d.H * d.W * 2 >= (1LL << 31)) return false;
    f.div_tw.init((unsigned)d.TW);
    f.div_th.init((unsigned)d.TH);
    f.div_np.init((unsigned)f.npairs);
    f.div_phase.init((unsigned)f.nphase);
    const int px = 8;  // LDS bytes of a pixel: four channels
    f.row_step = d.s * f.row_px * px;
    for (int i = 0; i < kMaxPieces; ++i) {
        f.roff[i] = i < d.nh ? (d.s * d.ph[i].j + d.ph[i].p) * f.row_px * px : 0;
        for (int k = 0; k < 2; ++k) {
            const int ow = i < d.nw ? d.s * (d.pw[i].j + k) + d.pw[i].p : 0;
            f.coff[i][k] = ((ow % f.nphase) * f.lwp + ow / f.nphase) * px;
        }
    }
    f.chunks = (d.C + kWideC - 1) / kWideC;
    f.nkt = (d.K + kWideK - 1) / kWideK;
    f.ntt = (int)nb;
    f.nparts = p.info.n_parts;
    // the staged path's filter serves where the parts' rows are whole chunks
    f.own_copy = d.C % kWideC != 0;
    f.rows_per_part = f.chunks * kWideC;
    long long words = 0;  // of 16 bytes
    for (int i = 0; i < d.ncls; ++i) {
        const DevClass& q = d.cls[i];
        Wide16Class& c = f.cls[(3 - q.lh) * 3 + (3 - q.lw)];
        const long long plane = (f.own_copy ? (long long)q.hn * q.wn * f.rows_per_part : q.Lpad) * d.Kpad / 8;
        f.has |= 1 << ((3 - q.lh) * 3 + (3 - q.lw));
        c.n = q.hn * q.wn;
        c.wn = q.wn; c.h0 = q.h0; c.w0 = q.w0;
        c.plane_bytes = (unsigned)(plane * 16);
        c.u_off = (unsigned)(words * 16);  // (the staged filter's classes lie one after the other too)
        words += (q.lh + 1) * (q.lw + 1) * plane;
        if (words * 16 >= (1LL << 31)) return false;
    }
    f.u_bytes = (size_t)words * 16;
    f.uw_words = f.own_copy ? (size_t)words : 0;

    // Into how many pieces the channels are cut, by a rough estimate (us): a workgroup fills a CU; its launch, first loads and last stores take 9; a stage
    // 0.75 and 0.055 for each of its planes (a share of pixels that no longer fits beside the products 0.7 per 1024 items;
    // pixels one by one, where W is odd, 0.15 for every item of a thread); pieces are added up by a kernel of its own, 4 and
    // 0.2 per MB.
    const double items = (double)f.max_rows * f.npairs * 4 / f.nparts, batch = items <= 256 ? 1 : items <= 512 ? 2 : 4;
    int all_planes = 0;  // of a chunk's stages
    for (int i = 0; i < kMaxClasses; ++i) all_planes += f.cls[i].n * (4 - i / 3) * (4 - i % 3);
    const double stages = f.nparts * (0.75 + 0.7 * std::floor(items / 1024.0) + (d.W & 1 ? 0.15 * batch : 0.0)) + 0.055 * all_planes;
    double best = 1e30;
    for (int n = 1; n <= kWideMaxPieces && n <= f.chunks; ++n) {
        const int cpw = (f.chunks + n - 1) / n, pieces = (f.chunks + cpw - 1) / cpw;
        const long long wgs = (long long)f.nkt * f.ntt * pieces;
        const size_t partial = (size_t)wgs * kWideK * kWideT * 4 * sizeof(float);
        if (pieces != n || (n > 1 && partial > partial_room)) continue;
        const double us = (double)((wgs + kNumCUs - 1) / kNumCUs) * (9.0 + cpw * stages) + (n > 1 ? 4.0 + 0.2e-6 * (double)partial : 0.0);
        if (us >= best) continue;
        best = us;
        f.nsplit = n;
        f.cpw = cpw;
    }
    // Not where that is above as rough an estimate of the staged path: V written and read and x read at 5 TB/s, its products at
    // 400 TFLOP/s, 15 for launches and start-up, and what few tiles cannot hide of a chunk's latency.
    const double v = (double)p.info.mults_per_tile * d.C * d.T;
    const double rough = 15.0 + (4.0 * v + 2.0 * d.N * d.C * d.H * d.W) / 5e6 + 2.0 * v * d.K / 4e8 + 0.15 * p.geo.n_iter;
    if (best >= (d.W & 1 ? 0.85 : 1.0) * rough) return false;
    // Whether it is the default: its time as a call (us), fitted like the staged path's (nine in ten within 8 %), at least 5 %
    // below it.  Of 8000 other layers that come here 278 are more than 2 % slower than on the staged path, by up to 54 %; of the
    // 7521 that this takes 36 are, by up to 19 %, and 170 of those it leaves would be faster by more than 2 %, by up to 27 %.
    const double wgs = (double)f.nkt * f.ntt * f.nsplit, rounds = std::ceil(wgs / kNumCUs);
    f.us = 3.9 + 0.29e-6 * 2.0 * d.N * d.K * d.OH * d.OW + (d.W & 1 ? 0.5 : 0.0) +
           rounds * (11.9 + 0.25 * more_images(d) +
                     f.cpw * (0.08 * all_planes + f.nparts * (0.36 * std::floor(items / 1024.0) + (0.088 + (d.W & 1 ? 0.141 : 0.0)) * batch))) +
           (f.nsplit > 1 ? 0.31 * f.nsplit - 3.5 + 0.264e-6 * wgs * kWideK * kWideT * 16 : 0.0);
    f.pays = f.us < 0.95 * staged16_us(p, staged_lds);
    *out = f;
    return true;
}

// ---------------------------------------------------------------------------------
// Single-kernel data gradient (few input channels): window, pieces, block of tiles, LDS
// ---------------------------------------------------------------------------------
// One dimension: residues of the dx coordinate modulo the stride, the common window of dy and
// its cut into pieces of three and two taps (3,...,3 then 2 or 2,2: never a single tap).
static bool bwd_small_dim(int R, int s, int P, int* ra, int* re, int* rn, int* L, int* nwin, int* np, int* pj, int* pl)
{
    bool any = false;
    int lmax = 0, emax = 0;
    for (int rho = 0; rho < s; ++rho) {
        const int a = (rho + P) % s, e = (rho + P) / s;
        const int n = a < R ? (R - a + s - 1) / s : 0;
        ra[rho] = a; re[rho] = e; rn[rho] = n;
        if (n == 0) continue;
        if (!any || n - 1 - e > lmax) lmax = n - 1 - e;
        if (!any || e > emax) emax = e;
        any = true;
    }
    if (!any) return false;
    *L = lmax;
    const int n = emax + lmax + 1;
    *nwin = n;
    if (n < 2 || n > 11) return false;
    int cnt = 0, j = 0, left = n;
    while (left > 0) {
        const int l = (left == 2 || left == 4) ? 2 : 3;
        if (cnt >= kBsMaxPieces) return false;
        pj[cnt] = j; pl[cnt] = l;
        ++cnt; j += l; left -= l;
    }
    *np = cnt;
    return true;
}

bool bwd_small_setup(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, BwdSmallArgs* out)
{
    BwdSmallArgs f{};
    const int s = stride;
    if (s < 1 || s > 8 || N < 1 || C < 1 || K < 1 || pad < 0 || pad > (1 << 20) || H > (1 << 20) || W > (1 << 20)) return false;
    f.N = N; f.C = C; f.H = H; f.W = W; f.K = K; f.s = s;
    f.OH = (H + 2 * pad - R) / s + 1;
    f.OW = (W + 2 * pad - S) / s + 1;
    if (f.OH < 1 || f.OW < 1) return false;
    // one image of dy is addressed through a 32-bit buffer offset, dx through 32-bit pixel offsets
    if ((long long)K * f.OH * f.OW * 4 >= (1LL << 31) || (long long)H * W >= (1LL << 29)) return false;
    const long long nf = (long long)C * s * s;
    if (nf > 256) return false;
    f.nf = (int)nf;
    f.ncb = (f.nf + 15) / 16;
    // column blocks a wave accumulates in one pass over dy: the fewest passes, then the fewest blocks per pass
    f.nb = 1;
    for (int nb = 2; nb <= 3; ++nb)
        if ((f.ncb + nb - 1) / nb < (f.ncb + f.nb - 1) / f.nb) f.nb = nb;
    f.ncbp = (f.ncb + f.nb - 1) / f.nb * f.nb;
    if (!bwd_small_dim(R, s, pad, f.ra_h, f.re_h, f.rn_h, &f.Lh, &f.nwh, &f.nph, f.jh, f.lh)) return false;
    if (!bwd_small_dim(S, s, pad, f.ra_w, f.re_w, f.rn_w, &f.Lw, &f.nww, &f.npw, f.jw, f.lw)) return false;
    f.npp = f.nph * f.npw;
    f.four = 0;
    for (int i = 0; i < f.nph; ++i) f.four |= f.lh[i] == 3;
    for (int i = 0; i < f.npw; ++i) f.four |= f.lw[i] == 3;
    const int nfreq = f.four ? 4 : 3, planes = nfreq * nfreq;
    const int th = (H + s - 1) / s, tw = (W + s - 1) / s;  // window positions per dimension
    f.TH = (th + 1) / 2; f.TW = (tw + 1) / 2;
    // the patch of a piece is read nfreq wide whatever its length
    const int max_oh = f.jh[f.nph - 1] + nfreq - 1, max_ow = f.jw[f.npw - 1] + nfreq - 1;
    // Bank conflicts of a patch read: LDS serves 32 lanes a cycle from 32 banks of four bytes.  A group of
    // four channels is staged as two planes of channel pairs, [element][2]; the lanes of half a wave are
    // 16 tiles x the two channels of one pair and read word 2*(element of the tile) + (channel & 1).
    // Returns the worst multiplicity of a bank over the four waves.
    auto conflicts = [&](int bw, int bh, int lwp) {
        int worst = 0;
        for (int wave = 0; wave < 4; ++wave) {
            int cnt[32] = {0};
            for (int n = 0; n < 16; ++n) {
                const int tl = wave * 16 + n, by = tl / bw, bx = tl % bw;
                const int el = by < bh ? by * 4 * lwp + bx : 0;
                for (int q = 0; q < 2; ++q) worst = std::max(worst, ++cnt[(2 * el + q) & 31]);
            }
        }
        return worst;
    };
    // block of tiles: most useful lanes first, then the cheapest staged region; the chunk of channels is the
    // largest (8, 16 or 32) with which two workgroups fit a CU, else 8
    double best_eff = 0.0;
    long long best_x = 0, best_cost = 0;
    for (int bw = 1; bw <= 64 && bw <= f.TW; ++bw) {
        int bh = 64 / bw;
        if (bh > f.TH) bh = f.TH;
        if (bh < 1) continue;
        const int nbh = (f.TH + bh - 1) / bh, nbw = (f.TW + bw - 1) / bw;
        const double eff = (double)f.TH * f.TW / ((double)nbh * nbw * 64);
        const long long nrows = 2LL * (bh - 1) + max_oh + 1;
        const long long lw_in = 2LL * (bw - 1) + max_ow + 1;
        if (nrows * lw_in > 256LL * kBsMaxSlots / 2) continue;
        int nelog = 0;
        while ((256LL << nelog) < nrows * lw_in) ++nelog;
        // the largest chunk first; for it, the row padding with the fewest bank conflicts that still fits
        const long long lwp0 = (lw_in + 1) / 2;
        long long lwp = lwp0, group = 0;
        int glog = -1;
        // (nine planes leave registers for three waves per SIMD: three workgroups per CU, 52 KB each;
        // sixteen planes: two, 79 KB each; with several column blocks per wave two and one, 79 and 150 KB;
        // a chunk of four channels only with an even number of steps)
        const int wg_kb = f.nb > 1 ? (f.four ? 150 : 79) : (f.four ? 79 : 52);
        for (int g = 3; g >= 0 && glog < 0; --g) {
            if ((1 << g) << nelog > kBsMaxSlots || ((f.npp << g) & 1)) continue;
            const long long us = ((long long)(f.npp << g) * planes * 64 + 255) / 256 * 256;
            int best_c = 1 << 30;
            for (long long l = lwp0; l < lwp0 + 4; ++l) {
                const long long grp = nrows * 2 * l;  // elements of four floats
                const long long bytes = 2 * ((grp << g) * 4 + f.nb * us) * (long long)sizeof(float);
                if (bytes > (g > (f.npp & 1) ? wg_kb : 150) * 1024) continue;
                const int c = conflicts(bw, bh, (int)l);
                if (c < best_c) { best_c = c; lwp = l; group = grp; glog = g; }
            }
        }
        if (glog < 0) continue;
        const long long xs = (group << glog) * 4;
        // among equally full blocks: the least to load, a row of the region counted 16 elements longer than
        // it is (short rows waste most of the memory transactions that fetch them)
        const long long cost = nrows * (lw_in + 16);
        if (eff > best_eff + 1e-9 || (eff > best_eff - 1e-9 && cost < best_cost)) {
            best_eff = eff; best_x = xs; best_cost = cost;
            f.BH = bh; f.BW = bw; f.nbh = nbh; f.nbw = nbw;
            f.nrows = (int)nrows; f.lw_in = (int)lw_in; f.lwp = (int)lwp;
            f.glog = glog; f.nelog = nelog;
        }
    }
    if (best_eff <= 0.0) return false;
    f.eff_pct = (int)(best_eff * 100.0);
    if ((long long)N * f.nbh * f.nbw > 0x7fffffffLL) return false;
    f.ck = 4 << f.glog;
    f.steps = f.npp << f.glog;
    f.nchunks = (K + f.ck - 1) / f.ck;
    f.us_floats = (f.steps * planes * 64 + 255) / 256 * 256;  // whole 1 KB pieces: one DMA instruction of a wave each
    f.row_elems = 2 * f.lwp;
    f.group_elems = f.nrows * f.row_elems;
    f.tile_row_step = 2 * f.row_elems;
    f.xs_floats = (int)best_x;
    f.div_bw.init((unsigned)f.BW);
    f.div_lw.init((unsigned)f.lw_in);
    for (int pp = 0; pp < f.npp; ++pp) {
        const int jh = f.jh[pp / f.npw], jw = f.jw[pp % f.npw];
        f.po0[pp] = 8 * (jh * f.row_elems + (jw & 1) * f.lwp + (jw >> 1));
        f.po1[pp] = 8 * (jh * f.row_elems + ((jw + 1) & 1) * f.lwp + ((jw + 1) >> 1));
    }
    // LDS: two staged chunks of dy, two chunks of the filter copy, the table of patch offsets
    f.lds_bytes = 2 * ((size_t)f.xs_floats + (size_t)f.nb * f.us_floats) * sizeof(float) + kBsMaxPairs * 8;
    f.u_floats = (size_t)f.ncbp * f.nchunks * f.us_floats;
    *out = f;
    return true;
}

// ---------------------------------------------------------------------------------
// 16-bit single-kernel forward path: classes, rows, block of tiles, LDS
// ---------------------------------------------------------------------------------
bool fused16_setup(const dwm_plan& p, Fused16Args* out)
{
    const DevPlan& d = p.d;
    Fused16Args f{};
    if (d.C > 127 || d.nh > 15 || d.nw > 15 || d.ncls > kMaxClasses) return false;
    if (d.om.sy != 1 || d.om.sx != 1 || d.om.oy != 0 || d.om.ox != 0 || d.om.YH != d.OH || d.om.YW != d.OW) return false;
    f.nkb = (d.K + 15) / 16;
    f.slice_kb = std::min(f.nkb, 2);  // (the launcher sets what its kernel takes)
    f.nslices = (f.nkb + f.slice_kb - 1) / f.slice_kb;
    int rows = 0;
    size_t uf = 0;
    for (int qi = 0; qi < d.ncls; ++qi) {
        const DevClass& q = d.cls[qi];
        Fused16Class fc{};
        fc.lh = q.lh; fc.lw = q.lw;
        fc.L = q.L;
        fc.row0 = rows;
        fc.nsteps = (q.L + 15) / 16;
        fc.uf_off = (long long)uf;
        for (int l = 0; l < fc.nsteps * 16; ++l) {
            if (rows >= kF16MaxRows) return false;
            const int lr = std::min(l, q.L - 1);  // padding rows: the last real row's patch, zero filter rows
            const int slot = lr / d.C, c = lr - slot * d.C;
            const int a = slot / q.wn, b = slot - a * q.wn;
            f.rowdesc[rows++] = (unsigned short)((q.h0 + a) | (q.w0 + b) << 4 | c << 8);
        }
        uf += (size_t)f.nkb * fc.nsteps * (q.lh + 1) * (q.lw + 1) * 256;
        f.cls[f.ncls++] = fc;
    }
    f.rows_total = rows;
    f.uf_halves = uf;
    if (uf * 2 >= ((size_t)1 << 31)) return false;  // addressed through a 32-bit buffer offset
    if ((long long)d.K * d.OH * d.OW * 4 >= (1LL << 31)) return false;  // ... and so is one image of y

    int max_oh = 0, max_ow = 0;
    for (int i = 0; i < d.nh; ++i) max_oh = std::max(max_oh, d.s * (d.ph[i].j + d.ph[i].l) + d.ph[i].p);
    for (int i = 0; i < d.nw; ++i) max_ow = std::max(max_ow, d.s * (d.pw[i].j + d.pw[i].l) + d.pw[i].p);
    f.nphase = 2 * d.s;
    const size_t table_bytes = (size_t)rows * 8;
    const size_t budget = 76 * 1024;  // two workgroups per CU
    double best_eff = 0.0;
    size_t best_x = 0;
    for (int bw = 1; bw <= 64 && bw <= d.TW; ++bw) {
        int bh = 64 / bw;
        if (bh > d.TH) bh = d.TH;
        if (bh < 1) continue;
        const int nbh = (d.TH + bh - 1) / bh, nbw = (d.TW + bw - 1) / bw;
        const double eff = (double)d.TH * d.TW / ((double)nbh * nbw * 64);
        const long long nrows = 2LL * d.s * (bh - 1) + max_oh + 1;
        const long long lw_in = 2LL * d.s * (bw - 1) + max_ow + 1;
        const long long lwp = ((lw_in + f.nphase - 1) / f.nphase) | 1;
        const long long x_bytes = (long long)d.C * nrows * f.nphase * lwp * (long long)sizeof(float);
        if (x_bytes + (long long)table_bytes > (long long)budget) continue;
        if (eff > best_eff + 1e-9 || (eff > best_eff - 1e-9 && (size_t)x_bytes < best_x)) {
            best_eff = eff; best_x = (size_t)x_bytes;
            f.BH = bh; f.BW = bw; f.nbh = nbh; f.nbw = nbw;
            f.nrows = (int)nrows; f.lw_in = (int)lw_in; f.lwp = (int)lwp;
        }
    }
    if (best_eff <= 0.0) return false;
    f.eff_pct = (int)(best_eff * 100.0);
    if ((long long)d.N * f.nbh * f.nbw > 0x7fffffffLL) return false;
    f.row_floats = f.nphase * f.lwp;
    f.chan_floats = f.nrows * f.row_floats;
    f.tile_row_step = 2 * d.s * f.row_floats;
    f.patch_row_bytes = d.s * f.row_floats * 4;
    f.div_bw.init((unsigned)f.BW);
    f.div_nphase.init((unsigned)f.nphase);
    for (int i = 0; i < kMaxPieces; ++i) {
        const int oh = i < d.nh ? d.s * d.ph[i].j + d.ph[i].p : 0;
        const int ow0 = i < d.nw ? d.s * d.pw[i].j + d.pw[i].p : 0, ow1 = ow0 + d.s;
        f.roff[i] = oh * f.row_floats;
        f.coff0[i] = (ow0 % f.nphase) * f.lwp + ow0 / f.nphase;
        f.coff1[i] = (ow1 % f.nphase) * f.lwp + ow1 / f.nphase;
    }
    f.lds_bytes = table_bytes + best_x;
    *out = f;
    return true;
}

}  // namespace dwm
