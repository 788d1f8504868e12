// HIP kernels of libdwm for gfx950 (MI355X): filter transform and input transform, the
// "Transformation" step of the paper's Sec. 4.1 list on the kernel and on the input side
// (the input side includes the "Splitting" of the input into per-part, per-phase views).
// Winograd matrices are those of Sec. 3.2 for F(2,3) and the 0/1-entry three- and
// two-multiplication forms for 2-tap and 1-tap pieces.
#include <hip/hip_runtime.h>

#include "direct_filter.hpp"
#include "fused_filter.hpp"
#include "plan.hpp"
#include "split.hpp"
#include "xform.hpp"

namespace dwm {

// ---------------------------------------------------------------------------------
// Filter transform: U = G_lh g G_lw^T for every part (Sec. 4.1 "Transformation")
// One thread per (row of the flattened (class, l) space, k); writes all planes of its
// class, zeros in the padding.  w is read where it lies (FilterSource), also by the data gradient.
// ---------------------------------------------------------------------------------
__device__ __forceinline__ void filter_part(const DevPlan& P, const DevClass& q, const FilterSource& F,
                                            const float* __restrict__ w, int l, int k, float (&u)[4][4])
{
    const int th = q.lh + 1, tw = q.lw + 1;
    const bool real = l < q.L && k < P.K;
    const int slot = real ? l / P.C : 0, c = real ? l - slot * P.C : 0;
    const int a = slot / q.wn, b = slot - a * q.wn;
    const DevPiece hp = P.ph[q.h0 + a], wp = P.pw[q.w0 + b];
    const float* wk = w + F.base + (real ? k * F.sk + c * F.sc : 0);
    float g[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            g[i][j] = real && i < q.lh && j < q.lw
                          ? wk[(P.s * (hp.j + i) + hp.p) * F.sr + (P.s * (wp.j + j) + wp.p) * F.ss] : 0.f;
    float t[4][3];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) t[i][j] = (i < th) ? g_row(q.lh, i, g[0][j], g[1][j], g[2][j]) : 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) u[i][j] = (i < th && j < tw) ? g_row(q.lw, j, t[i][0], t[i][1], t[i][2]) : 0.f;
}

__device__ __forceinline__ void filter_rows(const DevPlan& P, const FilterSource& F, const float* __restrict__ w, float* __restrict__ U,
                                            int row, int k)
{
    if (row >= P.rows_total) return;
    const int qi = find_class(P, row);
    const DevClass q = P.cls[qi];
    const int l = row - q.row0;
    const int th = q.lh + 1, tw = q.lw + 1;

    float u[4][4];
    filter_part(P, q, F, w, l, k, u);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (i < th && j < tw) {
                U[(size_t)q.u_off + ((size_t)(i * tw + j) * P.Kpad + k) * q.Lpad + l] = u[i][j];
            }
}

__global__ __launch_bounds__(256) void filter_transform_kernel(DevPlan P, FilterSource F, const float* __restrict__ w,
                                                               float* __restrict__ U)
{
    filter_rows(P, F, w, U, blockIdx.x * 256 + threadIdx.x, blockIdx.y);
}

// The same, and beside it the copies of the single-kernel path (fused.hip) and of the direct convolution (direct.hip), where the
// plan has them: workgroups 0.. write the class layout, fused0.. the first, direct0.. the second; gap: floats between the copies,
// which belong to the buffer.  A copy is a microsecond of work behind four of a launch: with the copies of fused.hip in a launch
// of their own, and w gathered by a third where a data gradient reads it, training steps of first layers took 4 us more (7x7 at
// stride 2, 64 224x224 images, 471 -> 466 us; 6x6 at stride 4, 7 101x101 images, 50 -> 46) and with nine such phases 97.
struct FilterCopies {
    int gx;  // workgroups of rows of the class layout
    int fused0, direct0, end;
    long long gap0, gap1, gap2, gap3;
};
__global__ __launch_bounds__(256) void filter_copies_kernel(DevPlan P, FilterSource F, FusedArgs Fu, DirectArgs D, FilterCopies B,
                                                            const float* __restrict__ w, float* __restrict__ U)
{
    const int b = blockIdx.x, t = threadIdx.x;
    if (b < B.fused0) {
        filter_rows(P, F, w, U, (b % B.gx) * 256 + t, b / B.gx);
        if (b == 0) {
            for (long long i = B.gap0 + t; i < B.gap1; i += 256) U[i] = 0.f;
            for (long long i = B.gap2 + t; i < B.gap3; i += 256) U[i] = 0.f;
        }
    } else if (b < B.direct0) {
        fused_filter(P, Fu, F, w, U, t, b - B.fused0);  // (kFusedMaxRows is one workgroup's)
    } else {
        const int nk = (D.Kpad + 127) / 128, e = b - B.direct0;
        direct_filter(D, F, w, U + B.gap3, e / nk, e % nk);
    }
}
static_assert(kFusedMaxRows <= 256, "rows of fused_filter");
static_assert(sizeof(DevPlan) + sizeof(FilterSource) + sizeof(FusedArgs) + sizeof(DirectArgs) + sizeof(FilterCopies) + 16 <= 4096, "kernel arguments");

// The same for several stride-1 sub-convolutions that read one w (the phases of a data gradient), one grid plane each: four
// launches of 4.3 us and the gaps between them for a 5x5 layer at stride 2 with 67 and 93 channels become one.  Further grid
// planes write the direct convolution's filter.
__global__ __launch_bounds__(256) void filter_transform_batch_kernel(FilterBatchArgs A, const float* __restrict__ w, float* __restrict__ U)
{
    if ((int)blockIdx.z >= A.nprob) {
        const int b = ((blockIdx.z - A.nprob) * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x, nk = (A.direct.Kpad + 127) / 128;
        if (b < A.direct_blocks) direct_filter(A.direct, FilterSource{0, A.sk, A.sc, A.sr, A.ss}, w, U + A.direct_off, b / nk, b % nk);
        return;
    }
    const FilterBatchProb& P = A.p[blockIdx.z];
    const int row = blockIdx.x * blockDim.x + threadIdx.x, k = blockIdx.y;
    if (row >= P.rows_total) return;
    int qi = 0;
    while (qi + 1 < P.ncls && row >= P.cls[qi + 1].row0) ++qi;
    const FilterBatchClass q = P.cls[qi];
    const int l = row - q.row0, th = q.lh + 1, tw = q.lw + 1;
    const bool real = l < q.L && k < A.K;
    const int slot = real ? l / A.C : 0, c = real ? l - slot * A.C : 0;
    const int a = slot / q.wn, b = slot - a * q.wn;
    const float* wk = w + P.base + (real ? k * A.sk + c * A.sc + P.jh[q.h0 + a] * A.sr + P.jw[q.w0 + b] * A.ss : 0);
    float g[3][3], t[4][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) g[i][j] = real && i < q.lh && j < q.lw ? wk[i * A.sr + j * A.ss] : 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) t[i][j] = i < th ? g_row(q.lh, i, g[0][j], g[1][j], g[2][j]) : 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (i < th && j < tw)
                U[(size_t)q.u_off + ((size_t)(i * tw + j) * A.Kpad + k) * q.Lpad + l] = g_row(q.lw, j, t[i][0], t[i][1], t[i][2]);
}

// The same, and beside it U split three ways for contract_split.hip (its layout is described there).  A workgroup takes
// 32 rows x 8 filters, a thread one of each: the stores of U are whole 128-byte lines.  The split copy has eight rows
// side by side in a lane and the filters next to each other, so the planes pass through LDS, and a thread then splits
// eight rows of one filter: again whole lines.  Bound by its 65 MB of stores and the scattered reads of w: 24.6 us for
// 256x256 filters of 7x7, read flipped and transposed by the data gradient; 58 us as a gather of w, a transform and a
// pass that split U.  (A thread with eight rows of its own and no LDS leaves the chip short of waves: 40 us.)
constexpr int kFtRows = 32, kFtK = 8, kFtPitch = kFtRows + 4;
__device__ __forceinline__ void filter_split_rows(const DevPlan& P, const FilterSource& F, const float* __restrict__ w,
                                                  float* __restrict__ U, uint32_t* __restrict__ US, int bx, int by)
{
    __shared__ alignas(16) float sm[16][kFtK][kFtPitch];
    const int t = threadIdx.x, rbase = bx * kFtRows, kbase = by * kFtK;
    {
        const int r = t & (kFtRows - 1), kk = t / kFtRows, row = rbase + r, k = kbase + kk;
        if (row < P.rows_total) {
            const DevClass q = P.cls[find_class(P, row)];
            const int l = row - q.row0, tw = q.lw + 1;
            float u[4][4];
            filter_part(P, q, F, w, l, k, u);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (i <= q.lh && j <= q.lw) {
                        U[(size_t)q.u_off + ((size_t)(i * tw + j) * P.Kpad + k) * q.Lpad + l] = u[i][j];
                        sm[i * tw + j][kk][r] = u[i][j];
                    }
        }
    }
    __syncthreads();
    const int kk = t & (kFtK - 1), rg = (t / kFtK) & 3, row = rbase + rg * 8;  // eight rows are of one class
    if (row >= P.rows_total) return;
    const DevClass q = P.cls[find_class(P, row)];
    const int l = row - q.row0, planes = (q.lh + 1) * (q.lw + 1);
    uint32_t* dst = US + (size_t)q.u_off / 2 * 3 + ((size_t)(l >> 4) * 6 + ((l >> 3) & 1)) * P.Kpad * 4 + (size_t)(kbase + kk) * 4;
    for (int p = t >> 5; p < planes; p += 8) {
        float x[8];
        *reinterpret_cast<float4*>(x) = *reinterpret_cast<const float4*>(&sm[p][kk][rg * 8]);
        *reinterpret_cast<float4*>(x + 4) = *reinterpret_cast<const float4*>(&sm[p][kk][rg * 8 + 4]);
        // (what its parts cannot hold is marked: contract_split.hip takes such filters on the fp32 matrix cores)
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (x[i] != 0.f && fabsf(x[i]) < kSplitMin) x[i] = __builtin_nanf("");
        bf16x8 f[3];
        split8(x, f);
        uint32_t* dp = dst + (size_t)p * P.Kpad * q.Lpad / 2 * 3;
#pragma unroll
        for (int part = 0; part < 3; ++part)
            *reinterpret_cast<puint4*>(dp + (size_t)part * 2 * P.Kpad * 4) = __builtin_bit_cast(puint4, f[part]);
    }
}

__global__ __launch_bounds__(256) void filter_transform_split_kernel(DevPlan P, FilterSource F, const float* __restrict__ w,
                                                                     float* __restrict__ U, uint32_t* __restrict__ US)
{
    filter_split_rows(P, F, w, U, US, blockIdx.x, blockIdx.y);
}

// The same, and beside it the direct convolution's copy: workgroups from direct0 on (the gap before it: filter_copies_kernel)
__global__ __launch_bounds__(256) void filter_split_copies_kernel(DevPlan P, FilterSource F, DirectArgs D, FilterCopies B,
                                                                  const float* __restrict__ w, float* __restrict__ U, uint32_t* __restrict__ US)
{
    const int b = blockIdx.x;
    if (b >= B.direct0) {
        const int nk = (D.Kpad + 127) / 128, e = b - B.direct0;
        direct_filter(D, F, w, U + B.gap3, e / nk, e % nk);
        return;
    }
    if (b == 0)
        for (long long i = B.gap2 + threadIdx.x; i < B.gap3; i += 256) U[i] = 0.f;
    filter_split_rows(P, F, w, U, US, b % B.gx, b / B.gx);
}

// ---------------------------------------------------------------------------------
// Input transform: V = B^T d B for every part (Sec. 4.1 "Splitting" of the input and
// "Transformation").
//
// A thread owns one tile t and FOUR consecutive rows l of the flattened (class, l) space
// (four channels of one part, as a rule).  For each row it gathers the part's
// (lh+1)x(lw+1) patch d[a][b] = xp[s(2ty+jh+a)+ph][s(2tx+jw+b)+pw] (phase p of the padded
// input, eq. 14 generalised to any stride) straight from global memory -- L1/L2 absorb the
// re-reads of overlapping patches; all four rows' loads are issued before the first use so
// that enough bytes are in flight -- applies the transform and writes one value per plane.
// V is blocked by 64 tiles: a wave's store is one 256-byte row, a workgroup (64 tiles x 16
// rows) writes 4 KB contiguous per plane.
// ---------------------------------------------------------------------------------
template <int LH, int LW>
__device__ __forceinline__ void input_rows4(const DevPlan& P, const DevClass& q, const float* __restrict__ x,
                                            float* __restrict__ V, int l0, int t)
{
    constexpr int TH_ = LH + 1, TW_ = LW + 1;
    float d[4][TH_][TW_];
    const bool t_ok = t < P.T;
    const int tiles = P.TH * P.TW;
    const int n = t / tiles, rem = t - n * tiles;
    const int ty = rem / P.TW, tx = rem - ty * P.TW;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int l = l0 + r;
        const bool ok = l < q.L && t_ok;
        const int slot = l / P.C, c = l - slot * P.C;
        const int a = slot / q.wn, b = slot - a * q.wn;
        const DevPiece hp = P.ph[q.h0 + (ok ? a : 0)], wp = P.pw[q.w0 + (ok ? b : 0)];
        const float* xc = x + ((size_t)n * P.C + c) * P.H * P.W;
#pragma unroll
        for (int i = 0; i < TH_; ++i) {
            const int ih = P.s * (2 * ty + hp.j + i) + hp.p - P.Ph;
#pragma unroll
            for (int j = 0; j < TW_; ++j) {
                const int iw = P.s * (2 * tx + wp.j + j) + wp.p - P.Pw;
                d[r][i][j] = (ok && ih >= 0 && ih < P.H && iw >= 0 && iw < P.W) ? xc[(size_t)ih * P.W + iw] : 0.f;
            }
        }
    }
    if (!t_ok) return;  // columns past the last tile are never read back into y
    float* vp = V + (size_t)(t >> 6) * P.vblock_rows * 64 + (size_t)(q.v_row0 + l0) * 64 + (t & 63);
    const size_t plane = (size_t)q.Lpad * 64;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        // columns first (B^T d), then rows ((B^T d) B)
        float tmp[4][4];
#pragma unroll
        for (int j = 0; j < TW_; ++j) {
            float col[4] = {0.f, 0.f, 0.f, 0.f}, o[4];
#pragma unroll
            for (int i = 0; i < TH_; ++i) col[i] = d[r][i][j];
            bt_apply<LH>(col, o);
#pragma unroll
            for (int i = 0; i < TH_; ++i) tmp[i][j] = o[i];
        }
#pragma unroll
        for (int i = 0; i < TH_; ++i) {
            float rowv[4] = {0.f, 0.f, 0.f, 0.f}, o[4];
#pragma unroll
            for (int j = 0; j < TW_; ++j) rowv[j] = tmp[i][j];
            bt_apply<LW>(rowv, o);
#pragma unroll
            for (int j = 0; j < TW_; ++j) vp[(size_t)(i * TW_ + j) * plane + r * 64] = o[j];
        }
    }
}

__global__ __launch_bounds__(256) void input_transform_kernel(DevPlan P, const float* __restrict__ x,
                                                              float* __restrict__ V, int* __restrict__ counters,
                                                              int n_counters, int rows_fast)
{
    // The contraction that follows counts partial-tile arrivals in `counters`; they start at zero.
    if (blockIdx.x == 0 && blockIdx.y == 0)
        for (int i = threadIdx.x; i < n_counters; i += blockDim.x) counters[i] = 0;

    // Workgroup order.  rows_fast: consecutive workgroups take consecutive row groups of the SAME
    // 64-tile block, so every part and channel of those tiles is in flight together and x is
    // fetched from HBM once (it matters when x outgrows the L2).  Otherwise consecutive
    // workgroups take consecutive blocks of the same rows (measured faster while x stays cached).
    const int bt = rows_fast ? blockIdx.y : blockIdx.x, br = rows_fast ? blockIdx.x : blockIdx.y;
    const int t = bt * 64 + (threadIdx.x & 63);          // < Tpad by construction of the grid
    const int row = br * 16 + (threadIdx.x >> 6) * 4;    // 4 rows, never across a class (Lpad % 16 == 0)
    const int qi = find_class(P, row);
    const DevClass q = P.cls[qi];
    const int l0 = row - q.row0;
    switch (q.lh * 4 + q.lw) {
        case 3 * 4 + 3: input_rows4<3, 3>(P, q, x, V, l0, t); break;
        case 3 * 4 + 2: input_rows4<3, 2>(P, q, x, V, l0, t); break;
        case 3 * 4 + 1: input_rows4<3, 1>(P, q, x, V, l0, t); break;
        case 2 * 4 + 3: input_rows4<2, 3>(P, q, x, V, l0, t); break;
        case 2 * 4 + 2: input_rows4<2, 2>(P, q, x, V, l0, t); break;
        case 2 * 4 + 1: input_rows4<2, 1>(P, q, x, V, l0, t); break;
        case 1 * 4 + 3: input_rows4<1, 3>(P, q, x, V, l0, t); break;
        case 1 * 4 + 2: input_rows4<1, 2>(P, q, x, V, l0, t); break;
        default: input_rows4<1, 1>(P, q, x, V, l0, t); break;
    }
}


// ---------------------------------------------------------------------------------
// Input transform, LDS-staged form.
//
// A workgroup owns one 64-tile block of V (lane = tile) and `cg` input channels.  Each of
// its four waves stages the input rows that the block's tiles touch, for ITS channels
// (c = c0 + wave, c0 + wave + 4, ...), once, with coalesced loads: zero padding is written
// explicitly and columns are de-interleaved modulo 2*stride, so that the same patch element
// of adjacent tiles sits in adjacent LDS words.  The wave then walks every part of every
// class for those channels: a patch element is one LDS read at (lane's tile base) + (an
// offset that is the same for the whole wave).  x is read from HBM about once and every
// load instruction is fully used; the global-memory gathers of the other form (one 4-byte
// load per patch element, lanes 2*stride floats apart) are gone.  Waves never wait for each
// other: a wave reads only what it staged itself.
// The 64 tiles of a block span a few tile rows, possibly of several images: the staged rows
// are the union per image ("segments"), stored one after the other.
// SHARED: a workgroup owns one channel, its waves take a quarter of the rows and then of the parts each.  For layers whose
// workgroups of four channels leave CUs without one, where a wave's chain of loads, rows and parts is the time: 13.0 ->
// 11.7 us for a 5x5 layer at stride 2 (67 channels, five 35x29 images).
// ---------------------------------------------------------------------------------
template <int LH, int LW, bool SHARED, bool TAIL>
__device__ __forceinline__ void lds_class_rows(const DevPlan& P, const InLdsArgs& A, const DevClass& q,
                                               const float* __restrict__ xl, float* __restrict__ vb, int c0,
                                               int cn, int wave, bool valid, int& part)
{
    constexpr int TH_ = LH + 1, TW_ = LW + 1;
    const size_t plane = (size_t)q.Lpad * 64;
    for (int a = 0; a < q.hn; ++a)
        for (int b = 0; b < q.wn; ++b) {
            if (SHARED && (part++ & 3) != wave) continue;
            int ro[TH_], co[TW_];
#pragma unroll
            for (int i = 0; i < TH_; ++i) ro[i] = A.roff[q.h0 + a][i];
#pragma unroll
            for (int j = 0; j < TW_; ++j) co[j] = A.coff[q.w0 + b][j];
            const int lbase = (a * q.wn + b) * P.C + c0;
            for (int cl = SHARED ? 0 : wave; cl < cn; cl += 4) {
                const float* xc = xl + cl * A.chan_floats;
                float d[TH_][TW_];
#pragma unroll
                for (int i = 0; i < TH_; ++i)
#pragma unroll
                    for (int j = 0; j < TW_; ++j) d[i][j] = xc[ro[i] + co[j]];
                float* vp = vb + (size_t)(q.v_row0 + lbase + cl) * 64;
                // columns first (B^T d), then rows ((B^T d) B)
                float tmp[4][4];
#pragma unroll
                for (int j = 0; j < TW_; ++j) {
                    float col[4] = {0.f, 0.f, 0.f, 0.f}, o[4];
#pragma unroll
                    for (int i = 0; i < TH_; ++i) col[i] = d[i][j];
                    bt_apply<LH>(col, o);
#pragma unroll
                    for (int i = 0; i < TH_; ++i) tmp[i][j] = o[i];
                }
#pragma unroll
                for (int i = 0; i < TH_; ++i) {
                    float rowv[4] = {0.f, 0.f, 0.f, 0.f}, o[4];
#pragma unroll
                    for (int j = 0; j < TW_; ++j) rowv[j] = tmp[i][j];
                    bt_apply<LW>(rowv, o);
                    if (TAIL || valid) {
#pragma unroll
                        for (int j = 0; j < TW_; ++j) vp[(size_t)(i * TW_ + j) * plane] = valid ? o[j] : 0.f;
                    }
                }
            }
        }
}

// TAIL: the columns past the last tile of the last block are written as zeros (a launch of its own took 4 us; stores after
// the rows' 2.5 for a 9x9 layer at stride 4, whose rows are many)
template <bool SHARED, bool TAIL>
__global__ __launch_bounds__(256) void input_transform_lds_kernel(DevPlan P, InLdsArgs A,
                                                                  const float* __restrict__ x,
                                                                  float* __restrict__ V, int* __restrict__ counters,
                                                                  int n_counters, int chan_fast, int write_pad_rows)
{
    extern __shared__ __attribute__((aligned(16))) float xs[];  // [cg][max_rows][nphase][lwp]
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < n_counters; i += blockDim.x) counters[i] = 0;

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int nbt = P.Tpad / 64;
    const int b = blockIdx.x;
    const int bt = chan_fast ? b / A.ncg : b % nbt, bc = chan_fast ? b % A.ncg : b / nbt;
    const int c0 = bc * A.cg, cn = min(A.cg, P.C - c0);
    const int t0 = bt * 64;
    if (t0 >= P.T) return;  // a block of padding only (Tpad is rounded up to 256)
    const int t1 = min(t0 + 63, P.T - 1);
    const int s2 = 2 * P.s;
    const int g0 = A.div_tw.div(t0), g1 = A.div_tw.div(t1);
    const int n0 = A.div_th.div(g0), n1 = A.div_th.div(g1);
    const int ty_a0 = g0 - n0 * P.TH, ty_b1 = g1 - n1 * P.TH;
    const int rows0 = s2 * ((n1 == n0 ? ty_b1 : P.TH - 1) - ty_a0) + A.foot_h;

    // ---- 1. this wave stages its channels: lanes along a row, rows in batches of up to
    // kInLdsBatch loads, segment by segment.  Rows above or below the image are written as
    // zeros; columns left or right of it are loaded from a clamped (legal) address and
    // replaced by zero on the way to LDS.
    if constexpr (SHARED) {
        stage_channels<float, 1, true>(P, A, x, xs, c0, 4, n0, n1, ty_a0, ty_b1, lane, wave);
        __syncthreads();
    } else {
        for (int cl = wave; cl < cn; cl += 4)
            stage_channels<float, 1>(P, A, x, xs + cl * A.chan_floats, c0 + cl, 4, n0, n1, ty_a0, ty_b1, lane);
    }

    // ---- 2. every part of every class for those channels ----
    const int t = t0 + lane;
    const bool valid = t < P.T;
    int lane_base = 0;
    if (valid) {
        const int g = A.div_tw.div(t), tx = t - g * P.TW;
        const int n = A.div_th.div(g), ty = g - n * P.TH;
        const int base_row = n == n0 ? s2 * (ty - ty_a0) : rows0 + (n - n0 - 1) * A.rows_full + s2 * ty;
        lane_base = base_row * A.row_floats + tx;
    }
    const float* xl = xs + lane_base;
    float* vb = V + (size_t)bt * P.vblock_rows * 64 + lane;
    int part = 0;
    for (int qi = 0; qi < P.ncls; ++qi) {
        const DevClass q = P.cls[qi];
        switch (q.lh * 4 + q.lw) {
            case 3 * 4 + 3: lds_class_rows<3, 3, SHARED, TAIL>(P, A, q, xl, vb, c0, cn, wave, valid, part); break;
            case 3 * 4 + 2: lds_class_rows<3, 2, SHARED, TAIL>(P, A, q, xl, vb, c0, cn, wave, valid, part); break;
            case 3 * 4 + 1: lds_class_rows<3, 1, SHARED, TAIL>(P, A, q, xl, vb, c0, cn, wave, valid, part); break;
            case 2 * 4 + 3: lds_class_rows<2, 3, SHARED, TAIL>(P, A, q, xl, vb, c0, cn, wave, valid, part); break;
            case 2 * 4 + 2: lds_class_rows<2, 2, SHARED, TAIL>(P, A, q, xl, vb, c0, cn, wave, valid, part); break;
            case 2 * 4 + 1: lds_class_rows<2, 1, SHARED, TAIL>(P, A, q, xl, vb, c0, cn, wave, valid, part); break;
            case 1 * 4 + 3: lds_class_rows<1, 3, SHARED, TAIL>(P, A, q, xl, vb, c0, cn, wave, valid, part); break;
            case 1 * 4 + 2: lds_class_rows<1, 2, SHARED, TAIL>(P, A, q, xl, vb, c0, cn, wave, valid, part); break;
            default: lds_class_rows<1, 1, SHARED, TAIL>(P, A, q, xl, vb, c0, cn, wave, valid, part); break;
        }
        // rows past the class's reduction length are zeros (the contraction multiplies them)
        if (bc == 0 && (TAIL || valid) && write_pad_rows) {
            const int planes = (q.lh + 1) * (q.lw + 1);
            for (int l = q.L + wave; l < q.Lpad; l += 4)
                for (int pl = 0; pl < planes; ++pl) vb[((size_t)q.v_row0 + (size_t)pl * q.Lpad + l) * 64] = 0.f;
        }
    }
}

// ---------------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------------
static dwm_status_t check_launch()
{
    return hipGetLastError() == hipSuccess ? DWM_OK : DWM_ERR_HIP;
}

dwm_status_t launch_filter_transform_from(const dwm_plan& p, const FilterSource& src, const float* w, float* U, void* stream)
{
    const DevPlan& d = p.d;
    if (p.direct_only) return launch_direct_filter(p.direct, src, w, U + p.ud_begin, stream);
    if (p.split_ok && p.direct_ok) {
        FilterCopies b{};
        b.gx = (d.rows_total + kFtRows - 1) / kFtRows;
        b.direct0 = b.gx * (d.Kpad / kFtK);
        b.end = b.direct0 + p.direct.all_steps * ((p.direct.Kpad + 127) / 128);
        b.gap2 = (long long)p.ud_gap; b.gap3 = (long long)p.ud_begin;
        hipLaunchKernelGGL(filter_split_copies_kernel, dim3(b.end), dim3(256), 0, (hipStream_t)stream, d, src, p.direct, b, w, U,
                           reinterpret_cast<uint32_t*>(U + p.us_begin));
    } else if (p.fused_ok || p.direct_ok) {
        FilterCopies b{};
        b.gx = (d.rows_total + 255) / 256;
        b.fused0 = b.gx * d.Kpad;
        b.direct0 = b.fused0 + (p.fused_ok ? p.fused.nslices * 32 : 0);
        b.end = b.direct0 + (p.direct_ok ? p.direct.all_steps * ((p.direct.Kpad + 127) / 128) : 0);
        if (p.fused_ok) { b.gap0 = (long long)p.uf_gap; b.gap1 = (long long)p.uf_begin; }
        if (p.direct_ok) { b.gap2 = (long long)p.ud_gap; b.gap3 = (long long)p.ud_begin; }
        hipLaunchKernelGGL(filter_copies_kernel, dim3(b.end), dim3(256), 0, (hipStream_t)stream, d, src, p.fused, p.direct, b, w, U);
    } else if (p.split_ok) {
        hipLaunchKernelGGL(filter_transform_split_kernel, dim3((d.rows_total + kFtRows - 1) / kFtRows, d.Kpad / kFtK), dim3(256), 0,
                           (hipStream_t)stream, d, src, w, U, reinterpret_cast<uint32_t*>(U + p.us_begin));
    } else {
        hipLaunchKernelGGL(filter_transform_kernel, dim3((d.rows_total + 255) / 256, d.Kpad), dim3(256), 0,
                           (hipStream_t)stream, d, src, w, U);
    }
    return check_launch();
}

dwm_status_t launch_filter_batch(const FilterBatchArgs& a, const float* w, float* U, void* stream)
{
    static_assert(sizeof(FilterBatchArgs) <= 4000, "kernel arguments");
    const int gx = (a.max_rows + 255) / 256, nd = (a.direct_blocks + gx * a.Kpad - 1) / (gx * a.Kpad);
    hipLaunchKernelGGL(filter_transform_batch_kernel, dim3(gx, a.Kpad, a.nprob + nd), dim3(256), 0, (hipStream_t)stream, a, w, U);
    return check_launch();
}

dwm_status_t launch_filter_transform(const dwm_plan& p, const float* w, float* U, void* stream)
{
    const long long rs = (long long)p.d.R * p.d.S;
    return launch_filter_transform_from(p, FilterSource{0, rs * p.d.C, rs, p.d.S, 1}, w, U, stream);
}

// variants: 0/1 = gather form (blocks-fast / rows-fast), 2/3 = LDS-staged form (channel groups
// fastest / blocks fastest); planner's choice: LDS-staged where it applies
static int input_variant(const dwm_plan& p)
{
    const DevPlan& d = p.d;
    if (p.variant_input >= 0) return p.variant_input;
    return p.inlds_ok ? 2 : ((size_t)d.N * d.C * d.H * d.W * sizeof(float) > ((size_t)64 << 20));
}

bool input_zeroes_tail(const dwm_plan& p) { return input_variant(p) >= 2; }

static dwm_status_t launch_input(const dwm_plan& p, const float* x, float* V, void* stream, bool zero_tail)
{
    const DevPlan& d = p.d;
    const int nb = d.Tpad / 64, nr = d.rows_total / 16;
    dim3 block(256);
    const int variant = input_variant(p);
    if (variant >= 2) {
        if (!p.inlds_ok) return DWM_ERR_INVALID_ARG;
        InLdsArgs a = p.inlds;
        int parts = 0, planes = 0;  // planes: summed over the parts
        for (int i = 0; i < d.ncls; ++i) {
            parts += d.cls[i].hn * d.cls[i].wn;
            planes += d.cls[i].hn * d.cls[i].wn * (d.cls[i].lh + 1) * (d.cls[i].lw + 1);
        }
        auto kernel = zero_tail ? input_transform_lds_kernel<false, true> : input_transform_lds_kernel<false, false>;
        // A channel a workgroup, where there is a part for every wave and workgroups of four channels would leave half the CUs
        // without one, or three in eight where a part has ten planes and more: of 900 layers with up to 256 of them the 850
        // that this takes go at 0.5 to 1.03 times, the others at 0.8 to 1.5 (2x2 at stride 3, 144 channels, 25 images of
        // 23x22, 252 workgroups: 8.1 -> 12.0 us; others' waves hide a wave's chain there).
        const long long wgs = (long long)((d.T + 63) / 64) * a.ncg;
        if (p.variant_input < 0 && a.cg == 4 && parts >= 4 && wgs * 8 <= kNumCUs * (planes >= 10 * parts ? 5 : 4)) {
            a.cg = 1;
            a.ncg = d.C;
            a.lds_bytes = (size_t)a.chan_floats * sizeof(float);
            kernel = zero_tail ? input_transform_lds_kernel<true, true> : input_transform_lds_kernel<true, false>;
        }
        if (a.lds_bytes > 64 * 1024) {
            // (a single channel's region is at most 64 KB: only the form of several needs more)
            static const hipError_t attr0 = hipFuncSetAttribute(reinterpret_cast<const void*>(input_transform_lds_kernel<false, false>),
                                                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
            static const hipError_t attr1 = hipFuncSetAttribute(reinterpret_cast<const void*>(input_transform_lds_kernel<false, true>),
                                                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
            if (attr0 != hipSuccess || attr1 != hipSuccess) return DWM_ERR_HIP;
        }
        hipLaunchKernelGGL(kernel, dim3((unsigned)(nb * a.ncg)), block, a.lds_bytes, (hipStream_t)stream, d, a, x, V,
                           p.sk_counters(V), p.active().n_sk_tiles, variant == 2, p.skip_pad_rows ? 0 : 1);
        return check_launch();
    }
    int rows_fast = variant;
    if ((rows_fast ? nb : nr) > 65535) rows_fast = !rows_fast;
    if ((rows_fast ? nb : nr) > 65535) return DWM_ERR_UNSUPPORTED;
    dim3 grid(rows_fast ? nr : nb, rows_fast ? nb : nr);
    hipLaunchKernelGGL(input_transform_kernel, grid, block, 0, (hipStream_t)stream, d, x, V, p.sk_counters(V),
                       p.active().n_sk_tiles, rows_fast);
    return check_launch();
}

dwm_status_t launch_input_transform(const dwm_plan& p, const float* x, float* V, void* stream)
{
    return launch_input(p, x, V, stream, false);
}

dwm_status_t launch_input_transform_zero_tail(const dwm_plan& p, const float* x, float* V, void* stream)
{
    return launch_input(p, x, V, stream, true);
}

}  // namespace dwm
