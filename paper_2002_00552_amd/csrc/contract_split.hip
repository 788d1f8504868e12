// Contraction + output transform + aggregation (paper Sec. 4.1 "Calculation", "Detransformation",
// "Aggregation") in single precision on the bfloat16 matrix cores.
//
// What it computes, how the tiles are shared out and how the planes are folded into the 2x2 outputs is
// contract.hip's; what differs is the multiplication.  An fp32 MFMA runs at the vector rate (157 TFLOP/s)
// and keeps the vector unit busy while it does; a bfloat16 MFMA takes a sixteenth of the cycles and leaves
// the vector unit free.  Every binary32 operand is therefore written as the sum of three bfloat16 numbers,
//     x = h + m + l,   h = rn(x), m = rn(x - h), l = x - h - m   (8 + 8 + 8 significant bits: l is exact),
// and a product is the six terms h*h, h*m, m*h, m*m, h*l, l*h, each exact in the matrix core's binary32
// accumulation; what is left out (m*l, l*m, l*l) is at most 2^-24 of the product and of either sign.
// Measured over sums of 128 to 1024 products (random signs, one-sided, spread over twelve binades): the
// error against 64 bits is 0.65 to 0.9 of the fp32 MFMA's, because sixteen products are added per
// rounding instead of two.  Six MFMAs of 32x32x16 take 192 cycles where eight of 32x32x2 take 512.
//
// The h*h terms and the other five are summed in accumulators of their own, which leaves one large
// rounding per sixteen products: against 64 bits, whole layers come out 1.6 to 3 times closer than from
// contract.hip (7x7 over 256 channels 4.1e-7 -> 2.6e-7, 3x3 over 256 channels 4.3e-7 -> 1.6e-7).
//
// U is split once, by the filter transform (transforms.hip; a copy beside the fp32 one, laid out so that a lane's
// fragment is 16 bytes and a DMA instruction's source is 1 KB contiguous):
//     US[plane][l/16][part h,m,l][(l/8)%2][k][l%8].
// V stays binary32 in memory and in LDS and is split by the lane that multiplies it, in registers
// (6.5 vector instructions an element): V is the larger traffic, and a split V would be half again as much.
//
// What bounds it, measured on the 7x7 layer with 256 channels (28x28, N = 32; 480 us = 171 TFLOP/s of the
// layer's multiplications, 1.03 PFLOP/s of bfloat16; contract.hip 650 to 700 us): with one thing compiled out at a
// time, at 500 us, all loads 370 us, V's misses 440, V's split 455; a loop of the same instructions over data in L2
// reaches 0.26 PFLOP/s x 6, held by the chip's power (the clock falls to 1.8 GHz).  Tried and no faster:
// 128x128 tiles with eight waves (518) or with four of 128x32 (570: one wave per SIMD hides nothing), V split
// once per workgroup through LDS (540), operands requested a chunk later (531), each against 475 to 500.
//
// Small operands: V is split as V * 2^16 and the fold multiplies by 2^-16, both exact, so that a V of any size is the
// sum of its parts (split.hpp).  U's copy is the parts of U as it is; where those are not U (0 < |U| < 2^-110) the filter
// transform writes NaN for them.  (V's multiplications take 0.4 % of the call on the 7x7 layer below, standing where the
// vector unit would wait for the first terms, and 1 to 2 % on small layers, wherever they stand.)
// Values the split cannot carry: those, an infinity or NaN (inf - inf), and |V| >= 2^112 - 2^103 or |U| >= 2^128 - 2^119, whose h
// becomes infinite.  Any of them, and an output of 2^112 or more before the fold, makes an output of the tile
// non-finite; a wave that finds one among its outputs computes its part of the tile again with fp32 MFMAs from the fp32
// operands (exact_segment), so such inputs give what contract.hip gives.
#include <hip/hip_runtime.h>

#include "dma.hpp"
#include "plan.hpp"
#include "split.hpp"

namespace dwm {

constexpr int kSplitFold = 1024;  // steps summed before a fold

struct SplitArgs {
    int K, T, Kpad;
    int OH, OW, TH, TW;
    int vblock;  // floats of one 64-tile block of V
    ContractGeometry g;
};

// tile index -> (kt, tt): the K tiles of one T tile on consecutive slots of one XCD (see contract.hip)
__device__ __forceinline__ void tile_coords(const ContractGeometry& G, int tile, int& kt, int& tt)
{
    const bool low = tile < G.full8;
    const int r0 = low ? tile >> 3 : tile - G.full8;
    kt = r0 % G.nkt;
    tt = low ? (r0 / G.nkt) * 8 + (tile & 7) : (G.ntt / 8) * 8 + r0 / G.nkt;
}

// the 2x2 outputs of filter k and tile t
__device__ __forceinline__ void put_tile(const SplitArgs& A, float* __restrict__ y, int t, int k, float y00, float y01,
                                         float y10, float y11)
{
    if (k >= A.K) return;
    const int tiles = A.TH * A.TW;
    const int n = t / tiles, rem = t - n * tiles;
    const int ty = rem / A.TW, tx = rem - ty * A.TW;
    const int oh = 2 * ty, ow = 2 * tx;
    float* yp = y + (((size_t)n * A.K + k) * A.OH + oh) * A.OW + ow;
    if ((A.OW & 1) == 0) {
        *reinterpret_cast<float2*>(yp) = make_float2(y00, y01);
        if (oh + 1 < A.OH) *reinterpret_cast<float2*>(yp + A.OW) = make_float2(y10, y11);
    } else {
        yp[0] = y00;
        if (ow + 1 < A.OW) yp[1] = y01;
        if (oh + 1 < A.OH) {
            yp[A.OW] = y10;
            if (ow + 1 < A.OW) yp[A.OW + 1] = y11;
        }
    }
}

__device__ __forceinline__ int lane_again()
{
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}

// Workgroup of WGM x WGN waves, wave tile 32*WM filters x 32 tiles, a ring of NS stages of LC = 16 reduction steps.
template <int WGM, int WGN, int WM, int NS>
__global__ __launch_bounds__(64 * WGM * WGN, WM > 1 ? 2 : 3) void contract_split_kernel(
    SplitArgs A, PlaneTable PT, const float* __restrict__ U, const unsigned char* __restrict__ US,
    const float* __restrict__ V, float* __restrict__ y, float* __restrict__ partial)
{
    constexpr int NW = WGM * WGN, NT = 64 * NW, LC = kSplitChunk;
    constexpr int KT = 32 * WM * WGM, TT = 32 * WGN;
    constexpr int U_STAGE = 6 * KT * 16, V_STAGE = LC * TT * 4, STAGE = U_STAGE + V_STAGE;
    // DMA instructions per wave and chunk (where U's do not split evenly, some pieces are loaded twice: a wave's count
    // of outstanding loads is the same for all)
    constexpr int NU = (U_STAGE / 1024 + NW - 1) / NW, NV = V_STAGE / 1024 / NW, N_DMA = NU + NV;
    static_assert(NV * NW * 1024 == V_STAGE, "V's DMA must split evenly over the waves");
    static_assert(KT % 64 == 0 && TT % 64 == 0 && NS >= 4 && (NS - 2) * N_DMA < 64, "ring");

    extern __shared__ __attribute__((aligned(1024))) unsigned char smem_s[];  // NS * STAGE bytes

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int wave_m = wave / WGN, wave_n = wave % WGN;
    const int li = lane & 31, lh = lane >> 5;
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem_s;
    const ContractGeometry& G = A.g;

    // This wave's DMA instructions of a chunk: the lane's byte offset from the chunk's base.  64 filters of one
    // (part, row group) of US, or four rows of 64 tiles of V: 1 KB each.
    uint32_t uoff[NU], udst[NU], voff[NV];
#pragma unroll
    for (int d = 0; d < NU; ++d) {
        const int id = (wave * NU + d) % (U_STAGE / 1024), piece = id / (KT / 64), part = id % (KT / 64);
        uoff[d] = (uint32_t)(piece * A.Kpad + part * 64 + lane) * 16u;
        udst[d] = (uint32_t)id * 1024u;
    }
#pragma unroll
    for (int d = 0; d < NV; ++d) {
        const int id = wave * NV + d, blk = id / (LC / 4), rr = id % (LC / 4);
        voff[d] = (uint32_t)(blk * A.vblock) * 4u + (uint32_t)(rr * 1024 + lane * 16);
    }
    // the lane's fragments inside a stage
    const uint32_t a_lane = (uint32_t)(lh * KT + wave_m * 32 * WM + li) * 16u;
    const int bcol = wave_n * 32 + li;
    const uint32_t b_lane = (uint32_t)(U_STAGE + (bcol >> 6) * LC * 256 + lh * 2048 + (bcol & 63) * 4);

    // Two accumulators a block: the h*h terms and the other five, a 256th of them.  Summed apart, the small terms'
    // roundings vanish against those of the large ones, of which there is one per sixteen products.
    floatx16 acc[WM][2];
    floatx16 Y[WM][4];

    auto fold_into = [&](floatx16 (&yb)[4], const floatx16& ab, int coef, float one) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int cq = (coef >> (2 * q)) & 3;
            if (cq != 0) {
                const float sg = cq == 1 ? one : -one;
#pragma unroll
                for (int e = 0; e < 16; ++e) yb[q][e] = fmaf(sg, ab[e], yb[q][e]);
            }
        }
    };

    // ---- one segment: iterations [it0, it0+nit) of tile (kt, tt); result in Y ----
    auto run_segment = [&](int kt, int tt, int it0, int nit) {
#pragma unroll
        for (int mi = 0; mi < WM; ++mi) {
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[mi][0][e] = acc[mi][1][e] = 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e = 0; e < 16; ++e) Y[mi][q][e] = 0.f;
        }
        // plane and chunk of the first iteration
        int p = 0, j = it0;
        int nch = PT.e[0].Lpad / LC;
        while (j >= nch) {
            j -= nch;
            ++p;
            nch = PT.e[p].Lpad / LC;
        }
        // Issue cursor: the chunk whose loads go out next, and how many chunks are left until it has to be pointed
        // elsewhere: at the next plane, or, past the segment's last chunk, nowhere (that chunk is loaded again into free
        // stages).
        int ip = p, ileft = nit, iuntil = min(nch - j, nit);
        const unsigned char* sa;
        const float* sb;
        uint32_t a_step = 6u * 16u * (uint32_t)A.Kpad, b_step = LC * 64;
        auto point_at = [&](int ch) {
            const DevPlaneEntry e = PT.e[ip];
            sa = US + (size_t)e.u_off64 * 384 + (size_t)ch * a_step + (size_t)(kt * KT) * 16;
            sb = V + (size_t)(tt * (TT / 64)) * A.vblock + ((size_t)e.v_off64 + ch * LC) * 64;
        };
        point_at(j);
        auto issue_one = [&](int d, uint32_t ls) {  // ls: LDS address of the stage
            if (d < NU) dma16s(reinterpret_cast<const float*>(sa), uoff[d], ls + udst[d]);
            else dma16s(sb, voff[d - NU], ls + (uint32_t)(U_STAGE + (wave * NV + d - NU) * 1024));
        };
        auto advance_issue = [&]() {
            sa += a_step;
            sb += b_step;
            --ileft;
            if (__builtin_expect(--iuntil == 0, 0)) {
                if (ileft <= 0) {
                    sa -= a_step;
                    sb -= b_step;
                    a_step = b_step = 0;
                    iuntil = 0x7fffffff;
                } else {
                    ++ip;
                    iuntil = min((int)PT.e[ip].Lpad / LC, ileft);
                    point_at(0);
                }
            }
        };
#pragma unroll
        for (int s = 0; s < NS - 1; ++s) {
#pragma unroll
            for (int d = 0; d < N_DMA; ++d) issue_one(d, lds0 + s * STAGE);
            advance_issue();
        }

        // The lane's operands of the chunk at hand are in registers.  While its MFMAs run, the wave reads those of the
        // next one (a part of A as soon as the terms that use it are done) and splits B's values.
        bf16x8 af[WM][3], bf[3];
        auto read_a = [&](const unsigned char* al, int s) {
#pragma unroll
            for (int mi = 0; mi < WM; ++mi)
                af[mi][s] = *reinterpret_cast<const bf16x8*>(al + (s * 2 * KT + mi * 32) * 16);
        };
        auto read_b = [&](const unsigned char* bl, float (&r)[8]) {
#pragma unroll
            for (int i = 0; i < 8; ++i) r[i] = *reinterpret_cast<const float*>(bl + i * 256);
        };
        auto split_b = [&](const float (&r)[8], int i, uint32_t (&w)[3][4]) {
            split2(r[2 * i], r[2 * i + 1], w[0][i], w[1][i], w[2][i]);
        };
        auto put_b = [&](const uint32_t (&w)[3][4], int s) {
            bf[s] = __builtin_bit_cast(bf16x8, puint4{w[s][0], w[s][1], w[s][2], w[s][3]});
        };
        auto term = [&](int ta, int tb) {
            const int c = ta + tb > 0;
#pragma unroll
            for (int mi = 0; mi < WM; ++mi)
                acc[mi][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[mi][ta], bf[tb], acc[mi][c], 0, 0, 0);
        };
        wait_vmcnt<(NS - 3) * N_DMA>();  // two chunks
        __syncthreads();
        {
            float r[8];
            uint32_t w[3][4];
            read_b(smem_s + b_lane, r);
#pragma unroll
            for (int s = 0; s < 3; ++s) read_a(smem_s + a_lane, s);
#pragma unroll
            for (int i = 0; i < 8; ++i) r[i] *= kSplitScale;
#pragma unroll
            for (int i = 0; i < 4; ++i) split_b(r, i, w);
#pragma unroll
            for (int s = 0; s < 3; ++s) put_b(w, s);
        }

        uint32_t next = STAGE, refill = (NS - 1) * STAGE;  // offsets of the next chunk's stage and of the one that is free
        auto chunk = [&]() {
            // The order below is kept (sched_barrier).  The next chunk landed before the last barrier: its reads start at
            // once and have the first terms' MFMAs to arrive behind.  The barrier, in the middle of the chunk, says that the
            // chunk after it has landed and that every wave is done with the one before this: that stage is refilled, a few
            // DMA instructions at a time between the terms (issued together they queue at the address unit and the matrix
            // core waits with the wave).
            float r[8];
            uint32_t w[3][4];
            const unsigned char* al = smem_s + next + a_lane;
            const uint32_t ls = lds0 + refill;
            read_b(smem_s + next + b_lane, r);
            __builtin_amdgcn_sched_barrier(0);
            term(2, 0);
            read_a(al, 2);
            __builtin_amdgcn_sched_barrier(0);
            term(1, 0);
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NS - 4) * N_DMA) : "memory");
#pragma unroll
            for (int d = 0; d < N_DMA / 4; ++d) issue_one(d, ls);
            __builtin_amdgcn_sched_barrier(0);
            term(1, 1);
#pragma unroll
            for (int i = 0; i < 8; ++i) r[i] *= kSplitScale;
            interleave<WM, 8 / WM>();
            read_a(al, 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int d = N_DMA / 4; d < 2 * N_DMA / 4; ++d) issue_one(d, ls);
            __builtin_amdgcn_sched_barrier(0);
            term(0, 1);
            split_b(r, 0, w);
            split_b(r, 1, w);
            interleave<WM, (22 + WM - 1) / WM>();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int d = 2 * N_DMA / 4; d < 3 * N_DMA / 4; ++d) issue_one(d, ls);
            __builtin_amdgcn_sched_barrier(0);
            term(0, 2);
            split_b(r, 2, w);
            split_b(r, 3, w);
            interleave<WM, (22 + WM - 1) / WM>();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int d = 3 * N_DMA / 4; d < N_DMA; ++d) issue_one(d, ls);
            __builtin_amdgcn_sched_barrier(0);
            term(0, 0);
            read_a(al, 0);
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                put_b(w, s);
                asm volatile("" : "+v"(bf[s]));  // made here, not sunk to where it is used
            }
            __builtin_amdgcn_sched_barrier(0);
            advance_issue();
            refill = next == 0 ? (NS - 1) * STAGE : next - STAGE;
            next = next == (NS - 1) * STAGE ? 0 : next + STAGE;
        };
        // A plane's chunks, kSplitFold steps at most, then a fold: the chunk loop is one straight piece of code with one branch
        // (unrolled over the ring, with the fold inside, its taken branches cost a third of the time).
        for (int left = nit; left > 0;) {
            const int n = min(left, min(nch - j, kSplitFold / LC));
#pragma unroll 1
            for (int c = 0; c < n; ++c) chunk();
            const int coef = PT.e[p].coef;
#pragma unroll
            for (int mi = 0; mi < WM; ++mi) {
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[mi][0][e] += acc[mi][1][e];
                fold_into(Y[mi], acc[mi][0], coef, 1.f / kSplitScale);
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[mi][0][e] = acc[mi][1][e] = 0.f;
            }
            left -= n;
            j += n;
            if (j == nch && left > 0) {
                ++p;
                j = 0;
                nch = PT.e[p].Lpad / LC;
            }
        }
        // every DMA write (the parked re-loads too) has landed and every wave is done reading
        // before the LDS ring is reused by the next segment or handed to another workgroup
        wait_vmcnt<0>();
        __syncthreads();
    };

    // Workgroups 0 .. n_full-1 own a whole tile; the others own piece g / n_sk_tiles of tile g % n_sk_tiles (equal
    // ranges of its iterations), so that workgroups launched together read the same part of U.
    const int b = blockIdx.x;
    const bool whole = b < G.n_full;
    const int g = b - G.n_full;
    const int trel = whole ? b : g % G.n_sk_tiles;
    const int piece = whole ? 0 : g / G.n_sk_tiles;
    const int it0 = piece * G.sk_ipw;
    const int nit = whole ? G.n_iter : min(G.sk_ipw, G.n_iter - it0);
    if (nit <= 0) return;
    int kt, tt;
    tile_coords(G, whole ? trel : G.n_full + trel, kt, tt);
    run_segment(kt, tt, it0, nit);

    // (the lane's place, kept beside the chunk loop's registers, would be spilled)
    const int ln = lane_again(), half = ln >> 5, col = wave_n * 32 + (ln & 31);

    // ---- the same segment on fp32 MFMAs, straight from memory: for operands the split cannot carry ----
    auto exact_segment = [&] {
        const float* vcol = V + (size_t)(tt * (TT / 64) + (col >> 6)) * A.vblock + (col & 63) + half * 8 * 64;
#pragma unroll
        for (int mi = 0; mi < WM; ++mi) {
            const size_t urow = (size_t)(kt * KT + (wave_m * WM + mi) * 32 + (ln & 31));
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e = 0; e < 16; ++e) Y[mi][q][e] = 0.f;
            int p = 0, left = nit, ch = it0;
#pragma unroll 1
            while (left > 0) {
                const DevPlaneEntry e = PT.e[p];
                const int n = e.Lpad / LC;
                if (ch >= n) {
                    ch -= n;
                    ++p;
                    continue;
                }
                const int take = min(left, min(n - ch, kFoldSteps / LC));
                const float* ua = U + (size_t)e.u_off64 * 64 + urow * e.Lpad + ch * LC + half * 8;
                const float* vb = vcol + ((size_t)e.v_off64 + ch * LC) * 64;
                floatx16 m;
#pragma unroll
                for (int i = 0; i < 16; ++i) m[i] = 0.f;
#pragma unroll 1
                for (int c = 0; c < take; ++c, ua += LC, vb += LC * 64) {  // (a chunk's loads together: 4.2 -> 1.35 ms for the whole 7x7 layer)
                    float a[8], v[8];
                    *reinterpret_cast<float4*>(a) = *reinterpret_cast<const float4*>(ua);
                    *reinterpret_cast<float4*>(a + 4) = *reinterpret_cast<const float4*>(ua + 4);
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = vb[i * 64];
#pragma unroll
                    for (int i = 0; i < 8; ++i) m = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], v[i], m, 0, 0, 0);
                }
                fold_into(Y[mi], m, e.coef, 1.f);
                left -= take;
                ch += take;
            }
        }
    };
    // (columns past the last tile hold whatever the workspace held)
    auto all_finite = [&] {
        float s = 0.f;
#pragma unroll
        for (int mi = 0; mi < WM; ++mi)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e = 0; e < 16; ++e) s = fmaf(Y[mi][q][e], 0.f, s);
        return __builtin_amdgcn_ballot_w64(s != 0.f && tt * TT + col < A.T) == 0;
    };

    if (!all_finite()) exact_segment();
    if (!whole) {
        // partial outputs [tile][piece][(block*4 + q)*4 + e/4][thread][4 floats]
        float* out = partial + ((size_t)trel * G.sk_f + piece) * (KT * TT * 4) + (wave * 64 + ln) * 4;
#pragma unroll
        for (int mi = 0; mi < WM; ++mi)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e4 = 0; e4 < 4; ++e4) {
                    const floatx16& v = Y[mi][q];
                    *reinterpret_cast<pfloat4*>(out + ((mi * 4 + q) * 4 + e4) * NT * 4) =
                        pfloat4{v[4 * e4], v[4 * e4 + 1], v[4 * e4 + 2], v[4 * e4 + 3]};
                }
        return;
    }
    // lane holds column t and rows k = 8*(e/4) + 4*half + e%4 of each block
    const int t = tt * TT + col;
    if (t >= A.T) return;
#pragma unroll
    for (int mi = 0; mi < WM; ++mi)
#pragma unroll
        for (int e = 0; e < 16; ++e)
            put_tile(A, y, t, kt * KT + (wave_m * WM + mi) * 32 + 8 * (e >> 2) + 4 * half + (e & 3), Y[mi][0][e],
                             Y[mi][1][e], Y[mi][2][e], Y[mi][3][e]);
}

// One row of a tile's 2x2 outputs (a = 0, 1), filter k.
__device__ __forceinline__ void put_row(const SplitArgs& A, float* __restrict__ y, int t, int k, int a, float y0, float y1)
{
    if (k >= A.K) return;
    const int tiles = A.TH * A.TW;
    const int n = t / tiles, rem = t - n * tiles;
    const int ty = rem / A.TW, tx = rem - ty * A.TW;
    const int oh = 2 * ty + a, ow = 2 * tx;
    if (oh >= A.OH) return;
    float* yp = y + (((size_t)n * A.K + k) * A.OH + oh) * A.OW + ow;
    if ((A.OW & 1) == 0) {
        *reinterpret_cast<float2*>(yp) = make_float2(y0, y1);
    } else {
        yp[0] = y0;
        if (ow + 1 < A.OW) yp[1] = y1;
    }
}

// The tiles that were cut into pieces: y = the sum of their partial outputs, in piece order.  A kernel of its own, so that
// the whole chip reads the partials, where the last workgroup to arrive (contract.hip's way) reads a tile's alone: 3x3 over
// 256 channels on one 14x14 image, cut into eight pieces, 38 -> 22 us for the contraction and this.  FEW: a wave per (tile,
// wave of the contraction, block of 32 filters, four of its sixteen rows, output row), eight pieces' loads in flight: that
// layer, now in sixteen pieces, 11.4 + 4.8 (6.5 in the other form, whose sixteen workgroups leave the chip idle).  Else a
// workgroup of the contraction's waves per (tile, block, four rows), both output rows a wave: 28 us for the 7x7 layer over
// 256 channels (196 tiles in five pieces; 34 in the first form).
template <int WGM, int WGN, int WM, bool FEW>
__global__ __launch_bounds__(FEW ? 64 : 64 * WGM * WGN) void split_sum_kernel(SplitArgs A, const float* __restrict__ partial,
                                                                              float* __restrict__ y)
{
    constexpr int NT = 64 * WGM * WGN, KT = 32 * WM * WGM, TT = 32 * WGN, STEP = KT * TT * 4, ROWS = FEW ? 1 : 2, AHEAD = FEW ? 8 : 1;
    const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
    const int trel = blockIdx.x, mi = (blockIdx.y >> 2) % WM, e4 = blockIdx.y & 3;
    const int wave = FEW ? (blockIdx.y >> 2) / WM : threadIdx.x >> 6, a0 = FEW ? blockIdx.z : 0;
    const int nc = (A.g.n_iter + A.g.sk_ipw - 1) / A.g.sk_ipw;
    int kt, tt;
    tile_coords(A.g, A.g.n_full + trel, kt, tt);
    const float* src = partial + (size_t)trel * A.g.sk_f * STEP + (size_t)(mi * 16 + a0 * 8 + e4) * NT * 4 + (wave * 64 + lane) * 4;
    pfloat4 v[2 * ROWS];
#pragma unroll
    for (int b = 0; b < 2 * ROWS; ++b) v[b] = *reinterpret_cast<const pfloat4*>(src + b * 4 * NT * 4);
#pragma unroll AHEAD
    for (int c = 1; c < nc; ++c) {
        src += STEP;
#pragma unroll
        for (int b = 0; b < 2 * ROWS; ++b) v[b] += *reinterpret_cast<const pfloat4*>(src + b * 4 * NT * 4);
    }
    const int t = tt * TT + wave % WGN * 32 + li;
    if (t >= A.T) return;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int k = kt * KT + (wave / WGN * WM + mi) * 32 + 8 * e4 + 4 * lh + e;
        if constexpr (FEW) put_row(A, y, t, k, a0, v[0][e], v[1][e]);
        else put_tile(A, y, t, k, v[0][e], v[1][e], v[2][e], v[3][e]);
    }
}

// ---------------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------------
template <int WGM, int WGN, int WM, int NS>
static dwm_status_t launch_variant(const dwm_plan& p, const float* U, float* ws, float* y, void* stream)
{
    constexpr int KT = 32 * WM * WGM, TT = 32 * WGN;
    static_assert(kKAlign % KT == 0 && kTAlign % TT == 0, "padding must cover the tile");
    SplitArgs a;
    a.K = p.d.K; a.T = p.d.T; a.Kpad = p.d.Kpad;
    a.OH = p.d.OH; a.OW = p.d.OW; a.TH = p.d.TH; a.TW = p.d.TW;
    a.vblock = p.d.vblock_rows * 64;
    a.g = p.split;
    // the geometry was computed for exactly this shape of variant
    if (a.g.nkt != (p.d.K + KT - 1) / KT || a.g.ntt != (p.d.T + TT - 1) / TT) return DWM_ERR_INVALID_ARG;
    // outputs lie densely in y: a forward pass, or a data gradient at stride 1
    const OutMap& m = p.d.om;
    if (m.sy != 1 || m.sx != 1 || m.oy != 0 || m.ox != 0 || m.YH != p.d.OH || m.YW != p.d.OW) return DWM_ERR_INVALID_ARG;
    constexpr int lds_bytes = NS * (6 * KT * 16 + kSplitChunk * TT * 4);
    static_assert(lds_bytes <= (WM > 1 ? 80 : 53) * 1024, "LDS");
    auto kernel = contract_split_kernel<WGM, WGN, WM, NS>;
    if (lds_bytes > 64 * 1024) {
        static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (attr != hipSuccess) return DWM_ERR_HIP;
    }
    float* partial = p.sk_partial(ws);
    hipLaunchKernelGGL(kernel, dim3((unsigned)(a.g.n_full + a.g.sk_wgs)), dim3(64 * WGM * WGN), lds_bytes,
                       (hipStream_t)stream, a, p.planes, U, reinterpret_cast<const unsigned char*>(U + p.us_begin),
                       static_cast<const float*>(ws), y, partial);
    if (a.g.n_sk_tiles > 0) {
        const float* part = partial;
        if (a.g.n_sk_tiles * WM * 4 < kNumCUs / 2)
            hipLaunchKernelGGL((split_sum_kernel<WGM, WGN, WM, true>), dim3((unsigned)a.g.n_sk_tiles, WM * 4 * WGM * WGN, 2), dim3(64), 0,
                               (hipStream_t)stream, a, part, y);
        else
            hipLaunchKernelGGL((split_sum_kernel<WGM, WGN, WM, false>), dim3((unsigned)a.g.n_sk_tiles, WM * 4), dim3(64 * WGM * WGN), 0,
                               (hipStream_t)stream, a, part, y);
    }
    return hipGetLastError() == hipSuccess ? DWM_OK : DWM_ERR_HIP;
}

dwm_status_t launch_contract_split(const dwm_plan& p, const float* U, float* ws, float* y, void* stream)
{
    switch (p.split.variant) {
        case 0: return launch_variant<2, 2, 2, 5>(p, U, ws, y, stream);
        case 1: return launch_variant<2, 2, 1, 5>(p, U, ws, y, stream);
        default: return DWM_ERR_INVALID_ARG;
    }
}

}  // namespace dwm
