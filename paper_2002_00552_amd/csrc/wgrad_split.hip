// The GEMM over the tiles of the filter gradient (wgrad.hip, steps 2 and 3) on the bfloat16 matrix cores:
//     dU[k][l] = sum_t dM[k][t] * V[l][t]   per plane,   dM = A dY A^T,
// with every binary32 operand the sum of three bfloat16 numbers and six products per product, in two
// accumulators: contract_split.hip has the arithmetic, its error and why.  dM is written split (nobody else reads it,
// and it is the smaller operand: planes x K against planes x parts x C rows), V stays binary32 and is split in
// registers by the wave that multiplies it.  Both are split as 2^16 times what they are, which every binary32 number's
// parts can hold (split.hpp), and the sums are multiplied by 2^-32, all of it exact; sums of 2^96 and more are computed again
// on fp32 MFMAs.  (V's multiplications take 2 % of the kernel on the layer below, wherever they stand among the terms.)
//
// There is nothing to fold here, so a wave's registers hold a 64x64 tile (two waves per SIMD), which needs half the
// LDS reads per MFMA of the forward contraction's 64x32: per 16 tiles a wave reads 6 KB of dM and 4 KB of V for 24
// MFMAs (768 cycles).  Workgroup 2x2 waves, 128 filters x 128 rows; chunks of 16 tiles through a ring of four LDS
// stages, two workgroups per CU.  Measured: 7x7 256->256 28x28 N=32 (400 tiles, three ranges) 600 -> 462 us, 178 TFLOP/s
// of the gradient's multiplications (1.07 PFLOP/s of bfloat16); the ring's loads two chunks ahead instead of one: 505 -> 480,
// neighbouring tiles on one XCD: 490 -> 475.  A row of V is 64 bytes of a chunk: its four 16-byte groups are XOR-swizzled by the
// row so that eight lanes' reads fall on different banks.
#include <hip/hip_runtime.h>

#include "dma.hpp"
#include "split.hpp"
#include "wgrad.hpp"

namespace dwm {

// ---------------------------------------------------------------------------------
// DMS[block of 64 tiles][distinct plane][t/16][part h,m,l][(t/8)%2][k][t%8], t inside the block: the parts of dM * 2^16.  A workgroup takes 64 filters,
// 32 tiles and up to kDyPlanes planes.  dy comes in along the tiles (a wave's load: one filter, 32 tiles' two pixel rows,
// 256 contiguous bytes each) and goes out along the filters (64 of them, 1 KB contiguous), through LDS; reading it with a
// thread per filter, 64 bytes a lane, took 96 us where this takes 80 (256 filters, 6272 tiles, 36 planes: 347 MB written; 46 us for the 16 distinct ones).
// ---------------------------------------------------------------------------------
constexpr int kDyPlanes = 16;
__global__ __launch_bounds__(256) void wgrad_dy_split_kernel(DyShape P, PlaneTable PT, const float* __restrict__ dy,
                                                             unsigned char* __restrict__ DMS)
{
    constexpr int ROW = 132;  // floats per filter: 2 pixel rows x 32 tiles x 2, and four that spread the banks
    __shared__ __attribute__((aligned(16))) float px[64 * ROW];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int k0 = blockIdx.y * 64;
    {
        const int t = blockIdx.x * 32 + (lane & 31), a = lane >> 5, tiles = P.TH * P.TW;
        const int n = t / tiles, ty = (t - n * tiles) / P.TW, tx = t - n * tiles - ty * P.TW;
        // filters k >= K and tiles t >= T are zeros: the GEMM multiplies them
        const bool ok = t < P.T && 2 * ty + a < P.OH, c1 = 2 * tx + 1 < P.OW;
        const float* yp = dy + (((size_t)n * P.K + k0 + wave * 16) * P.OH + 2 * ty + a) * P.OW + 2 * tx;
        const size_t kstep = (size_t)P.OH * P.OW;
        const bool pair_ok = (P.OW & 1) == 0 && (P.OH & 1) == 0 && (reinterpret_cast<uintptr_t>(dy) & 7) == 0;
        float2 v[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            v[j] = make_float2(0.f, 0.f);
            if (ok && k0 + wave * 16 + j < P.K) {
                if (pair_ok) {
                    v[j] = *reinterpret_cast<const float2*>(yp + j * kstep);
                } else {
                    v[j].x = yp[j * kstep];
                    if (c1) v[j].y = yp[j * kstep + 1];
                }
            }
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) *reinterpret_cast<float2*>(px + (wave * 16 + j) * ROW + a * 64 + (lane & 31) * 2) = v[j];
    }
    __syncthreads();
    const int tg = blockIdx.x * 4 + wave;  // group of eight tiles
    const int k = k0 + lane;
    float g[4][8];  // [2a + b][tile]
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 q = *reinterpret_cast<const float4*>(px + lane * ROW + a * 64 + wave * 16 + i * 4);
            g[2 * a][2 * i] = q.x; g[2 * a + 1][2 * i] = q.y; g[2 * a][2 * i + 1] = q.z; g[2 * a + 1][2 * i + 1] = q.w;
        }
    const size_t piece = (size_t)P.Kp * 16;  // bytes of one (part, half)
    unsigned char* out = DMS + (size_t)(tg >> 3) * PT.n * (24 * piece) + (size_t)((tg & 7) >> 1) * (6 * piece) +
                         (size_t)(tg & 1) * piece + (size_t)k * 16;
    const int p1 = min((int)(blockIdx.z + 1) * kDyPlanes, PT.n);
    out += (size_t)blockIdx.z * kDyPlanes * 24 * piece;
    for (int p = blockIdx.z * kDyPlanes; p < p1; ++p, out += 24 * piece) {
        const int coef = PT.e[p].coef;
        float s[4], m[8];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int cq = (coef >> (2 * q)) & 3;
            s[q] = cq == 1 ? kSplitScale : cq == 3 ? -kSplitScale : 0.f;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            m[i] = 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (s[q] != 0.f) m[i] = fmaf(s[q], g[q][i], m[i]);
        }
        bf16x8 f[3];
        split8(m, f);
#pragma unroll
        for (int x = 0; x < 3; ++x)
            *reinterpret_cast<puint4*>(out + (size_t)x * 2 * piece) = __builtin_bit_cast(puint4, f[x]);
    }
}

// ---------------------------------------------------------------------------------
// partial dU of one 128x128 tile of one plane over one range of tile blocks
// ---------------------------------------------------------------------------------
constexpr int kWsplitStages = 4;
__global__ __launch_bounds__(256, 2) void wgrad_split_kernel(WgradArgs A, DyShape P, const float* __restrict__ dy,
                                                             const unsigned char* __restrict__ DMS,
                                                             const float* __restrict__ V, float* __restrict__ partial)
{
    constexpr int NS = kWsplitStages, KT = kWsplitTile, LT = kWsplitTile;
    constexpr int A_STAGE = 6 * KT * 16, B_STAGE = LT * 64, STAGE = A_STAGE + B_STAGE;
    constexpr int NA = A_STAGE / 1024 / 4, NB = B_STAGE / 1024 / 4, N_DMA = NA + NB;
    static_assert(NS >= 3 && NS * STAGE <= 80 * 1024, "two workgroups per CU");

    extern __shared__ __attribute__((aligned(1024))) unsigned char smem_w[];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int wave_m = wave >> 1, wave_n = wave & 1;
    const int li = lane & 31, lh = lane >> 5;
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem_w;

    // Which output tile, which range of blocks.  Workgroups are dealt round-robin to the 8 XCDs: each gets a run of
    // neighbouring tiles (those of a few planes), which share their rows of dM and of V in its L2.
    const int total = A.n_tiles * A.splits, per_xcd = (total + 7) >> 3;
    const int pos = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((blockIdx.x >> 3) >= per_xcd || pos >= total) return;
    const int tile = pos % A.n_tiles, split = pos / A.n_tiles;
    int p = 0;
    while (p + 1 < A.n_planes && tile >= A.tile0[p + 1]) ++p;
    const int r = tile - A.tile0[p];
    const int kt = r / A.nlt[p], lt = r - kt * A.nlt[p];
    const int c0 = split * A.chunks_per_split, c1 = min(c0 + A.chunks_per_split, A.tblocks);
    const int nit = 4 * (c1 - c0);  // chunks of 16 tiles

    // This wave's DMA instructions: 64 filters of one (part, half), or 16 rows of V (64 bytes each, four lanes a row)
    const uint32_t piece = (uint32_t)A.Kp * 16u;
    uint32_t aoff[NA], boff[NB];
#pragma unroll
    for (int d = 0; d < NA; ++d) {
        const int id = wave * NA + d;
        aoff[d] = (uint32_t)(id >> 1) * piece + (uint32_t)((id & 1) * 64 + lane) * 16u;
    }
#pragma unroll
    for (int d = 0; d < NB; ++d) {
        const int row = (wave * NB + d) * 16 + (lane >> 2);
        boff[d] = (uint32_t)(row * 256 + (((lane & 3) ^ ((row >> 1) & 3)) << 4));
    }
    const int dmp = A.dmp[p];
    const unsigned char* sa = DMS + ((size_t)c0 * A.n_dm + (dmp & 255)) * (24 * (size_t)piece) + (size_t)(kt * KT) * 16;
    const float* sb = V + ((size_t)c0 * A.vblock_rows + A.vrow[p] + lt * LT) * 64;
    // from the last chunk of a block to the first of the next
    const size_t a_block = (size_t)(A.n_dm - 1) * 24 * piece + 6 * (size_t)piece;
    const size_t b_block = (size_t)A.vblock_rows * 64 - 48;
    int ileft = nit, iq = 0;
    auto issue_one = [&](int d, uint32_t ls) {
        if (d < NA) dma16s(reinterpret_cast<const float*>(sa), aoff[d], ls + (uint32_t)(wave * NA + d) * 1024);
        else dma16s(sb, boff[d - NA], ls + (uint32_t)(A_STAGE + (wave * NB + d - NA) * 1024));
    };
    auto advance_issue = [&]() {  // past the last chunk: that chunk is loaded again into free stages
        if (--ileft > 0) {
            iq = (iq + 1) & 3;
            sa += iq == 0 ? a_block : 6 * (size_t)piece;
            sb += iq == 0 ? b_block : 16;
        }
    };
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) {
#pragma unroll
        for (int d = 0; d < N_DMA; ++d) issue_one(d, lds0 + s * STAGE);
        advance_issue();
    }

    floatx16 acc[2][2][2];  // [row block][column block][h*h terms, the others]
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i >> 2][(i >> 1) & 1][i & 1][e] = 0.f;
    // the lane's fragments inside a stage: filter wave_m*64 + mi*32 + li; row wave_n*64 + nj*32 + li, tiles 8*lh .. +7
    const uint32_t a_lane = (uint32_t)(lh * KT + wave_m * 64 + li) * 16u;
    const int brow = wave_n * 64 + li, swz = (brow >> 1) & 3;  // (32 rows on: the same swizzle)
    const uint32_t b_lane0 = (uint32_t)(A_STAGE + brow * 64 + (((2 * lh) ^ swz) << 4));
    const uint32_t b_lane1 = (uint32_t)(A_STAGE + brow * 64 + (((2 * lh + 1) ^ swz) << 4));
    bf16x8 af[2][3], bf[2][3];
    auto read_a = [&](const unsigned char* st, int s) {
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
            af[mi][s] = *reinterpret_cast<const bf16x8*>(st + a_lane + (s * 2 * KT + mi * 32) * 16);
    };
    auto read_b = [&](const unsigned char* st, float (&v)[2][8]) {
#pragma unroll
        for (int nj = 0; nj < 2; ++nj) {
            *reinterpret_cast<float4*>(v[nj]) = *reinterpret_cast<const float4*>(st + b_lane0 + nj * 2048);
            *reinterpret_cast<float4*>(v[nj] + 4) = *reinterpret_cast<const float4*>(st + b_lane1 + nj * 2048);
        }
    };
    auto split_b = [&](const float (&v)[2][8], int nj, int i, uint32_t (&w)[2][3][4]) {
        split2(v[nj][2 * i] * kSplitScale, v[nj][2 * i + 1] * kSplitScale, w[nj][0][i], w[nj][1][i], w[nj][2][i]);
    };
    auto put_b = [&](const uint32_t (&w)[2][3][4], int nj, int s) {
        bf[nj][s] = __builtin_bit_cast(bf16x8, puint4{w[nj][s][0], w[nj][s][1], w[nj][s][2], w[nj][s][3]});
    };
    auto term = [&](int ta, int tb) {
        const int c = ta + tb > 0;
#pragma unroll
        for (int nj = 0; nj < 2; ++nj)
#pragma unroll
            for (int mi = 0; mi < 2; ++mi)
                acc[mi][nj][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[mi][ta], bf[nj][tb], acc[mi][nj][c], 0, 0, 0);
    };
    wait_vmcnt<(NS - 2) * N_DMA>();
    __syncthreads();
    {
        float v[2][8];
        uint32_t w[2][3][4];
        read_b(smem_w, v);
#pragma unroll
        for (int s = 0; s < 3; ++s) read_a(smem_w, s);
#pragma unroll
        for (int i = 0; i < 8; ++i) split_b(v, i >> 2, i & 3, w);
#pragma unroll
        for (int i = 0; i < 6; ++i) put_b(w, i & 1, i >> 1);
    }
    uint32_t next = STAGE, refill = (NS - 1) * STAGE;  // offsets of the next chunk's stage and of the one that is free
    // The chunk's operands are in registers; those of the next one are read and split beside its MFMAs, the barrier and
    // the refill sit between the terms: the order is contract_split.hip's, kept by sched_barrier.
#pragma unroll 1
    for (int it = 0; it < nit; ++it) {
        float v[2][8];
        uint32_t w[2][3][4];
        const unsigned char* st = smem_w + next;
        const uint32_t ls = lds0 + refill;
        term(2, 0);
        term(1, 0);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NS - 3) * N_DMA) : "memory");
        read_b(st, v);
        read_a(st, 2);
        __builtin_amdgcn_sched_barrier(0);
        issue_one(0, ls);
        __builtin_amdgcn_sched_barrier(0);
        term(1, 1);
        read_a(st, 1);
        __builtin_amdgcn_sched_barrier(0);
        issue_one(1, ls);
        __builtin_amdgcn_sched_barrier(0);
        term(0, 1);
#pragma unroll
        for (int i = 0; i < 3; ++i) split_b(v, 0, i, w);
        interleave<4, 10>();
        __builtin_amdgcn_sched_barrier(0);
        issue_one(2, ls);
        __builtin_amdgcn_sched_barrier(0);
        term(0, 2);
        split_b(v, 0, 3, w);
#pragma unroll
        for (int i = 0; i < 2; ++i) split_b(v, 1, i, w);
        interleave<4, 10>();
        __builtin_amdgcn_sched_barrier(0);
        issue_one(3, ls);
        __builtin_amdgcn_sched_barrier(0);
        term(0, 0);
#pragma unroll
        for (int i = 2; i < 4; ++i) split_b(v, 1, i, w);
        interleave<4, 7>();
        read_a(st, 0);
#pragma unroll
        for (int nj = 0; nj < 2; ++nj)
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                put_b(w, nj, s);
                asm volatile("" : "+v"(bf[nj][s]));  // made here, not sunk to where it is used
            }
        __builtin_amdgcn_sched_barrier(0);
        issue_one(4, ls);
        static_assert(N_DMA == 5, "the refill's instructions are spelled out");
        advance_issue();
        refill = next == 0 ? (NS - 1) * STAGE : next - STAGE;
        next = next == (NS - 1) * STAGE ? 0 : next + STAGE;
    }
    wait_vmcnt<0>();

    // lane holds column l and rows k = 8*(e/4) + 4*lh + e%4 of each 32x32 block
    const int Lp = A.lstride[p], lcol = lt * LT + wave_n * 64 + li;
    float* out = partial + (size_t)split * A.split_floats + (size_t)A.poff64[p] * 64 +
                 (size_t)(kt * KT + wave_m * 64) * Lp + lcol;
    const int lreal = A.lreal[p];
#pragma unroll
    for (int nj = 0; nj < 2; ++nj) {
        float s = 0.f;
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                acc[mi][nj][0][e] += acc[mi][nj][1][e];
                s = fmaf(acc[mi][nj][0][e], 0.f, s);
            }
        float factor = (dmp & 256 ? -1.f : 1.f) / (kSplitScale * kSplitScale);
        // operands the split cannot carry (infinities, NaN, from about 2^112 on) and scaled sums past the range: again
        // on fp32 MFMAs, dM from dy (columns past the class's rows hold what the workspace held)
        if (__builtin_amdgcn_ballot_w64(s != 0.f && lcol + nj * 32 < lreal) != 0) {
            const int coef = (dmp >> 16) & 255, tiles = P.TH * P.TW;
#pragma unroll
            for (int mi = 0; mi < 2; ++mi) {
                const int k = kt * KT + wave_m * 64 + mi * 32 + li;
                floatx16 m;
#pragma unroll
                for (int e = 0; e < 16; ++e) m[e] = 0.f;
#pragma unroll 1
                for (int t0 = c0 * 64; t0 < c1 * 64; t0 += 2) {
                    const int t = t0 + lh;
                    float a = 0.f, b = 0.f;
                    if (t < P.T) {
                        b = V[((size_t)(t >> 6) * A.vblock_rows + A.vrow[p] + lcol + nj * 32) * 64 + (t & 63)];
                        if (k < P.K) {
                            const int n = t / tiles, ty = (t - n * tiles) / P.TW, tx = t - n * tiles - ty * P.TW;
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                const int cq = (coef >> (2 * q)) & 3, oh = 2 * ty + (q >> 1), ow = 2 * tx + (q & 1);
                                if (cq != 0 && oh < P.OH && ow < P.OW) {
                                    const float g = dy[(((size_t)n * P.K + k) * P.OH + oh) * P.OW + ow];
                                    a += cq == 1 ? g : -g;
                                }
                            }
                        }
                    }
                    m = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, m, 0, 0, 0);
                }
                acc[mi][nj][0] = m;
            }
            factor = 1.f;  // (the pattern was the plane's own)
        }
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                out[(size_t)(mi * 32 + 8 * (e >> 2) + 4 * lh + (e & 3)) * Lp + nj * 32] = acc[mi][nj][0][e] * factor;
    }
}

dwm_status_t launch_wgrad_split(const WgradArgs& a, const DyShape& ds, const PlaneTable& dm_table, const float* dy,
                                const float* V, unsigned char* dm, float* partial, hipStream_t stream)
{
    constexpr int lds_bytes = kWsplitStages * (6 * kWsplitTile * 16 + kWsplitTile * 64);
    auto kernel = wgrad_split_kernel;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (attr != hipSuccess || a.Kp % kWsplitTile != 0) return DWM_ERR_HIP;
    hipLaunchKernelGGL(wgrad_dy_split_kernel, dim3(a.tblocks * 2, a.Kp / 64, (dm_table.n + kDyPlanes - 1) / kDyPlanes), dim3(256), 0, stream, ds,
                       dm_table, dy, dm);
    hipLaunchKernelGGL(kernel, dim3((unsigned)((a.n_tiles * a.splits + 7) / 8 * 8)), dim3(256), lds_bytes, stream, a, ds, dy,
                       static_cast<const unsigned char*>(dm), V, partial);
    return hipGetLastError() == hipSuccess ? DWM_OK : DWM_ERR_HIP;
}

}  // namespace dwm
