// Convolution without Winograd transforms, in single precision on the bfloat16 matrix cores: one launch from x to y.
//
// Why: a layer of few tiles spends its time on launches that wait for one another (input transforms -- one for each phase
// of a strided layer's data gradient --, contraction, sum of pieces), each with its own start, first loads and last stores.
// Six bfloat16 products of split operands (contract_split.hip) cost so little there that the taps of the plain convolution,
// 1.4 to 2.25 times the method's multiplications, are done before the transformed input were written.
//
// What it does: an implicit GEMM of [filters] x [taps, channels] x [output pixels].  x is staged a chunk of channels at a
// time in LDS, split into its three bfloat16 parts once per pixel and channel (6.5 vector instructions an element, shared by
// all the taps and filters that meet it), eight channels together, which is a lane's operand.  A tap is then an offset into
// the staged pixels.  The filter, split by direct_filter_kernel, goes from memory straight to registers, each part asked
// for again as soon as its last MFMA is issued.  Where tiles are few a workgroup's waves share a tile and take every
// wk-th step of it (WK), and add up their sums in LDS, in wave order; where that still leaves CUs idle, a tile's chunks are
// shared by up to 16 workgroups (blockIdx.y), each with outputs of its own that direct_sum_kernel adds in order: 3x3, 256 -> 256
// channels, one 14x14 image 23.8 us by the model in one piece, 11.7 measured in 16.
//
// Operands: x and w are split as x * 2^16 and w * 2^16, sums multiplied by 2^-32: exact at every scale up to 2^112.  What
// the parts cannot carry (|x| or |w| from about 2^112 on, infinities, NaN, sums from 2^96 on) makes outputs non-finite; the
// wave that finds one among its outputs computes them again on fp32 MFMAs, from x and an fp32 copy of the filter.
// 3x3, 128 -> 128 channels, 64 28x28 images: 93 us, with one infinity in x 192, NaN throughout 294 (one block of 32 x 32 at a
// time, each load waited for, 476 and 823); 3x3 at stride 2, 128 -> 256, 32 56x56 images 99, 289, 299 (556 and 700).
//
// Long sums (two_level, setup.cpp): where a wave adds up many steps in one accumulator, each step's rounding is one of the whole
// sum: with positive operands errors grew to three times those of the transforms (11x11 at stride 2, 214 filters of dy, 486 steps: 4.1e-7
// against 1.4e-7 in the 2-norm).  There all six products go to one accumulator, which is added to the other every eight steps:
// 1.1e-7; the same of dy of zero mean 4.9e-7 -> 2.3e-7 (transforms 4.8e-7); 11x11, 384 filters, 28x28 6.4e-7 -> 3.1e-7.  Time: 7x7 at
// stride 2, 256 channels, 256 14x14 images 468 -> 473 us, others within 1 %; folds every 4 steps 487 us and no better, every 16 as fast
// and less exact with operands of zero mean (each small product rounds at the first level's size, so that has to stay short).
//
// Bound by latency where the chip is not full (first loads, the barrier of each chunk), and where it is by CUs without a tile and by what
// does not run beside the MFMAs (a chunk's first loads and splitting, between barriers): at 2.2 GHz MFMAs are busy for 0.40 of all cycles and
// CUs for 0.66 of 3x3 at stride 2, 128 -> 256 channels, 32 56x56 images (196 tiles), 0.44 and 0.71 of 3x3, 128 -> 128, 64 28x28 images (392
// tiles of half the size), 0.44 and 0.59 of the gradient of 7x7 at stride 2, 256 channels, 256 14x14 images.  As a
// data gradient, before -> now: 5x5 at stride 2, 67 -> 93 channels, five 35x29 images, the training step 111 -> 101 us; drawn strided layers
// 173 -> 136, 205 -> 105, 248 -> 129, 208 -> 180.  Errors against 64 bits, operands of zero mean: 1.2 to 5 times below those of the transforms.
// Forward passes: plan.cpp, at the rule that takes it.  As that of a large first layer it loses (7x7 at stride 2 141 -> 168, 11x11 at stride 4 188 -> 260 us).
#include <hip/hip_runtime.h>

#include "direct_filter.hpp"
#include "plan.hpp"
#include "split.hpp"

namespace dwm {

__global__ __launch_bounds__(256) void direct_filter_kernel(DirectArgs A, FilterSource F, const float* __restrict__ w, float* __restrict__ U)
{
    direct_filter(A, F, w, U, blockIdx.x, blockIdx.y);
}

// The arguments read again where they are used, not kept in registers across the step loop
typedef const __attribute__((address_space(4))) DirectArgs ColdArgs;
__device__ __forceinline__ ColdArgs& cold_args()
{
    ColdArgs* a = (ColdArgs*)__builtin_amdgcn_kernarg_segment_ptr();  // (they are the kernel's first argument)
    asm volatile("" : "+s"(a));
    return *a;
}
#define DWM_DIV(field, n) ((int)((__umulhi((unsigned)(n), B.field.mul) + (unsigned)(n)) >> B.field.shift))

constexpr uint32_t kDirectTable = 2 * kDirectMaxUnits * 4;  // LDS bytes of the units' offsets, before the staged pixels

// Workgroup of WF x WP x WK waves: 32*MB*WF filters x 64*WP output pixels; a wave 32*MB x 64 and every WK-th step.
// LONG: sums in two levels (see the head of the file)
template <int WF, int WP, int WK, int MB, bool LONG>
__global__ __launch_bounds__(64 * WF * WP * WK, 2) void direct_kernel(DirectArgs A, const float* __restrict__ x,
                                                                      const unsigned char* __restrict__ Wd,
                                                                      const float* __restrict__ W32, float* __restrict__ out_y)
{
    constexpr int NT = 64 * WF * WP * WK, NPX = 64 * WP, KT = 32 * MB * WF, NB = 2, NS = kDirectSlots, AHEAD = 4;
    static_assert(NS == 3, "load_slot");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_d[];  // the units' offsets, then groups[0] * P pixels

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int li = lane & 31, half = lane >> 5;
    const int wk = wave / (WF * WP), wf = wave / WP % WF, wp = wave % WP;
    const uint32_t gbytes = (uint32_t)A.P * 48u;

    // the tiles of one pixel tile, all problems and filters, on one XCD
    const int per = A.nkt * A.nprob;
    const bool low = (int)blockIdx.x < A.full8;
    const int r0 = low ? (int)blockIdx.x >> 3 : (int)blockIdx.x - A.full8;
    const int place0 = r0 % per, tt = low ? (r0 / per) * 8 + ((int)blockIdx.x & 7) : (A.ntt / 8) * 8 + r0 / per;
    // (an XCD's 32 CUs get its workgroups in turn, problems lie longest first: every other 32 the other way round, or, with four problems,
    // a CU's workgroups were all long or all short, and CUs busy for 0.57 of the time: 3x3 at stride 2, 128 <- 256 channels)
    const int inner = (r0 - place0) / 32 % 2 == 0 ? place0 : per - 1 - place0;
    const int pi = inner / A.nkt, kt = inner - pi * A.nkt;

    // ---- this thread's staged pixels and this lane's output pixels ----
    uint32_t go[NS];  // byte offset in x from the tile's first image, or past its end
    uint32_t lb[NB];  // LDS offset
    __amdgpu_buffer_rsrc_t xrs;
    int steps0, steps1, S;
    uint32_t wat0;    // the problem's and filter tile's place in Wd
    const uint32_t part_bytes = 2u * (uint32_t)A.Kpad * 16u, step_bytes = 3u * part_bytes;
    {
        ColdArgs& B = cold_args();
        const auto& q = B.p[pi];
        steps0 = q.steps[0];
        steps1 = q.steps[1];
        S = q.S;
        wat0 = (uint32_t)q.step0 * step_bytes + (uint32_t)kt * KT * 16u;
        const int g0 = DWM_DIV(div_bw, tt * NPX), v0 = DWM_DIV(div_oh, g0), oh0 = g0 - v0 * B.OH;
        const int n0 = DWM_DIV(div_strips, v0), nr0 = B.rstep * (B.OH - 1 - oh0) + B.run;
        const int image = B.C * B.H * B.W;
        const size_t left = ((size_t)(B.N - n0) * image + B.bias) * 4;
        xrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x + (size_t)n0 * image) - B.bias, 0,
                                                (int)(left < 0x7ffffff0u ? left : 0x7ffffff0u), 0x00020000);
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            go[i] = 0x80000000u;
            if (i >= B.ns) continue;
            const int px = tid + i * NT;
            const int j = DWM_DIV(div_row, px), pc = px - j * B.row_px;
            const int ph = DWM_DIV(div_lwp, pc), jc = pc - ph * B.lwp;
            // staged row j: of image (strip) v, tap row jj - k*rstep of its output row k
            int v = v0, jj = j, base = oh0;
            if (j >= nr0) {
                const int d = DWM_DIV(div_rows, j - nr0);
                v = v0 + 1 + d;
                jj = j - nr0 - d * B.rows_full;
                base = 0;
            }
            const int k = DWM_DIV(div_rstep, jj), n = DWM_DIV(div_strips, v), strip = v - n * B.nstrips;
            const int ih = B.s * (base + k) + (jj - k * B.rstep) - q.Ph, iw = B.s * (strip * B.bw + jc) + ph - q.Pw;
            const bool in = px < B.P && n < B.N && (unsigned)ih < (unsigned)B.H && (unsigned)iw < (unsigned)B.W;
            go[i] = in ? (uint32_t)((n - n0) * image + ih * B.W + iw + B.bias) * 4u : 0x80000000u;
        }
#pragma unroll
        for (int ni = 0; ni < NB; ++ni) {
            const int p = min(tt * NPX + wp * 64 + ni * 32 + li, B.total_px - 1);
            const int g = DWM_DIV(div_bw, p), ow = p - g * B.bw, v = DWM_DIV(div_oh, g), oh = g - v * B.OH;
            const int j = v == v0 ? B.rstep * (oh - oh0) : nr0 + (v - v0 - 1) * B.rows_full + B.rstep * oh;
            lb[ni] = kDirectTable + (uint32_t)(j * B.row_px + ow) * 48u;
        }
    }
    // the units' offsets: tap outer, group inner; past the last unit that unit's (zeros of the filter meet it)
#pragma unroll 1
    for (int t = A.nchunks > 1 ? 0 : 1; t < 2; ++t) {
        ColdArgs& B = cold_args();
        const int G = B.groups[t], units = G * B.p[pi].R * S;
        for (int i = tid; i < units + 1; i += NT) {
            const int u = min(i, units - 1), tap = u / G, r = tap / S, s = tap - r * S, sq = s / B.s;
            reinterpret_cast<uint32_t*>(smem_d)[t * kDirectMaxUnits + i] =
                (uint32_t)(u - tap * G) * gbytes + (uint32_t)(r * B.row_px + (s - sq * B.s) * B.lwp + sq) * 48u;
        }
    }

    // ---- the filter: this lane's fragments ----
    const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(Wd), 0, (int)A.wd_bytes, 0x00020000);
    const uint32_t wlane = (uint32_t)(half * A.Kpad + wf * MB * 32 + li) * 16u;
    uint32_t wat = 0;  // a step's place in Wd
    auto load_a = [&](bf16x8 (&a)[MB], int part) {
#pragma unroll
        for (int mi = 0; mi < MB; ++mi)
            a[mi] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(wrs, wlane + mi * 512u, wat + part * part_bytes, 0));
    };

    floatx16 acc[MB][NB][2];
#pragma unroll
    for (int mi = 0; mi < MB; ++mi)
#pragma unroll
        for (int ni = 0; ni < NB; ++ni)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[mi][ni][0][e] = acc[mi][ni][1][e] = 0.f;

    // ---- staging: slots of (group, this thread's i-th pixel) ----
    const uint32_t hw = (uint32_t)(A.H * A.W) * 4u;
    struct Slot {
        int g, i;
    };
    auto next_slot = [&](Slot& q) {
        if (++q.i == A.ns) {
            q.i = 0;
            ++q.g;
        }
    };
    auto load_slot = [&](int chunk, const Slot& q, float (&v)[8]) {  // (channels past the last meet zeros of the filter: they repeat it)
        const uint32_t one = q.i == 1 ? 0xffffffffu : 0u, two = q.i == 2 ? 0xffffffffu : 0u;
        uint32_t off = (go[1] & one) | (go[0] & ~one);
        off = (go[2] & two) | (off & ~two);
        const int c0 = (chunk * A.groups[0] + q.g) * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            v[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xrs, off, (uint32_t)min(c0 + e, A.C - 1) * hw, 0));
    };
    auto put_slot = [&](const Slot& q, float (&v)[8]) {
        const int px = tid + q.i * NT;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] *= kSplitScale;
        bf16x8 f[3];
        split8(v, f);
        if (px < A.P) {
            unsigned char* d = smem_d + kDirectTable + ((uint32_t)q.g * gbytes + (uint32_t)px * 48u);
#pragma unroll
            for (int p = 0; p < 3; ++p) *reinterpret_cast<puint4*>(d + p * 16) = __builtin_bit_cast(puint4, f[p]);
        }
    };
    float ahead[AHEAD][8];  // a chunk's first slots, on their way while the chunk before is multiplied
    auto load_ahead = [&](int chunk) {
        const int groups = chunk == A.nchunks - 1 ? A.groups[1] : A.groups[0];
        Slot q{0, 0};
#pragma unroll
        for (int j = 0; j < AHEAD; ++j)
            if (q.g < groups) {
                load_slot(chunk, q, ahead[j]);
                next_slot(q);
            }
    };
    auto stage = [&](int chunk, int groups) {
        Slot q{0, 0};
        for (;;) {
            Slot l = q;
#pragma unroll
            for (int j = 0; j < AHEAD; ++j)
                if (q.g < groups) {
                    put_slot(q, ahead[j]);
                    next_slot(q);
                }
            if (q.g >= groups) return;
            l = q;
#pragma unroll
            for (int j = 0; j < AHEAD; ++j)
                if (l.g < groups) {
                    load_slot(chunk, l, ahead[j]);
                    next_slot(l);
                }
        }
    };
    auto barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    // ---- operands ----
    bf16x8 a0[MB], a1[MB], a2[MB], b0[NB], b1[NB], b2[NB];
    uint32_t at[NB], unext, table = 0;
    auto unit_at = [&](int i) { return *reinterpret_cast<const uint32_t*>(smem_d + table + (uint32_t)i * 8u); };
    auto point = [&](uint32_t o) {
#pragma unroll
        for (int ni = 0; ni < NB; ++ni) at[ni] = lb[ni] + o;
    };
    auto read_b = [&](bf16x8 (&b)[NB], int part) {
#pragma unroll
        for (int ni = 0; ni < NB; ++ni) b[ni] = *reinterpret_cast<const bf16x8*>(smem_d + at[ni] + part * 16);
    };
    auto term = [&](const bf16x8 (&a)[MB], const bf16x8 (&b)[NB], int which) {
#pragma unroll
        for (int mi = 0; mi < MB; ++mi)
#pragma unroll
            for (int ni = 0; ni < NB; ++ni)
                acc[mi][ni][LONG ? 0 : which] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[mi], b[ni], acc[mi][ni][LONG ? 0 : which], 0, 0, 0);
    };
    int run = 0;  // steps since the last fold
    auto fold = [&] {
        if constexpr (LONG) {
            if (++run < kDirectFold) return;
            run = 0;
#pragma unroll
            for (int mi = 0; mi < MB; ++mi)
#pragma unroll
                for (int ni = 0; ni < NB; ++ni)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        acc[mi][ni][1][e] += acc[mi][ni][0][e];
                        acc[mi][ni][0][e] = 0.f;
                    }
        }
    };
    // A step: the MFMAs of two units, while the operands of the next one (at `to` in Wd, at unext in LDS) replace those that are
    // done with, part by part.  The sections' order is kept.
    auto step = [&](uint32_t to, int after) {
        wat = to;
        bf16x8 a0n[MB];
        load_a(a0n, 0);
        point(unext);
        unext = unit_at(after);
        __builtin_amdgcn_sched_barrier(0);
        term(a2, b0, 1);
        __builtin_amdgcn_sched_barrier(0);
        load_a(a2, 2);
        __builtin_amdgcn_sched_barrier(0);
        term(a0, b0, 0);
        term(a1, b0, 1);
        __builtin_amdgcn_sched_barrier(0);
        read_b(b0, 0);
        __builtin_amdgcn_sched_barrier(0);
        term(a1, b1, 1);
        __builtin_amdgcn_sched_barrier(0);
        load_a(a1, 1);
        __builtin_amdgcn_sched_barrier(0);
        term(a0, b1, 1);
        __builtin_amdgcn_sched_barrier(0);
        read_b(b1, 1);
        __builtin_amdgcn_sched_barrier(0);
        term(a0, b2, 1);
        __builtin_amdgcn_sched_barrier(0);
        read_b(b2, 2);
#pragma unroll
        for (int mi = 0; mi < MB; ++mi) a0[mi] = a0n[mi];
    };

    const int chunk0 = (int)blockIdx.y * A.cpp, chunk1 = min(chunk0 + A.cpp, A.nchunks);  // this piece's
    load_ahead(chunk0);
#pragma unroll 1
    for (int chunk = chunk0; chunk < chunk1; ++chunk) {
        const bool last = chunk == A.nchunks - 1;
        const int nst = last ? steps1 : steps0, top = nst - 1;
        const uint32_t wchunk = wat0 + (uint32_t)(chunk * steps0) * step_bytes;
        const bool some = WK == 1 || wk < nst;
        wat = wchunk + (uint32_t)min(wk, top) * step_bytes;
        load_a(a2, 2);
        load_a(a0, 0);
        load_a(a1, 1);
        stage(chunk, last ? A.groups[1] : A.groups[0]);
        barrier();
        table = (uint32_t)half * 4u + (last ? kDirectMaxUnits * 4u : 0u);
        point(unit_at(min(wk, top)));
        read_b(b0, 0);
        read_b(b1, 1);
        read_b(b2, 2);
        unext = unit_at(min(wk + WK, top));
        asm volatile("" : "+v"(unext));
        __builtin_amdgcn_s_waitcnt(0xf70);  // vmcnt(0): the first step's operands, not what comes next, are waited for
        if (chunk + 1 < chunk1) load_ahead(chunk + 1);
        if (some) {
            step(wchunk + (uint32_t)min(wk + WK, top) * step_bytes, min(wk + 2 * WK, top));
            fold();
#pragma unroll 1
            for (int st = wk + WK; st < nst; st += WK) {
                step(wchunk + (uint32_t)min(st + WK, top) * step_bytes, min(st + 2 * WK, top));
                fold();
            }
        }
        barrier();
    }

    // ---- outputs: of a tile's MB x NB x 16 values a lane, this wave stores a WK-th ----
    constexpr int VALUES = MB * NB * 16, OWN = VALUES / WK;
    float out[OWN];
    if constexpr (WK == 1) {
#pragma unroll
        for (int i = 0; i < OWN; ++i) out[i] = (acc[i / 32][i / 16 % 2][0][i % 16] + acc[i / 32][i / 16 % 2][1][i % 16]) * (1.f / kSplitScale / kSplitScale);
    } else {
        float* sum = reinterpret_cast<float*>(smem_d + kDirectTable) + (size_t)(wf * WP + wp) * WK * VALUES * 64 + lane;
#pragma unroll
        for (int i = 0; i < VALUES; ++i)
            sum[(wk * VALUES + i) * 64] = (acc[i / 32][i / 16 % 2][0][i % 16] + acc[i / 32][i / 16 % 2][1][i % 16]) * (1.f / kSplitScale / kSplitScale);
        barrier();
#pragma unroll
        for (int i = 0; i < OWN; ++i) out[i] = sum[(wk * OWN + i) * 64];
#pragma unroll
        for (int w = 1; w < WK; ++w)
#pragma unroll
            for (int i = 0; i < OWN; ++i) out[i] += sum[(w * VALUES + wk * OWN + i) * 64];
    }
    ColdArgs& B = cold_args();
    const auto& q = B.p[pi];
    const int g0 = DWM_DIV(div_bw, tt * NPX), n0 = DWM_DIV(div_strips, DWM_DIV(div_oh, g0));
    float* y = out_y + blockIdx.y * B.piece_floats;
    const int plane = B.YH * B.YW, kw = kt * KT + wf * MB * 32;
    const __amdgpu_buffer_rsrc_t yrs = __builtin_amdgcn_make_buffer_rsrc(y + ((size_t)n0 * B.K + kw) * plane, 0, 0x7ffffff0, 0x00020000);
    struct Place {
        int n, oh, ow;
        bool in;
    };
    auto place = [&](int ni) {
        const int p = tt * NPX + wp * 64 + ni * 32 + li, pc = min(p, B.total_px - 1);
        const int g = DWM_DIV(div_bw, pc), v = DWM_DIV(div_oh, g), n = DWM_DIV(div_strips, v);
        const int oh = g - v * B.OH, ow = (v - n * B.nstrips) * B.bw + (pc - g * B.bw);
        return Place{n, oh, ow, p < B.total_px && oh < q.OH && ow < q.OW};
    };
    auto store = [&](const Place& a, int k, float f) {  // filter kw + k (k: of the wave's first half); past the last: dropped
        const uint32_t yo = (uint32_t)(((a.n - n0) * B.K + 4 * half) * plane + (B.sy * a.oh + q.oy) * B.YW + B.sx * a.ow + q.ox) * 4u;
        const int room = a.in ? B.K - kw - 4 * half : 0;
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, f), yrs, k < room ? yo : 0x80000000u, (uint32_t)(k * plane) * 4u, 0);
    };
    // value i of the wave's own: block i / 16 of (filters, pixels), element i % 16
    uint64_t lost = 0;
    constexpr int SPAN = OWN < 16 ? OWN : 16;
#pragma unroll
    for (int b = 0; b < OWN / SPAN; ++b) {
        const int v0 = wk * OWN + b * SPAN, mi = v0 / 32, ni = v0 / 16 % 2;
        const Place a = place(ni);
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < SPAN; ++i) {
            const float f = out[b * SPAN + i];
            const int e = v0 % 16 + i;
            t = fmaf(f, 0.f, t);
            store(a, mi * 32 + 8 * (e >> 2) + (e & 3), f);
        }
        lost |= __builtin_amdgcn_ballot_w64(t != 0.f && a.in);
    }
    if (__builtin_expect(lost != 0, 0)) {
        // operands or sums that the parts cannot carry: the wave's outputs again, on fp32 MFMAs, from x and W32 -- all of a tile that
        // is the wave's alone, of a shared one the block of 32 x 32 that holds its values -- 16 channels of a tap at a time, the next
        // ones on their way.  What is not there (channels past the piece's last, pixels outside x) is loaded as zero.
        constexpr bool ALL = WK == 1;
        static_assert(ALL || OWN <= 16, "values of one block");
        constexpr int RM = ALL ? MB : 1, RN = ALL ? NB : 1;
        const int v0 = ALL ? 0 : wk * OWN, mi0 = v0 / 32, ni0 = v0 / 16 % 2;
        const int c_begin = (int)blockIdx.y * B.cpp * B.groups[0] * 8, c_end = min(B.C, c_begin + B.cpp * B.groups[0] * 8);
        const int image = B.C * B.H * B.W, taps = q.R * q.S;
        const uint32_t krow = (uint32_t)B.Kpad * 4u;
        const size_t left = ((size_t)(B.N - n0) * image + B.bias) * 4;
        const __amdgpu_buffer_rsrc_t xs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x + (size_t)n0 * image) - B.bias, 0,
                                                                            (int)(left < 0x7ffffff0u ? left : 0x7ffffff0u), 0x00020000);
        const __amdgpu_buffer_rsrc_t ws = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(W32 + q.w32), 0, taps * B.C * (int)krow, 0x00020000);
        Place pl[RN];
#pragma unroll
        for (int ni = 0; ni < RN; ++ni) pl[ni] = place(ni0 + ni);
        const uint32_t wo = (uint32_t)(half * 8) * krow + (uint32_t)(kw + mi0 * 32 + li) * 4u;
        uint32_t xo[RN];
        int t = -1, c = c_end;
        auto next = [&] {  // the next 16 channels, or the next tap's first
            c += 16;
            if (c < c_end) return;
            c = c_begin;
            ++t;
            const int r = t / q.S, s = t - r * q.S;
#pragma unroll
            for (int ni = 0; ni < RN; ++ni) {
                const int ih = B.s * pl[ni].oh - q.Ph + r, iw = B.s * pl[ni].ow - q.Pw + s;
                const bool ok = pl[ni].in && (unsigned)ih < (unsigned)B.H && (unsigned)iw < (unsigned)B.W;
                xo[ni] = ok ? (uint32_t)((pl[ni].n - n0) * image + ih * B.W + iw + B.bias) * 4u + (uint32_t)(half * 8) * hw : 0x80000000u;
            }
        };
        auto load = [&](float (&a)[RM][8], float (&v)[RN][8]) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bool there = c + half * 8 + e < c_end;
                const int ce = min(c + e, B.C - 1);  // (no scalar offset lies past its buffer)
#pragma unroll
                for (int mi = 0; mi < RM; ++mi)
                    a[mi][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ws, there ? wo + mi * 128u : 0x80000000u,
                                                                                              (uint32_t)(t * B.C + ce) * krow, 0));
#pragma unroll
                for (int ni = 0; ni < RN; ++ni)
                    v[ni][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xs, there ? xo[ni] : 0x80000000u, (uint32_t)ce * hw, 0));
            }
        };
        floatx16 sum[RM][RN];
#pragma unroll
        for (int mi = 0; mi < RM; ++mi)
#pragma unroll
            for (int ni = 0; ni < RN; ++ni)
#pragma unroll
                for (int e = 0; e < 16; ++e) sum[mi][ni][e] = 0.f;
        auto multiply = [&](const float (&a)[RM][8], const float (&v)[RN][8]) {
#pragma unroll
            for (int mi = 0; mi < RM; ++mi)
#pragma unroll
                for (int ni = 0; ni < RN; ++ni) {
                    floatx16 m;
#pragma unroll
                    for (int e = 0; e < 16; ++e) m[e] = 0.f;
#pragma unroll
                    for (int e = 0; e < 8; ++e) m = __builtin_amdgcn_mfma_f32_32x32x2f32(a[mi][e], v[ni][e], m, 0, 0, 0);
                    sum[mi][ni] += m;
                }
        };
        float a0f[RM][8], v0f[RN][8], a1f[RM][8], v1f[RN][8];
        next();
        load(a0f, v0f);
#pragma unroll 1
        for (int left_over = taps * ((c_end - c_begin + 15) / 16);;) {
            if (left_over > 1) {
                next();
                load(a1f, v1f);
            }
            multiply(a0f, v0f);
            if (--left_over == 0) break;
            if (left_over > 1) {
                next();
                load(a0f, v0f);
            }
            multiply(a1f, v1f);
            if (--left_over == 0) break;
        }
#pragma unroll
        for (int mi = 0; mi < RM; ++mi)
#pragma unroll
            for (int ni = 0; ni < RN; ++ni)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (ALL || (e >= v0 % 16 && e < v0 % 16 + OWN)) store(pl[ni], (mi0 + mi) * 32 + 8 * (e >> 2) + (e & 3), sum[mi][ni][e]);
    }
}

// The outputs of layers whose tiles were cut into pieces: the pieces' sums, added in order.  Bound by its launch and the one round
// of loads that a thread has under way at a time.
__global__ __launch_bounds__(256) void direct_sum_kernel(const float* __restrict__ partial, float* __restrict__ y, size_t n, size_t stride, int pieces)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    float v[kDirectMaxPieces];
#pragma unroll
    for (int p = 0; p < kDirectMaxPieces; ++p) v[p] = p < pieces ? partial[p * stride + i] : 0.f;
    float sum = v[0];
#pragma unroll
    for (int p = 1; p < kDirectMaxPieces; ++p)
        if (p < pieces) sum += v[p];
    y[i] = sum;
}

// ---------------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------------
template <int WF, int WP, int WK, int MB, bool LONG = false>
static dwm_status_t launch_shape(const DirectArgs& a, const float* x, const unsigned char* Wd, const float* W32, float* y, float* partial, void* stream)
{
    if constexpr (!LONG)
        if (a.two_level) return launch_shape<WF, WP, WK, MB, true>(a, x, Wd, W32, y, partial, stream);
    if (a.kt != 32 * MB * WF || a.npx != 64 * WP || (a.pieces > 1 && !partial)) return DWM_ERR_INVALID_ARG;
    auto kernel = direct_kernel<WF, WP, WK, MB, LONG>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr != hipSuccess) return DWM_ERR_HIP;
    hipLaunchKernelGGL(kernel, dim3((unsigned)a.ntiles, (unsigned)a.pieces), dim3(64 * WF * WP * WK), a.lds_bytes, (hipStream_t)stream, a, x, Wd, W32,
                       a.pieces > 1 ? partial : y);
    if (hipGetLastError() != hipSuccess) return DWM_ERR_HIP;
    if (a.pieces == 1) return DWM_OK;
    const size_t n = (size_t)a.N * a.K * a.YH * a.YW;
    hipLaunchKernelGGL(direct_sum_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, partial, y, n, a.piece_floats, a.pieces);
    return hipGetLastError() == hipSuccess ? DWM_OK : DWM_ERR_HIP;
}

dwm_status_t launch_direct(const dwm_plan& p, const float* x, const float* U, float* y, float* ws, void* stream)
{
    const DirectArgs& a = p.direct;
    const unsigned char* Wd = reinterpret_cast<const unsigned char*>(U + p.ud_begin);
    const float* W32 = U + p.ud_begin + a.wd_bytes / 4;
    float* partial = p.sk_partial(ws);
    switch (a.shape) {
        case 0: return launch_shape<4, 2, 1, 2>(a, x, Wd, W32, y, partial, stream);
        case 1: return launch_shape<2, 2, 1, 2>(a, x, Wd, W32, y, partial, stream);
        case 2: return launch_shape<1, 1, 8, 1>(a, x, Wd, W32, y, partial, stream);
        case 3: return launch_shape<1, 1, 4, 1>(a, x, Wd, W32, y, partial, stream);
        case 4: return launch_shape<1, 1, 4, 2>(a, x, Wd, W32, y, partial, stream);
    }
    return DWM_ERR_INVALID_ARG;
}

dwm_status_t launch_direct_filter(const DirectArgs& a, const FilterSource& src, const float* w, float* U, void* stream)
{
    hipLaunchKernelGGL(direct_filter_kernel, dim3((unsigned)a.all_steps, (unsigned)((a.Kpad + 127) / 128)), dim3(256), 0, (hipStream_t)stream,
                       a, src, w, U);
    return hipGetLastError() == hipSuccess ? DWM_OK : DWM_ERR_HIP;
}

}  // namespace dwm
