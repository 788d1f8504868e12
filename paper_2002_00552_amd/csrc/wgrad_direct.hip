// Gradient of the convolution with respect to its filter without Winograd transforms, in single precision on the bfloat16
// matrix cores:  dw[k][c,r,q] = sum over output pixels of dy[k][pixel] * xp[c][s * pixel + (r,q)].
//
// Why: the transforms' way writes the transformed input (a first layer's is several times x) and reads it back, on top of
// three to five launches; its products run on fp32 matrix cores where channels are few.  Here x and dy are read from where they
// are, and the product is a GEMM [filters] x [pixels] x [channels, taps] that wastes nothing on channels that there are not.
//
// What it does: eight images make the eight elements of an operand (where there are fewer, bands of an image's rows stand
// for images), so that the same staged element serves every tap: a lane's operand is eight images' value of one pixel, at any
// offset a whole 16-byte read.  A unit is a patch of 16 output pixels in eight images: dy's 16 x KT and x's patch of it with
// the taps' margin are split into their three bfloat16 parts (split.hpp) and staged in LDS, 48 bytes each; four waves take
// two steps of two pixels each, all KT x 32*NB products of a tile, and add up their sums in LDS at the end.  Tiles are
// KT filters x 32*NB (channel, tap) columns in the order that dw has; the units are cut into pieces that fill the chip, each
// writes its sums, and a second launch adds those up in order: results do not vary from run to run.
//
// Operands are split as v * 2^16, sums multiplied by 2^-32, as in direct.hip; a sum that is not finite (infinities, NaN, values
// from 2^112 on) is computed again in binary32: the workgroup that has one goes through its units a second time, the values
// staged as they are in the same places, on fp32 MFMAs, one an image and two pixels, and replaces the sums that were not finite.  7x7 at
// stride 2, 3 -> 64 channels, 64 224x224 images 122 us, with one infinity in x 242, NaN throughout 291 (each such tap summed by a
// thread of its own 7500 and 16200).
//
// Bound by what a unit takes besides its MFMAs: splitting (7 vector instructions an element), the lines of dy that a patch's short
// rows touch, and the latency of both, which only the other workgroup on the CU covers.  Measured, whole gradient, transforms
// -> here (us): 7x7 at stride 2, 3 -> 64 channels, 64 224x224 images 322 -> 122 (0.74 PFLOP/s of bf16 products; dy alone takes 40
// at 5.2 TB/s); 5x5 at stride 2, 3 -> 31, ten 151x147 images 91 -> 19; 5x5, 16 -> 16, one 32x32 image 27 -> 7.9.  What it
// took: patches side by side in the hands of one XCD at a time (282 -> 148: with pieces of consecutive units every line of dy
// came from memory eight times), one offset for eight images (149 -> 137: 600 scalar instructions a unit fewer).
// Errors against 64 bits are a third to a tenth of the transforms'.
#include <hip/hip_runtime.h>

#include "plan.hpp"
#include "split.hpp"

namespace dwm {

// where a unit lies: its group of eight images, first output row of its patch within the band, first column
struct WdUnit {
    int g, oh, ow;
};
__device__ __forceinline__ WdUnit wd_unit(const WdArgs& A, int u)
{
    const int t = A.div_npx.div(u), px = u - t * A.npx, g = A.div_npy.div(t), py = t - g * A.npy;
    return WdUnit{g, py * (16 >> A.lgw), px << A.lgw};
}

// All of workgroup `block`'s units; EXACT: in binary32, in the place of the sums that are not finite.  Returns whether one of the
// workgroup's is not.
template <int MB, int NB, bool BANDS, bool EXACT>
__device__ __forceinline__ bool wd_pass(const WdArgs& A, const float* __restrict__ x, const float* __restrict__ dy, float* __restrict__ out, int tid, int block)
{
    constexpr int KT = 32 * MB, CT = 32 * NB;
    constexpr uint32_t PITCH = KT * 48 + 16;  // bytes of a pixel's KT elements of dy, banks moved on by four words
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_w[];
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = tid & 31, half = tid >> 5 & 1;
    // An XCD's units are a range of their own, which its pieces take in turn: patches side by side share lines of dy and x, and
    // are read at about the same time.  A piece's tiles, which read the same, are next to one another.
    // (Fewer than eight units: each is a piece, and its tiles go to all XCDs.)
    const int ranges = A.nunits < 8 ? A.nunits : 8, range = block % ranges, r0 = block / ranges;
    const int tile = r0 % A.ntiles, piece = r0 / A.ntiles * ranges + range;
    const int kt = tile % A.nkt, ct = tile / A.nkt;
    const int first = range * A.xunits, u0 = first + r0 / A.ntiles, u1 = min(first + A.xunits, A.nunits);
    const int RS = A.R * A.S, plane = A.rows * A.pcols, mask = (1 << A.lgw) - 1;
    const int clo = A.div_rs.div(ct * CT), chi = A.div_rs.div(min(ct * CT + CT, A.cols) - 1), npix = (chi - clo + 1) * plane;
    unsigned char* const sx = smem_w + 16 * PITCH;

    floatx16 acc[MB][NB];

    // (EXACT: the binary32 values as they are, the last third of their place unused)
    auto put = [&](unsigned char* d, float (&v)[8], float scale, int images) {
        if constexpr (EXACT) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = e < images ? v[e] : 0.f;
            *reinterpret_cast<pfloat4*>(d) = pfloat4{v[0], v[1], v[2], v[3]};
            *reinterpret_cast<pfloat4*>(d + 16) = pfloat4{v[4], v[5], v[6], v[7]};
            return;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] *= e < images ? scale : 0.f;
        bf16x8 f[3];
        split8(v, f);
#pragma unroll
        for (int p = 0; p < 3; ++p) *reinterpret_cast<puint4*>(d + p * 16) = __builtin_bit_cast(puint4, f[p]);
    };
    const uint32_t ohw = (uint32_t)(A.OH * A.OW);

    uint32_t bo[NB];  // this lane's columns' taps in the staged patch
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int col = min(ct * CT + nb * 32 + li, A.cols - 1), c = A.div_rs.div(col), tap = col - c * RS, r = tap / A.S, q = tap - r * A.S;
        bo[nb] = (uint32_t)((c - clo) * plane + r * A.pcols + q) * 48u;
    }
#pragma unroll
    for (int mi = 0; mi < MB; ++mi)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[mi][nb][e] = 0.f;
#pragma unroll 1
    for (int u = u0; u < u1; u += A.ustep) {
        const WdUnit un = wd_unit(A, u);
        // ---- dy: filter k, pixel p of the patch (filters past the last: whatever follows; their sums are not stored) ----
        float vd[2 * MB][8], vx[2][8];
        const int p = tid & 15, ol = un.oh + (p >> A.lgw), ow = un.ow + (p & mask);
        uint32_t off[2 * MB];
#pragma unroll
        for (int j = 0; j < 2 * MB; ++j) {
            const int k = kt * KT + (tid >> 4) + 16 * j;
            off[j] = k < A.K && ol < A.BH && ow < A.OW ? ((uint32_t)k * ohw + (uint32_t)(ol * A.OW + ow)) * 4u : 0x80000000u;
        }
        const int n0 = un.g * 8;  // (without bands)
        const __amdgpu_buffer_rsrc_t drs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(dy) + (size_t)n0 * A.K * ohw, 0, 0x7ffffff0, 0x00020000);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if constexpr (BANDS) {
                const int vi = un.g * 8 + e, n = A.div_nb.div(vi), oh0 = (vi - n * A.NB) * A.BH;
                const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                    const_cast<float*>(dy) + ((size_t)n * A.K * A.OH + oh0) * A.OW, 0, n < A.N ? 0x7ffffff0 : 0, 0x00020000);
#pragma unroll
                for (int j = 0; j < 2 * MB; ++j)
                    vd[j][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, ol < A.OH - oh0 ? off[j] : 0x80000000u, 0, 0));
            } else {
                const uint32_t image = (uint32_t)(min(n0 + e, A.N - 1) - n0) * (A.K * ohw * 4u);
#pragma unroll
                for (int j = 0; j < 2 * MB; ++j) vd[j][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(drs, off[j], image, 0));
            }
        }
        // ---- x: the patch with the taps' margin, two pixels a turn ----
        const int iw0 = A.s * un.ow - A.P, ih0 = A.s * un.oh - A.P;
        const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float*>(x) + ((long long)n0 * A.C * A.H + ih0) * A.W, 0, 0x7ffffff0, 0x00020000);
        auto load_x = [&](int i0, float (&v)[2][8]) {
            int row[2];
            uint32_t at[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int i = i0 + 256 * j, c = A.div_plane.div(i), t = i - c * plane;
                row[j] = A.div_pcols.div(t);
                const int iw = iw0 + t - row[j] * A.pcols;
                const bool ok = i < npix && (unsigned)iw < (unsigned)A.W && (BANDS || (unsigned)(ih0 + row[j]) < (unsigned)A.H);
                at[j] = ok ? (uint32_t)(((clo + c) * A.H + row[j]) * A.W + iw) * 4u : 0x80000000u;
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if constexpr (BANDS) {
                    const int vi = un.g * 8 + e, n = A.div_nb.div(vi), top = ih0 + A.s * (vi - n * A.NB) * A.BH;
                    // (the first row may lie before the image: what would be read there is out of range)
                    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                        const_cast<float*>(x) + ((long long)n * A.C * A.H + top) * A.W, 0, n < A.N ? 0x7ffffff0 : 0, 0x00020000);
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        v[j][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                                rs, (unsigned)(top + row[j]) < (unsigned)A.H ? at[j] : 0x80000000u, 0, 0));
                } else {
                    const uint32_t image = (uint32_t)(min(n0 + e, A.N - 1) - n0) * (uint32_t)(A.C * A.H * A.W * 4);
#pragma unroll
                    for (int j = 0; j < 2; ++j) v[j][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xrs, at[j], image, 0));
                }
            }
        };
        load_x(tid, vx);
        // (the second steps' pixels with the sign turned, see below)
#pragma unroll
        for (int j = 0; j < 2 * MB; ++j)
            put(smem_w + (uint32_t)p * PITCH + (uint32_t)((tid >> 4) + 16 * j) * 48u, vd[j], p < 8 ? kSplitScale : -kSplitScale, BANDS ? 8 : A.N - n0);
#pragma unroll 1
        for (int i0 = tid;;) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
                if (i0 + 256 * j < npix) put(sx + (uint32_t)(i0 + 256 * j) * 48u, vx[j], kSplitScale, EXACT && !BANDS ? A.N - n0 : 8);
            i0 += 512;
            if (i0 - tid >= npix) break;
            load_x(i0, vx);
        }
        __syncthreads();
        // ---- products: this wave's two steps ----
        auto pixel_of = [&](int q) { return smem_w + (uint32_t)q * PITCH + (uint32_t)li * 48u; };
        auto patch_of = [&](int q) { return sx + (uint32_t)((q >> A.lgw) * A.s * A.pcols + (q & mask) * A.s) * 48u; };
        if constexpr (EXACT) {
            // one MFMA for each image, two pixels deep.  (Where there is no output pixel an infinity of x meets no zero of dy.)
            auto eight = [](const unsigned char* from, float (&v)[8]) {
                const pfloat4 lo = *reinterpret_cast<const pfloat4*>(from), hi = *reinterpret_cast<const pfloat4*>(from + 16);
#pragma unroll
                for (int e = 0; e < 4; ++e) { v[e] = lo[e]; v[e + 4] = hi[e]; }
            };
#pragma unroll 1
            for (int t = 0; t < 2; ++t) {
                const int q = 2 * (wave + 4 * t) + half, oq = un.oh + (q >> A.lgw);
                uint32_t in = 0;
#pragma unroll 1
                for (int e = 0; e < 8; ++e) {
                    const int vi = un.g * 8 + e, oh0 = BANDS ? (vi - A.div_nb.div(vi) * A.NB) * A.BH : 0;
                    in |= (uint32_t)(oq < A.BH && oq < A.OH - oh0 && un.ow + (q & mask) < A.OW) << e;
                }
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    float b[8];
                    eight(patch_of(q) + bo[nb], b);
#pragma unroll
                    for (int e = 0; e < 8; ++e) b[e] = in >> e & 1 ? b[e] : 0.f;
#pragma unroll
                    for (int mi = 0; mi < MB; ++mi) {
                        float a[8];
                        eight(pixel_of(q) + mi * 32 * 48, a);
                        floatx16 now;
#pragma unroll
                        for (int e = 0; e < 16; ++e) now[e] = 0.f;
#pragma unroll
                        for (int e = 0; e < 8; ++e) now = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], now, 0, 0, 0);
                        acc[mi][nb] += now;
                        __builtin_amdgcn_sched_barrier(0);  // (registers: what the other products take is not exceeded)
                    }
                }
            }
            __syncthreads();
            continue;
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int q = 2 * (wave + 4 * t) + half;
            const unsigned char* pa = pixel_of(q);
            const unsigned char* pb = patch_of(q);
            bf16x8 a[MB][3];
#pragma unroll
            for (int mi = 0; mi < MB; ++mi)
#pragma unroll
                for (int w = 0; w < 3; ++w) a[mi][w] = *reinterpret_cast<const bf16x8*>(pa + mi * 32 * 48 + w * 16);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                bf16x8 b[3];
#pragma unroll
                for (int w = 0; w < 3; ++w) b[w] = *reinterpret_cast<const bf16x8*>(pb + bo[nb] + w * 16);
                // A step's products by themselves: one rounding at the sums' size, not six.  These MFMAs round down, which over the
                // 800 000 pixels of a first layer is 2e-6 of a sum: of two steps one is multiplied with the sign turned.
                constexpr int M = MB * NB < 10 ? MB : 1;  // (both chains at once where registers allow)
#pragma unroll
                for (int m0 = 0; m0 < MB; m0 += M) {
                    floatx16 now[M];
#pragma unroll
                    for (int mi = 0; mi < M; ++mi)
#pragma unroll
                        for (int e = 0; e < 16; ++e) now[mi][e] = 0.f;
#pragma unroll
                    for (int term = 0; term < 6; ++term) {
                        constexpr int wa[6] = {2, 0, 1, 1, 0, 0}, wb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
                        for (int mi = 0; mi < M; ++mi)
                            now[mi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[m0 + mi][wa[term]], b[wb[term]], now[mi], 0, 0, 0);
                    }
#pragma unroll
                    for (int mi = 0; mi < M; ++mi) acc[m0 + mi][nb] += t == 0 ? now[mi] : -now[mi];
                }
            }
        }
        __syncthreads();
    }

    // ---- the four waves' sums, a block of 32 x 32 at a time (EXACT: in the place of those that were not finite) ----
    float* sum = reinterpret_cast<float*>(smem_w);
    float* const mine = out + (size_t)piece * A.stride;
    auto finite = [](float v) { return fabsf(v) <= 3.402823466e38f; };
    int* const lost = reinterpret_cast<int*>(smem_w) + 4096;  // one of the workgroup's was not (behind the waves' sums, 16 KB of at least 24)
    asm volatile("" : "+v"(tid));  // (where a thread's sums go is not worked out before the units)
    const int lane = tid & 63;
    if (!EXACT && tid == 0) *lost = 0;
#pragma unroll
    for (int mi = 0; mi < MB; ++mi)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
            for (int e = 0; e < 16; ++e) sum[wave * 1024 + e * 64 + lane] = acc[mi][nb][e] * (EXACT ? 1.f : 1.f / kSplitScale / kSplitScale);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int at = tid + 256 * i, e = at >> 6;
                const float v = (sum[at] + sum[1024 + at]) + (sum[2048 + at] + sum[3072 + at]);
                const int k = kt * KT + mi * 32 + 8 * (e >> 2) + (e & 3) + 4 * (lane >> 5), col = ct * CT + nb * 32 + (lane & 31);
                if (k < A.K && col < A.cols) {
                    float* to = mine + (size_t)k * A.cols + col;
                    if (!EXACT || !finite(*to)) *to = v;
                    if (!EXACT && !finite(v)) *lost = 1;
                }
            }
            __syncthreads();
        }
    return *lost != 0;
}

struct WdCall {  // the kernel's arguments
    WdArgs A;
    const float *x, *dy;
    float* out;
};

template <int MB, int NB, bool BANDS>
__global__ __launch_bounds__(256, MB == 1 ? 3 : 2) void wgrad_direct_kernel(WdArgs A, const float* __restrict__ x, const float* __restrict__ dy, float* __restrict__ out)
{
    int block = blockIdx.x, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (__builtin_expect(!wd_pass<MB, NB, BANDS, false>(A, x, dy, out, threadIdx.x, block), 1)) return;
    // (nothing is kept in vector registers from the first pass to this one, not even the thread's number, nor are the arguments)
    __syncthreads();
    typedef const __attribute__((address_space(4))) WdCall Args;
    Args* call = (Args*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(call), "+s"(block), "+s"(wave));
    const WdCall& c = *(const WdCall*)call;
    const int tid = wave * 64 + (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0));
    wd_pass<MB, NB, BANDS, true>(c.A, c.x, c.dy, c.out, tid, block);
}

// dw = the pieces' sums, in order: a thread four neighbours of every 16th piece
__global__ __launch_bounds__(256) void wgrad_direct_sum_kernel(const float* __restrict__ part, float* __restrict__ dw, int n, int stride, int pieces)
{
    __shared__ pfloat4 sm[16][16];
    const int q = threadIdx.x & 15, g = threadIdx.x >> 4, e = (blockIdx.x * 16 + q) * 4;
    pfloat4 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = pfloat4{0.f, 0.f, 0.f, 0.f};
    if (e < n) {
        const float* src = part + e;
        int s = g;
        for (; s + 48 < pieces; s += 64) {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] += *reinterpret_cast<const pfloat4*>(src + (size_t)(s + 16 * j) * stride);
        }
#pragma unroll
        for (int j = 0; j < 3; ++j)
            if (s + 16 * j < pieces) v[j] += *reinterpret_cast<const pfloat4*>(src + (size_t)(s + 16 * j) * stride);
    }
    sm[g][q] = (v[0] + v[1]) + (v[2] + v[3]);
    __syncthreads();
    if (threadIdx.x < 64) {
        const float* p = reinterpret_cast<const float*>(sm) + threadIdx.x;
        float r[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 16; ++i) r[i & 3] += p[i * 64];
        const int at = blockIdx.x * 64 + threadIdx.x;
        if (at < n) dw[at] = (r[0] + r[1]) + (r[2] + r[3]);
    }
}

template <int MB, int NB, bool BANDS>
static dwm_status_t launch_bands(const WdArgs& a, const float* x, const float* dy, float* out, void* stream)
{
    auto kernel = wgrad_direct_kernel<MB, NB, BANDS>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr != hipSuccess) return DWM_ERR_HIP;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(a.pieces * a.ntiles)), dim3(256), a.lds_bytes, (hipStream_t)stream, a, x, dy, out);
    return hipGetLastError() == hipSuccess ? DWM_OK : DWM_ERR_HIP;
}

template <int MB, int NB>
static dwm_status_t launch_tile(const WdArgs& a, const float* x, const float* dy, float* out, void* stream)
{
    return a.per_image ? launch_bands<MB, NB, true>(a, x, dy, out, stream) : launch_bands<MB, NB, false>(a, x, dy, out, stream);
}

dwm_status_t launch_wgrad_direct(const WdArgs& a, const float* x, const float* dy, float* partial, float* dw, void* stream)
{
    float* out = a.pieces > 1 ? partial : dw;
    dwm_status_t st = DWM_ERR_INVALID_ARG;
    switch (a.mb * 8 + a.nb) {
        case 8 + 1: st = launch_tile<1, 1>(a, x, dy, out, stream); break;
        case 8 + 2: st = launch_tile<1, 2>(a, x, dy, out, stream); break;
        case 8 + 3: st = launch_tile<1, 3>(a, x, dy, out, stream); break;
        case 8 + 5: st = launch_tile<1, 5>(a, x, dy, out, stream); break;
        case 16 + 1: st = launch_tile<2, 1>(a, x, dy, out, stream); break;
        case 16 + 2: st = launch_tile<2, 2>(a, x, dy, out, stream); break;
        case 16 + 3: st = launch_tile<2, 3>(a, x, dy, out, stream); break;
        case 16 + 5: st = launch_tile<2, 5>(a, x, dy, out, stream); break;
    }
    if (st != DWM_OK || a.pieces == 1) return st;
    const int n = a.K * a.cols;
    hipLaunchKernelGGL(wgrad_direct_sum_kernel, dim3((unsigned)((n + 63) / 64)), dim3(256), 0, (hipStream_t)stream, partial, dw, n, a.stride, a.pieces);
    return hipGetLastError() == hipSuccess ? DWM_OK : DWM_ERR_HIP;
}

}  // namespace dwm
