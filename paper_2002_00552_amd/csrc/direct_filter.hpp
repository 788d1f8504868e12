// The filter of a direct convolution on split operands (direct.hip), from w where it lies; also transforms.hip's, where the
// filters of a data gradient's sub-convolutions are written in the same launch.
#pragma once

#include "plan.hpp"
#include "split.hpp"

namespace dwm {

// Wd[step][part h,m,l][half][filter (Kpad)][8] of w * 2^16, then W32[problem][tap][channel][Kpad] floats
// (U: both, in this order.)  A workgroup of 256 threads: 128 filters of one step.
__device__ __forceinline__ void direct_filter(const DirectArgs& A, const FilterSource& F, const float* __restrict__ w,
                                              float* __restrict__ U, int step, int kblock)
{
    unsigned char* Wd = reinterpret_cast<unsigned char*>(U);
    float* W32 = U + A.wd_bytes / 4;
    const int half = threadIdx.x >> 7, k = kblock * 128 + (threadIdx.x & 127);
    if (k >= A.Kpad) return;
    int i = 0;
    while (i + 1 < A.nprob && A.p[i + 1].step0 <= step) ++i;
    const DirectProb& q = A.p[i];
    const int rel = step - q.step0, chunk = min(rel / q.steps[0], A.nchunks - 1), st = rel - chunk * q.steps[0];
    const int G = chunk == A.nchunks - 1 ? A.groups[1] : A.groups[0], unit = 2 * st + half;
    const int tap = unit / G, c0 = (chunk * A.groups[0] + unit - tap * G) * 8, r = tap / q.S, s = tap - r * q.S;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        v[e] = 0.f;
        if (r < q.R && c0 + e < A.C) {
            if (k < A.K) v[e] = w[q.at(F, k, c0 + e, r, s)];
            W32[q.w32 + ((long long)tap * A.C + c0 + e) * A.Kpad + k] = v[e];
        }
        v[e] *= kSplitScale;
    }
    bf16x8 f[3];
    split8(v, f);
#pragma unroll
    for (int p = 0; p < 3; ++p)
        *reinterpret_cast<puint4*>(Wd + (((size_t)step * 3 + p) * 2 + half) * A.Kpad * 16 + (size_t)k * 16) = __builtin_bit_cast(puint4, f[p]);
}

}  // namespace dwm
