// Binary32 operands as sums of three bfloat16 numbers (h = rn(x), m = rn(x - h), l = x - h - m), for the kernels that
// multiply them on the bfloat16 matrix cores: contract_split.hip has the reasons and what it measured.
//
// The three parts are the number itself as long as its last bit is one that bfloat16 has: 2^-133, that of its
// subnormals, which the matrix cores keep.  From |x| = 2^-110 on that is so; below, the last part loses bits, then the
// middle one (x around 1e-35 is off by 5e-6 of itself, around 1e-37 by 5e-4).  What is split on the fly is therefore
// split as x * 2^16: every binary32 number, the subnormals too, is then its parts' sum, up to the 2^112 where h
// becomes an infinity.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace dwm {

constexpr float kSplitScale = 0x1p16f;   // what an operand is multiplied by before it is split
constexpr float kSplitMin = 0x1p-110f;   // the smallest magnitude whose parts are exact unscaled

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float pfloat4 __attribute__((ext_vector_type(4)));
typedef unsigned int puint4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// (x0, x1) -> their bfloat16 parts, packed; x0, x1 become what is left over
__device__ __forceinline__ uint32_t take_bf16(float& x0, float& x1)
{
    const floatx2 v = {x0, x1};
    const uint32_t p = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
    x0 -= __builtin_bit_cast(float, p << 16);
    x1 -= __builtin_bit_cast(float, p & 0xffff0000u);
    return p;
}

// two binary32 values -> their three parts, packed
__device__ __forceinline__ void split2(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l)
{
    h = take_bf16(a, b);
    m = take_bf16(a, b);
    const floatx2 r = {a, b};
    l = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, bf16x2));
}

// eight binary32 values -> their three parts as MFMA fragments
__device__ __forceinline__ void split8(const float x[8], bf16x8 out[3])
{
    uint32_t w[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) split2(x[2 * i], x[2 * i + 1], w[0][i], w[1][i], w[2][i]);
#pragma unroll
    for (int s = 0; s < 3; ++s) out[s] = __builtin_bit_cast(bf16x8, puint4{w[s][0], w[s][1], w[s][2], w[s][3]});
}

// instruction classes of __builtin_amdgcn_sched_group_barrier
constexpr int kValu = 0x2, kMfma = 0x8;

// asks the scheduler for MFMAS times: an MFMA, then VALUS vector instructions
template <int MFMAS, int VALUS>
__device__ __forceinline__ void interleave()
{
#pragma unroll
    for (int x = 0; x < MFMAS; ++x) {
        __builtin_amdgcn_sched_group_barrier(kMfma, 1, 0);
        __builtin_amdgcn_sched_group_barrier(kValu, VALUS, 0);
    }
}

}  // namespace dwm
