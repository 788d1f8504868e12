// What the host code of a .hip file names of HIP's header, for a build by g++ that launches nothing (backward_fuzz.cpp).
#pragma once
#include <cstddef>
#include <cstdint>

#define __global__
#define __launch_bounds__(...)
struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
static const dim3 blockIdx, gridDim, threadIdx;
typedef void* hipStream_t;
enum hipError_t { hipSuccess };
inline hipError_t hipGetLastError() { return hipSuccess; }
template <typename... T>
void hipLaunchKernelGGL(const T&...)
{
}
