// Expert sets as 128-bit masks, for the kernels that walk routing traces.
#pragma once

#include "common.h"

namespace remoe {

struct __attribute__((aligned(16))) Mask {
    uint32_t w[4];
    __device__ __forceinline__ Mask &operator|=(const Mask &o)
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] |= o.w[q];
        return *this;
    }
};

__device__ __forceinline__ Mask without(const Mask &a, const Mask &b)
{
    Mask r;
#pragma unroll
    for (int q = 0; q < 4; ++q) r.w[q] = a.w[q] & ~b.w[q];
    return r;
}

__device__ __forceinline__ bool any(const Mask &a) { return (a.w[0] | a.w[1] | a.w[2] | a.w[3]) != 0u; }
__device__ __forceinline__ int count(const Mask &a) { return __popc(a.w[0]) + __popc(a.w[1]) + __popc(a.w[2]) + __popc(a.w[3]); }

__device__ __forceinline__ Mask single(int e)
{
    Mask r;
#pragma unroll
    for (int q = 0; q < 4; ++q) r.w[q] = (e >> 5) == q ? 1u << (e & 31) : 0u;
    return r;
}

__device__ __forceinline__ void drop_lowest(Mask &a)
{
    if (a.w[0]) a.w[0] &= a.w[0] - 1u;
    else if (a.w[1]) a.w[1] &= a.w[1] - 1u;
    else if (a.w[2]) a.w[2] &= a.w[2] - 1u;
    else a.w[3] &= a.w[3] - 1u;
}

// the rows of a [T, K] table can be read 16 bytes at a time
__device__ __forceinline__ bool rows_are_wide(const int32_t *table, int K)
{
    return (K & 3) == 0 && (reinterpret_cast<uintptr_t>(table) & 15) == 0;
}

__device__ __forceinline__ void mask_add(Mask &m, int e, int N)
{
    const uint32_t bit = (uint32_t)e < (uint32_t)N ? 1u << (e & 31) : 0u;      // ids outside [0, N) are ignored
#pragma unroll
    for (int q = 0; q < 4; ++q) m.w[q] |= (e >> 5) == q ? bit : 0u;
}

// set of the distinct ids of one step
__device__ __forceinline__ Mask step_mask(const int32_t *__restrict__ row, int K, int N, bool wide)
{
    Mask m{};
    if (wide) {
        for (int j = 0; j < K; j += 4) {
            const int4 v = *reinterpret_cast<const int4 *>(row + j);
            mask_add(m, v.x, N);
            mask_add(m, v.y, N);
            mask_add(m, v.z, N);
            mask_add(m, v.w, N);
        }
    } else {
        for (int j = 0; j < K; ++j) mask_add(m, row[j], N);
    }
    return m;
}

}  // namespace remoe
