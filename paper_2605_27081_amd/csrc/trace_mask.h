// Expert sets as 128-bit masks, for the kernels that walk routing traces.
#pragma once

#include "common.h"

namespace remoe {

template <int W>
struct __attribute__((aligned(4 * W))) Set {     // W = 4, or 2 where there are no more than 64 experts
    uint32_t w[W];
    __device__ __forceinline__ Set &operator|=(const Set &o)
    {
#pragma unroll
        for (int q = 0; q < W; ++q) w[q] |= o.w[q];
        return *this;
    }
};
typedef Set<4> Mask;

template <int W> __device__ __forceinline__ Set<W> without(const Set<W> &a, const Set<W> &b)
{
    Set<W> r;
#pragma unroll
    for (int q = 0; q < W; ++q) r.w[q] = a.w[q] & ~b.w[q];
    return r;
}

template <int W> __device__ __forceinline__ bool any(const Set<W> &a)
{
    uint32_t o = a.w[0];
#pragma unroll
    for (int q = 1; q < W; ++q) o |= a.w[q];
    return o != 0u;
}

template <int W> __device__ __forceinline__ int count(const Set<W> &a)
{
    int n = 0;
#pragma unroll
    for (int q = 0; q < W; ++q) n += __popc(a.w[q]);
    return n;
}

template <int W> __device__ __forceinline__ Set<W> single(int e)
{
    Set<W> r;
#pragma unroll
    for (int q = 0; q < W; ++q) r.w[q] = (e >> 5) == q ? 1u << (e & 31) : 0u;
    return r;
}

template <int W> __device__ __forceinline__ bool holds(const Set<W> &a, int e)
{
    uint32_t in = 0u;
#pragma unroll
    for (int q = 0; q < W; ++q) in |= a.w[q] & ((e >> 5) == q ? 1u << (e & 31) : 0u);
    return in != 0u;
}

// the n lowest members leave (n may be negative: none)
template <int W> __device__ __forceinline__ void drop_lowest(Set<W> &a, int n)
{
#pragma unroll
    for (int q = 0; q < W; ++q) {
        const int c = __popc(a.w[q]);
        const bool all = c <= n;
        uint32_t v = all ? 0u : a.w[q];
        for (int k = all ? 0 : n; k > 0; --k) v &= v - 1u;
        a.w[q] = v;
        n = all ? n - c : 0;
    }
}

// the same one member at a time, for lanes that all drop a few: 768 x 4096 steps, top-8, C = 4 27.9 us, with the loops above 30.5
template <int W> __device__ __forceinline__ void drop_one_by_one(Set<W> &a, int n)
{
    for (; n > 0; --n) {
        bool open = true;
#pragma unroll
        for (int q = 0; q < W; ++q) {
            const bool here = open && a.w[q] != 0u;
            a.w[q] = here ? a.w[q] & (a.w[q] - 1u) : a.w[q];
            open = open && !here;
        }
    }
}

// the rows of a [T, K] table can be read 16 bytes at a time
__device__ __forceinline__ bool rows_are_wide(const int32_t *table, int K)
{
    return (K & 3) == 0 && (reinterpret_cast<uintptr_t>(table) & 15) == 0;
}

// The word is picked by a one-hot number, a bit of which is shifted into place: two instructions a word instead of three.
template <int W> __device__ __forceinline__ void mask_add(Set<W> &m, int e, int N)
{
    const uint32_t word = (uint32_t)e < (uint32_t)N ? 1u << (e >> 5) : 0u;      // ids outside [0, N) are ignored
#pragma unroll
    for (int q = 0; q < W; ++q) m.w[q] |= ((word >> q) & 1u) << (e & 31);
}

// set of the distinct ids of one step
template <int W = 4> __device__ __forceinline__ Set<W> step_mask(const int32_t *__restrict__ row, int K, int N, bool wide)
{
    Set<W> m{};
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
