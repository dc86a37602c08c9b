// What the loss and the loss-gradient kernels share: fp64 wavefront sums and the logarithms of a block of
// routing distributions in LDS.
#pragma once

#include "common.h"

namespace remoe {

// Sum over the 64 lanes, the same value in every lane, always in the same order.
__device__ __forceinline__ double wsum64(double v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// ---- ln of an fp32 value in fp64, to about one unit in the last place
//
// Table-driven (the method of Tang, "Table-driven implementation of the logarithm function in IEEE floating-point
// arithmetic", ACM TOMS 16, 1990): x = 2^k m with m in [0.7, 1.4); the interval is cut into 128 bins, the table
// holds a c close to 1 / m and -ln c for each, and ln x = k ln 2 - ln c + ln(1 + r) with r = m c - 1, |r| < 0.008,
// so seven terms of the series are exact to 1e-18.  Around m = 1 the table has c = 1, so that the result keeps
// its relative accuracy there.  About 20 instructions against about 100 of the library's fp64 log, which these
// kernels spent most of their time in: loss values 26 -> 22 us, loss gradient 30 -> 23 us (8 x 2048 steps, 64 experts).
constexpr uint32_t LT_FIRST = 0x3f330000u;      // 0.69921875, the lower end of m
constexpr int LT_BINS = 128;

// one entry per thread of a workgroup of at least 128; the caller synchronises
__device__ __forceinline__ void fill_log_table(double2 *table)
{
    if (threadIdx.x < LT_BINS) {
        const uint32_t lo = LT_FIRST + ((uint32_t)threadIdx.x << 16);      // 128 bins of 2^16 floats: one binade
        const bool one = lo <= 0x3f800000u && 0x3f800000u < lo + 0x10000u;
        const bool below = lo + 0x10000u == 0x3f800000u;                   // 1.0 opens a bin: its left neighbour keeps c = 1 too
        const double c = one || below ? 1.0 : 1.0 / (double)__uint_as_float(lo + 0x8000u);
        table[threadIdx.x] = make_double2(c, one || below ? 0.0 : -log(c));
    }
}

// ln p: -inf for 0, inf for inf, NaN for NaN and for p < 0 (what the hardware's logarithm says of them)
__device__ __forceinline__ double log_f32(float p, const double2 *table)
{
    uint32_t u = __float_as_uint(p);
    int k = 0;
    if (u < 0x00800000u) {                       // denormal: scaled into the normal range
        u = __float_as_uint(p * 0x1p24f);
        k = -24;
    }
    const uint32_t d = u - LT_FIRST;
    k += (int)d >> 23;
    const double m = (double)__uint_as_float(u - (d & 0xFF800000u));
    const double2 e = table[(d >> 16) & (LT_BINS - 1)];
    const double r = fma(m, e.x, -1.0);
    double q = fma(r, 1.0 / 7.0, -1.0 / 6.0);
    q = fma(r, q, 1.0 / 5.0);
    q = fma(r, q, -1.0 / 4.0);
    q = fma(r, q, 1.0 / 3.0);
    q = fma(r, q, -0.5);
    const double v = fma((double)k, 0.693147180559945309417, e.y) + fma(r * r, q, r);
    return p > 0.f && p < __builtin_inff() ? v : (double)__builtin_amdgcn_logf(p);
}

// Every logarithm a step needs belongs to its own row or to the row of a partner step t +- d, and every row is
// the partner of several steps.  A workgroup therefore takes a block of consecutive steps, computes the
// logarithms of the block's rows and of `halo` rows around it once, and keeps them in LDS as fp64
// (-inf for a zero probability), the probabilities beside them.  (Read from memory again for every partner, these kept a wavefront
// waiting a round trip to the caches per lag: 8 x 2048 steps, 64 experts, 5 lags, loss values 21.5 us, gradient 22.5.)
// Partners farther away than the halo are read and computed on the spot: with 128 experts from a lag of 34 on (17 for the gradient, whose
// halo is on both sides), with 64 experts 68 and 34.  (With 8 bytes an entry and the probabilities in memory the halo reached 40 and
// 20, 80 and 40, and these lags took longer all the same: 16 x 4096 steps, 128 experts, lags 1, 2, 4, 8 and 20, gradient 208 us, now 142; 1, 2,
// 4, 8 and 40, values 140 and 88.  90 KB, which reach as far, leave one workgroup on a compute unit: 213 and 151.)
constexpr int LR_BYTES = 76 * 1024;      // LDS for both: two workgroups per compute unit
constexpr int LR_ENTRY = sizeof(double) + sizeof(float);
constexpr int LR_WAVES = 8;
constexpr int LR_MAX_ROWS = 128;

struct RowBlocks {
    int rows;         // rows that fit the LDS
    int halo;         // rows on one side of a block
    int steps;        // steps per block
};

// sides: 1 when only earlier partners are needed, 2 for both.
inline RowBlocks plan_rows(int N, const int32_t *lags, int n_lags, int sides)
{
    RowBlocks b;
    b.rows = LR_BYTES / (LR_ENTRY * N);
    if (b.rows > LR_MAX_ROWS) b.rows = LR_MAX_ROWS;
    b.halo = 1;       // adjacent steps are always partners (L_Smooth)
    for (int i = 0; i < n_lags; ++i)
        if (lags[i] > b.halo && lags[i] <= b.rows * 2 / (3 * sides)) b.halo = lags[i];      // at least a third is steps
    b.steps = b.rows - sides * b.halo;
    return b;
}

// ln of the rows [r_lo, r_hi) of P ([T, N]) -> logs[(r - r_lo) * N + e], and the rows -> vals
template <int UNROLL>
__device__ __forceinline__ void stage_rows(const float *__restrict__ P, int64_t r_lo, int64_t r_hi, int N, const double2 *table, double *logs, float *vals)
{
    const int n = (int)(r_hi - r_lo) * N;
    const float *src = P + r_lo * N;
#pragma unroll UNROLL
    for (int q = threadIdx.x; q < n; q += LR_WAVES * 64) {
        const float v = src[q];
        vals[q] = v;
        logs[q] = log_f32(v, table);
    }
}

// Means of the windows of `window` steps, entry by entry: 8 wavefronts share one window's rows (lane = expert, a
// second half for N > 64) and are added in wavefront order.  The result is valid in wavefront 0.
__device__ __forceinline__ void window_mean(const float *__restrict__ P, int64_t t0, int window, int N, double *part, double &m0, double &m1)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    m0 = 0.0;
    m1 = 0.0;
#pragma unroll 4
    for (int j = wave; j < window; j += LR_WAVES) {
        const float *row = P + (t0 + j) * N;
        if (lane < N) m0 += (double)row[lane];
        if (lane + 64 < N) m1 += (double)row[lane + 64];
    }
    part[wave * 128 + lane] = m0;
    part[wave * 128 + 64 + lane] = m1;
    __syncthreads();
    if (wave == 0) {
        m0 = 0.0;
        m1 = 0.0;
        for (int w = 0; w < LR_WAVES; ++w) {
            m0 += part[w * 128 + lane];
            m1 += part[w * 128 + 64 + lane];
        }
        m0 /= (double)window;
        m1 /= (double)window;
    }
    __syncthreads();
}

}  // namespace remoe
