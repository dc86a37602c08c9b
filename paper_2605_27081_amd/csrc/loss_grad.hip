// Gradient of ReMoE's router regularisers with respect to the router logits, and the gate gradient
// it induces (the backward half of the gate-only fine-tuning step of Sec. 4.1; losses of Sec. 4.2-4.4).
//
// Per sequence L = c0 L_Reuse + c1 L_Trust + c2 L_Smooth + c3 L_Lag + c4 L_WS (Eq. 3, 6), P_t =
// softmax(z_t).  With g = dL/dP_t (each entry of P_t taken as a free variable):
//
//   L_Reuse :  -1 / ((rho + 1e-8) (T-1) K) on the entries of E_{t-1} (t >= 2): the previous routed
//              set is a stop-gradient target (Eq. 2, 7)
//   L_Trust :  (ln P_t - ln P_t^ref + 1) / T                                            (Eq. 4-5)
//   SymKL(P, R) w.r.t. P:  phi(P, R) = (ln P - ln R + 1 - R / P) / 2, and the same with the roles
//              exchanged w.r.t. R, so every partner of P_t contributes phi(P_t, partner)   (Eq. 8)
//   L_Smooth:  partners t-1 and t+1, / (T-1)          (no stop-gradient, Sec. 4.4)     (Eq. 9)
//   L_Lag   :  partners t-d and t+d for d in D, / ((T-1) |D|)                           (Eq. 10)
//   L_WS    :  -(ln Pbar_b + 1) / (n W) for the steps of complete windows               (Eq. 11-12)
//
// and dL/dz_t = P_t (g - <P_t, g>).  Entries with P_t[k] = 0 get 0.  The gate gradient of a router
// without bias (Sec. 3.1) is dL/dW_r = sum_t dz_t x_t^T.
//
// loss_window_log_kernel: ln of the window means (fp64), one workgroup per window.
// loss_grad_kernel: blocks of consecutive steps whose logarithms, and those of the partners on both
//   sides, lie in LDS (loss_rows.h); one wavefront per step, lane l holding experts l and l + 64; fp64
//   arithmetic from the fp32 probabilities, fp32 result.  8 sequences x 2048 steps, 64 experts, |D| = 5:
//   81 us + 19 us for the window logarithms at first, 23 us + 5 us with the logarithms in LDS, 21 us with the probabilities
//   beside them (16 x 4096 steps, 128 experts: 195 -> 140 us for both).
// gate_grad_bf16_kernel (bf16 hidden states): dz^T x on the bf16 matrix cores.  x is exact in bf16; each fp32
//   dz is split into three bf16 pieces (hi + mid + lo, 24+ significand bits in all), so that every product is
//   exact in fp32 and the sums are fp32, as with fp32 instructions but at a fifth of their matrix time.  The
//   reduction runs over tokens, the slow index of both operands: a lane reads its own column of eight token rows
//   (4-byte loads, 128 contiguous bytes per half wavefront and row) and packs neighbouring tokens in registers; for
//   x every 4-byte load is two neighbouring columns, which belong to two MFMA column tiles.  A wavefront owns
//   64 experts x 128 hidden columns for a range of tokens; the four wavefronts
//   of a workgroup add their accumulators through LDS and gate_grad_reduce_kernel adds the workgroups' tiles,
//   both in a fixed order.  16,384 tokens, 64 experts, H 2048: 61 + 9 us with fp32 MFMAs, 27 + 5 us now.
// gate_grad_partial_kernel (fp32 hidden states): the same on the fp32 matrix cores (v_mfma_f32_32x32x2_f32), both
//   operands read from global memory directly in the instruction's operand layout (lane (i, k) takes
//   dz[t0 + k][e0 + i] and x[t0 + k][h0 + i]: 32 consecutive floats per half wavefront).
#include "common.h"
#include "loss_rows.h"

namespace remoe {

namespace {

struct GradArgs {
    const float *probs, *probs_ref;
    const int32_t *idx;
    const double *loss_values;          // [S, 6]: rho at [s, 0]
    int64_t T;
    int N, K, n_lags, window;
    int lags[8];
    double coef[5];
    RowBlocks blk;
    double *logbar;                     // [S, n_win, N]
    float *dlogits;                     // [S, T, N]
};

__global__ __launch_bounds__(LR_WAVES * 64) void loss_window_log_kernel(const GradArgs a)
{
    __shared__ double part[LR_WAVES * 128];
    const int lane = threadIdx.x;
    const int64_t s = blockIdx.y, b = blockIdx.x, n_win = a.T / a.window;
    const int N = a.N;
    double m0, m1;
    window_mean(a.probs + s * a.T * N, b * a.window, a.window, N, part, m0, m1);
    double *o = a.logbar + (s * n_win + b) * N;
    if (lane >= 64) return;              // the means are in wavefront 0
    if (lane < N) o[lane] = log(m0);
    if (lane + 64 < N) o[lane + 64] = log(m1);
}

template <int HALVES>        // (up to 64 experts: registers for three workgroups on a compute unit, where their LDS leaves room for them)
__global__ __launch_bounds__(LR_WAVES * 64, HALVES == 1 ? 6 : 4) void loss_grad_kernel(const GradArgs a)
{
    extern __shared__ double logs[];
    __shared__ double2 table[LT_BINS];
    float *const vals = reinterpret_cast<float *>(logs + a.blk.rows * a.N);
    fill_log_table(table);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t s = blockIdx.y;
    const int N = a.N, K = a.K;
    const int64_t T = a.T;
    const float *P = a.probs + s * T * N, *Q = a.probs_ref + s * T * N;
    const int32_t *E = a.idx + s * T * K;
    const int64_t n_win = T / a.window;
    const double rho = a.loss_values[s * 6];
    const double c_reuse = T > 1 ? a.coef[0] * -1.0 / ((rho + 1e-8) * (double)(T - 1) * (double)K) : 0.0;
    const double c_trust = a.coef[1] / (double)T;
    const double c_smooth = T > 1 ? 0.5 * a.coef[2] / (double)(T - 1) : 0.0;
    const double c_lag = T > 1 && a.n_lags > 0 ? 0.5 * a.coef[3] / ((double)(T - 1) * (double)a.n_lags) : 0.0;
    const double c_ws = n_win > 0 ? a.coef[4] / ((double)n_win * (double)a.window) : 0.0;

    const int64_t b0 = (int64_t)blockIdx.x * a.blk.steps, b1 = b0 + a.blk.steps < T ? b0 + a.blk.steps : T;
    const int64_t r0 = b0 > a.blk.halo ? b0 - a.blk.halo : 0, r1 = b1 + a.blk.halo < T ? b1 + a.blk.halo : T;
    __syncthreads();
    stage_rows<4>(P, r0, r1, N, table, logs, vals);
    __syncthreads();
    // what the wavefront's next step reads from memory is on its way during this one
    float ref[HALVES];
    double bar[HALVES];
    int ids = 0;
    auto request = [&](int64_t t) {
        if (t >= b1) t = b1 - 1;
        const int64_t b = t / a.window;
#pragma unroll
        for (int h = 0; h < HALVES; ++h) {
            const int e = lane + 64 * h < N ? lane + 64 * h : N - 1;
            ref[h] = Q[t * N + e];
            if (b < n_win) bar[h] = a.logbar[(s * n_win + b) * N + e];
        }
        if (t >= 1 && lane < K) ids = E[(t - 1) * K + lane];
    };
    request(b0 + wave);
    for (int64_t t = b0 + wave; t < b1; t += LR_WAVES) {
        double p[HALVES], g[HALVES];
        const int64_t b = t / a.window;
        const int row = (int)(t - r0) * N, before = ids;
        float q[HALVES];
        double lbar[HALVES];
#pragma unroll
        for (int h = 0; h < HALVES; ++h) {
            q[h] = ref[h];
            lbar[h] = bar[h];
        }
        request(t + LR_WAVES);
#pragma unroll
        for (int h = 0; h < HALVES; ++h) {
            const int e = lane + 64 * h;
            p[h] = 0.0;
            g[h] = 0.0;
            if (e >= N) continue;
            p[h] = (double)vals[row + e];
            if (!(p[h] > 0.0)) continue;
            const double lp = logs[row + e], inv = 1.0 / p[h];
            // 2 phi(P_t, R) = ln P_t - ln R + 1 - R / P_t for the partner step t + by
            auto phi2 = [&](int by, bool near) {
                float r;
                double lr;
                if (near) {
                    r = vals[row + by * N + e];
                    lr = logs[row + by * N + e];
                } else {
                    r = P[(t + by) * N + e];
                    lr = log_f32(r, table);
                }
                return lp - lr + 1.0 - (double)r * inv;
            };
            double sm = 0.0, lg = 0.0;
            if (t >= 1) sm += phi2(-1, true);
            if (t + 1 < T) sm += phi2(1, true);
            for (int i = 0; i < a.n_lags; ++i) {
                const int d = a.lags[i];
                if (d == 1) { lg += sm; continue; }
                const bool near = d <= a.blk.halo;
                if (t - d >= 0) lg += phi2(-d, near);
                if (t + d < T) lg += phi2(d, near);
            }
            g[h] = c_trust * (lp - log_f32(q[h], table) + 1.0) + c_smooth * sm + c_lag * lg;
            if (b < n_win) g[h] -= c_ws * (lbar[h] + 1.0);
        }
        if (t >= 1)
            for (int j = 0; j < K; ++j) {
                const int e = __builtin_amdgcn_readlane(before, j);
#pragma unroll
                for (int h = 0; h < HALVES; ++h)
                    if (e == lane + 64 * h && p[h] > 0.0) g[h] += c_reuse;
            }
        double dot = 0.0;
#pragma unroll
        for (int h = 0; h < HALVES; ++h) dot += p[h] * g[h];      // g = 0 where P = 0; a NaN goes into every entry of its step
        dot = wsum64(dot);
        float *o = a.dlogits + (s * T + t) * N;
#pragma unroll
        for (int h = 0; h < HALVES; ++h)
            if (lane + 64 * h < N) o[lane + 64 * h] = (float)(p[h] * (g[h] - dot));
    }
}

// ---- gate gradient ---------------------------------------------------------------------------------

constexpr int GG_NH = 2;                // 32-column tiles of hidden per wavefront
constexpr int GG_COLS = GG_NH * 32;     // hidden columns per workgroup
constexpr int GG_MAX_NE = 4;            // 32-row tiles of experts (N <= 128)
constexpr int GG_WAVES = 4;

struct GateArgs {
    const float *dz;                    // [T, N]
    const void *x;                      // [T, H] bf16 or fp32
    int64_t T;
    int N, H, chunks;
    float *partial;                     // [chunks, N, H]
    float *dw;                          // [N, H]
};

// loads through pointers known to point to device memory (global, not flat, address space)
__device__ __forceinline__ float load_global_f32(const void *p) { return *(const __attribute__((address_space(1))) float *)p; }
// two neighbouring bf16 values (the row they lie in need not be 4-byte aligned)
__device__ __forceinline__ uint32_t load_global_bf16x2(const void *p)
{
    typedef uint32_t __attribute__((aligned(2))) u32_a2;
    return *(const __attribute__((address_space(1))) u32_a2 *)p;
}

// The tokens [t_lo, t_hi) of a wavefront: the workgroup's chunk in equal parts, a multiple of `unit` each.
__device__ __forceinline__ void wave_tokens(const GateArgs &a, int chunk, int wave, int unit, int64_t &t_lo, int &n_tok)
{
    const int64_t per_wg = (a.T + a.chunks - 1) / a.chunks;
    const int64_t per_wave = ((per_wg + GG_WAVES - 1) / GG_WAVES + unit - 1) / unit * unit;
    const int64_t wg_lo = chunk * per_wg, wg_hi = (wg_lo + per_wg < a.T) ? wg_lo + per_wg : a.T;
    t_lo = wg_lo + wave * per_wave;
    const int64_t t_hi = t_lo + per_wave < wg_hi ? t_lo + per_wave : wg_hi;
    n_tok = (int)(t_hi > t_lo ? t_hi - t_lo : 0);
}

// Adds the four wavefronts' accumulators in wavefront order (one at a time through one LDS buffer: a small
// footprint lets several workgroups share a compute unit); wavefront 0 ends with the sum.
template <int TILES>
__device__ __forceinline__ void sum_waves(floatx16_t (&acc)[TILES], float *red, int wave, int lane)
{
    for (int w = 1; w < GG_WAVES; ++w) {
        if (wave == w) {
#pragma unroll
            for (int i = 0; i < TILES; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) red[(i * 16 + r) * 64 + lane] = acc[i][r];
        }
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int i = 0; i < TILES; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][r] += red[(i * 16 + r) * 64 + lane];
        }
        __syncthreads();
    }
}

// NE: 32-row tiles of experts; NP: pairs of 32-column tiles (64 hidden columns each)
template <int NE, int NP>
__global__ __launch_bounds__(GG_WAVES * 64, 2) void gate_grad_bf16_kernel(const GateArgs a)
{
    __shared__ float red[NE * NP * 2 * 16 * 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 31, lh = lane >> 5;
    const int h0 = blockIdx.x * NP * 64, e0 = blockIdx.z * NE * 32;
    const int N = a.N, H = a.H;
    floatx16_t acc[NE * NP * 2];
#pragma unroll
    for (int i = 0; i < NE * NP * 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;

    int64_t t_lo;
    int n_tok;
    wave_tokens(a, blockIdx.y, wave, 16, t_lo, n_tok);
    const char *dz_w = reinterpret_cast<const char *>(a.dz + t_lo * N);
    const char *x_w = reinterpret_cast<const char *>(static_cast<const bf16_t *>(a.x) + t_lo * H + h0);
    uint32_t dz_col[NE], x_col[NP];
    float live_e[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const int col = e0 + e * 32 + li;
        dz_col[e] = (uint32_t)(col < N ? col : N - 1) * 4u;
        live_e[e] = col < N ? 1.0f : 0.f;
    }
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int col = h0 + p * 64 + 2 * li < H ? p * 64 + 2 * li : 0;      // a ragged last block: columns past H are not stored
        x_col[p] = (uint32_t)col * 2u;
    }

    // 16 tokens per pass: the lane's eight are 16 i + 8 lh + {0..7}.  Tokens past the end repeat the last
    // one with a factor 0 on dz; the loads of the next pass are in flight during the MFMAs of this one.
    float dv[NE][8];
    uint32_t xv[NP][8];
#define GB_LOAD(i)                                                                                              \
    _Pragma("unroll") for (int j = 0; j < 8; ++j) {                                                             \
        const int t_ = 16 * (i) + 8 * lh + j;                                                                   \
        const uint32_t tc_ = (uint32_t)(t_ < n_tok ? t_ : n_tok - 1);                                           \
        _Pragma("unroll") for (int e = 0; e < NE; ++e) dv[e][j] = load_global_f32(dz_w + tc_ * (uint32_t)N * 4u + dz_col[e]); \
        _Pragma("unroll") for (int p = 0; p < NP; ++p) xv[p][j] = load_global_bf16x2(x_w + tc_ * (uint32_t)H * 2u + x_col[p]);    \
    }
    const int passes = (n_tok + 15) >> 4;
    if (passes > 0) { GB_LOAD(0) }
#pragma unroll 1
    for (int i = 0; i < passes; ++i) {
        u32x4_t piece[NE][3], col[NP][2];
        const int left = n_tok - 16 * i - 8 * lh;             // live tokens of this lane's eight
#pragma unroll
        for (int e = 0; e < NE; ++e)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float w0 = 2 * q < left ? dv[e][2 * q] * live_e[e] : 0.f, w1 = 2 * q + 1 < left ? dv[e][2 * q + 1] * live_e[e] : 0.f;
                const uint32_t hi = pack_bf16x2(w0, w1);
                const float r0 = w0 - __uint_as_float(hi << 16), r1 = w1 - __uint_as_float(hi & 0xFFFF0000u);
                const uint32_t mid = pack_bf16x2(r0, r1);
                piece[e][0][q] = hi;
                piece[e][1][q] = mid;
                piece[e][2][q] = pack_bf16x2(r0 - __uint_as_float(mid << 16), r1 - __uint_as_float(mid & 0xFFFF0000u));
            }
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                col[p][0][q] = __builtin_amdgcn_perm(xv[p][2 * q + 1], xv[p][2 * q], 0x05040100u);       // low halves: column 2 li
                col[p][1][q] = __builtin_amdgcn_perm(xv[p][2 * q + 1], xv[p][2 * q], 0x07060302u);       // high halves: column 2 li + 1
            }
        __builtin_amdgcn_sched_barrier(0);
        if (i + 1 < passes) { GB_LOAD(i + 1) }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int pc = 0; pc < 3; ++pc)
#pragma unroll
            for (int e = 0; e < NE; ++e)
#pragma unroll
                for (int p = 0; p < NP * 2; ++p)
                    acc[e * NP * 2 + p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, piece[e][pc]),
                                                                                 __builtin_bit_cast(bf16x8_t, col[p >> 1][p & 1]),
                                                                                 acc[e * NP * 2 + p], 0, 0, 0);
    }
#undef GB_LOAD
    sum_waves(acc, red, wave, lane);
    if (wave == 0) {
        float *out = a.partial + (int64_t)blockIdx.y * N * H;
#pragma unroll
        for (int e = 0; e < NE; ++e)
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = e0 + e * 32 + (r >> 2) * 8 + lh * 4 + (r & 3), c = h0 + p * 64 + 2 * li;     // expert, first column
                    if (row < N && c < H)
                        *reinterpret_cast<float2 *>(out + (int64_t)row * H + c) =
                            make_float2(acc[e * NP * 2 + 2 * p][r], acc[e * NP * 2 + 2 * p + 1][r]);
                }
    }
}

template <int NE>
__global__ __launch_bounds__(GG_WAVES * 64) void gate_grad_partial_kernel(const GateArgs a)
{
    __shared__ float red[NE * GG_NH * 16 * 64];   // one wavefront's accumulators at a time
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 31, lh = lane >> 5;
    const int h0 = blockIdx.x * GG_COLS;
    const int chunk = blockIdx.y;
    const int N = a.N, H = a.H;
    const float *x = static_cast<const float *>(a.x);

    floatx16_t acc[NE][GG_NH];
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
        for (int n = 0; n < GG_NH; ++n)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[e][n][r] = 0.f;

    int64_t t_lo;
    int n_tok;
    wave_tokens(a, chunk, wave, 2, t_lo, n_tok);       // an even number per wavefront so that token pairs never straddle

    // GG_UN token pairs per pass.  The operand loads of the next pass are issued before the MFMAs of
    // the current one (two register sets), so that a wavefront alone on its SIMD still overlaps load
    // latency with matrix-core work.  Loads are unconditional (clamped indices) and masked by a
    // multiplication: a conditional load is a branch, and behind every branch the compiler waits for
    // all loads in flight.  (What a masked load reads is other tokens' or experts' data of the same call.)
    constexpr int GG_UN = 2;
    const int n_pairs = (n_tok + 1) >> 1;
    const char *dz_w = reinterpret_cast<const char *>(a.dz + t_lo * N);
    const char *x_w = reinterpret_cast<const char *>(x + t_lo * H + h0);
    uint32_t dz_col[NE];
    float col_live[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const int col = e * 32 + li;
        dz_col[e] = (uint32_t)(col < N ? col : N - 1) * 4u;
        col_live[e] = col < N ? 1.0f : 0.f;
    }
#define GG_LOAD(av, bv, first_pair)                                                                      \
    _Pragma("unroll") for (int u = 0; u < GG_UN; ++u) {                                                  \
        const int t_ = 2 * ((first_pair) + u) + lh;      /* k index of the instruction = which token of the pair */ \
        const int tc_ = t_ < n_tok ? t_ : n_tok - 1;                                                     \
        _Pragma("unroll") for (int e = 0; e < NE; ++e)                                                   \
            av[u][e] = load_global_f32(dz_w + (uint32_t)(tc_ * N) * 4u + dz_col[e]);                     \
        _Pragma("unroll") for (int n = 0; n < GG_NH; ++n)                                                \
            bv[u][n] = load_global_f32(x_w + (uint32_t)(tc_ * H + n * 32 + li) * 4u);                     \
    }
    // the masks are applied here, not where the values are requested: a use right behind a load is a wait
#define GG_MFMA(av, bv, first_pair)                                                                      \
    _Pragma("unroll") for (int u = 0; u < GG_UN; ++u) {                                                  \
        const float live_ = (2 * ((first_pair) + u) + lh < n_tok) ? 1.0f : 0.f;                          \
        _Pragma("unroll") for (int e = 0; e < NE; ++e)                                                   \
            _Pragma("unroll") for (int n = 0; n < GG_NH; ++n)                                            \
                acc[e][n] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[u][e] * col_live[e], bv[u][n] * live_, acc[e][n], 0, 0, 0); \
    }
    if (n_tok > 0) {
        float avA[GG_UN][NE], bvA[GG_UN][GG_NH], avB[GG_UN][NE], bvB[GG_UN][GG_NH];
        GG_LOAD(avA, bvA, 0)
#pragma unroll 1
        for (int i = 0; i < n_pairs; i += 2 * GG_UN) {
            __builtin_amdgcn_sched_barrier(0);
            GG_LOAD(avB, bvB, i + GG_UN)                 // past the end: clamped and masked to zero
            __builtin_amdgcn_sched_barrier(0);
            GG_MFMA(avA, bvA, i)
            __builtin_amdgcn_sched_barrier(0);
            GG_LOAD(avA, bvA, i + 2 * GG_UN)
            __builtin_amdgcn_sched_barrier(0);
            GG_MFMA(avB, bvB, i + GG_UN)
        }
    }
#undef GG_LOAD
#undef GG_MFMA

    sum_waves(reinterpret_cast<floatx16_t (&)[NE * GG_NH]>(acc), red, wave, lane);
    if (wave == 0) {
        float *out = a.partial + (int64_t)chunk * N * H;
#pragma unroll
        for (int e = 0; e < NE; ++e)
#pragma unroll
            for (int n = 0; n < GG_NH; ++n)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = e * 32 + (r >> 2) * 8 + lh * 4 + (r & 3);     // expert
                    if (row < N) out[(int64_t)row * H + h0 + n * 32 + li] = acc[e][n][r];
                }
    }
}

// FROM_BF16: an infinite dz, or one that rounds to infinity in bf16 (about 3.4e38 and more), leaves inf - inf in its
// pieces and so a NaN in its expert's sums.  A sum that is NaN is therefore taken again from the values themselves (in
// fp64, up to the first NaN).  Looking for such dz while they are split costs 1.6 of 27 us, walking the tokens a second time
// in the kernel above 10 us (registers).
template <bool FROM_BF16>
__global__ void gate_grad_reduce_kernel(const GateArgs a)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t total = (int64_t)a.N * a.H;
    if (q >= total) return;
    float v = 0.f;
#pragma unroll 8
    for (int c = 0; c < a.chunks; ++c) v += a.partial[(int64_t)c * total + q];
    if (FROM_BF16 && v != v) {
        const float *dz = a.dz + q / a.H;
        const bf16_t *x = static_cast<const bf16_t *>(a.x) + q % a.H;
        double sum = 0.0;
        for (int64_t t = 0; t < a.T && sum == sum; ++t) sum += (double)dz[t * a.N] * (double)__uint_as_float((uint32_t)x[t * a.H] << 16);
        v = (float)sum;
    }
    a.dw[q] = v;
}

int gate_grad_chunks(int64_t T, int H)
{
    // about four workgroups per compute unit at the widest hidden sizes, at least 64 tokens each
    int64_t c = 1024 / (H / GG_COLS > 0 ? H / GG_COLS : 1);
    if (c < 1) c = 1;
    if (c > 64) c = 64;
    while (c > 1 && T / c < 64) c >>= 1;
    return (int)c;
}

}  // namespace

size_t loss_backward_workspace_bytes(int64_t S, int64_t T, int N, int window)
{
    const int64_t n_win = window > 0 ? T / window : 0;
    return align_up(sizeof(double) * (size_t)(S * n_win * N) + 8, 256);
}

remoe_status launch_loss_backward(const float *probs, const float *probs_ref, const int32_t *idx, int64_t S, int64_t T,
                                  int N, int K, const int32_t *lags, int n_lags, int window, const double *coef,
                                  const double *loss_values, float *dlogits, void *workspace, hipStream_t stream)
{
    if (S == 0 || T == 0) return REMOE_OK;
    if (S > 65535) return fail(REMOE_E_UNSUPPORTED, "remoe_loss_backward handles at most 65535 sequences per call (got %lld)", (long long)S);
    GradArgs a;
    a.probs = probs; a.probs_ref = probs_ref; a.idx = idx; a.loss_values = loss_values;
    a.T = T; a.N = N; a.K = K; a.n_lags = n_lags; a.window = window;
    for (int i = 0; i < 8; ++i) a.lags[i] = i < n_lags ? lags[i] : 0;
    for (int i = 0; i < 5; ++i) a.coef[i] = coef[i];
    a.logbar = static_cast<double *>(workspace);
    a.dlogits = dlogits;
    a.blk = plan_rows(N, lags, n_lags, 2);
    const int64_t n_win = T / window;
    if (n_win > 0) {
        if (n_win > 0x7FFFFFFF) return fail(REMOE_E_UNSUPPORTED, "too many windows");
        hipLaunchKernelGGL(loss_window_log_kernel, dim3((unsigned)n_win, (unsigned)S), dim3(LR_WAVES * 64), 0, stream, a);
    }
    // short blocks where the sequences alone do not fill the chip: at least 8 steps (one per wavefront), as many
    // workgroups as are resident at once
    const int64_t want = ceil_div(512, S);
    int64_t steps = ceil_div(ceil_div(T, want), LR_WAVES) * LR_WAVES;
    if (steps < a.blk.steps) a.blk.steps = (int)steps;
    a.blk.rows = a.blk.steps + 2 * a.blk.halo;
    const dim3 grid((unsigned)ceil_div(T, a.blk.steps), (unsigned)S), block(LR_WAVES * 64);
    const size_t lds = (size_t)LR_ENTRY * a.blk.rows * N;
    if (N <= 64) hipLaunchKernelGGL(loss_grad_kernel<1>, grid, block, lds, stream, a);
    else hipLaunchKernelGGL(loss_grad_kernel<2>, grid, block, lds, stream, a);
    return check_hip(hipGetLastError(), "loss gradient kernels launch");
}

size_t gate_grad_workspace_bytes(int64_t T, int N, int H)
{
    return align_up(sizeof(float) * (size_t)gate_grad_chunks(T, H) * (size_t)N * (size_t)H, 256);
}

remoe_status launch_gate_grad(const float *dz, const void *x, int x_dtype, int64_t T, int N, int H, float *dw, void *workspace,
                              hipStream_t stream)
{
    if (H % GG_COLS != 0) return fail(REMOE_E_UNSUPPORTED, "remoe_gate_grad needs hidden %% %d == 0 (got %d)", GG_COLS, H);
    if (N > GG_MAX_NE * 32) return fail(REMOE_E_UNSUPPORTED, "remoe_gate_grad handles at most %d experts", GG_MAX_NE * 32);
    GateArgs a;
    a.dz = dz; a.x = x; a.T = T; a.N = N; a.H = H;
    a.chunks = gate_grad_chunks(T, H);
    a.partial = static_cast<float *>(workspace);
    a.dw = dw;
    const dim3 block(GG_WAVES * 64);
    const int ne = (N + 31) / 32;
    if (x_dtype == REMOE_BF16) {
        // more than 64 experts in two passes over x: four expert tiles with both operands' next loads do not fit the registers
        const dim3 grid((unsigned)ceil_div(H, 128), (unsigned)a.chunks, (unsigned)ceil_div(ne, 2));
        if (ne == 1) hipLaunchKernelGGL((gate_grad_bf16_kernel<1, 2>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((gate_grad_bf16_kernel<2, 2>), grid, block, 0, stream, a);
    } else {
        const dim3 grid((unsigned)(H / GG_COLS), (unsigned)a.chunks);
        switch (ne) {
        case 1: hipLaunchKernelGGL(gate_grad_partial_kernel<1>, grid, block, 0, stream, a); break;
        case 2: hipLaunchKernelGGL(gate_grad_partial_kernel<2>, grid, block, 0, stream, a); break;
        case 3: hipLaunchKernelGGL(gate_grad_partial_kernel<3>, grid, block, 0, stream, a); break;
        default: hipLaunchKernelGGL(gate_grad_partial_kernel<4>, grid, block, 0, stream, a); break;
        }
    }
    const int64_t total = (int64_t)N * H;
    auto reduce = x_dtype == REMOE_BF16 ? gate_grad_reduce_kernel<true> : gate_grad_reduce_kernel<false>;
    hipLaunchKernelGGL(reduce, dim3((unsigned)ceil_div(total, 256)), dim3(256), 0, stream, a);
    return check_hip(hipGetLastError(), "gate gradient kernels launch");
}

}  // namespace remoe
