// Forward values of ReMoE's router regularisers on a batch of routing distributions (Sec. 4.2-4.4):
//
//   m_t      = (1/K) sum_{k in E_{t-1}} P_t[k]                               (Eq. 2, reuse mass)
//   rho      = mean_{t>=2} m_t,   L_Reuse = -log(rho + 1e-8)                 (Eq. 7)
//   L_Trust  = mean_t KL(P_t || P_t^ref)                                     (Eq. 4-5)
//   L_Smooth = mean_{t>=2} SymKL(P_t, P_{t-1})                               (Eq. 8-9)
//   L_Lag    = mean_{t>=2} (1/|D|) sum_{d in D, t-d>=1} SymKL(P_t, P_{t-d})  (Eq. 10)
//   L_WS     = mean_b H(mean of the W distributions of window b)             (Eq. 11-12)
//
// per sequence.  The inputs are the fp32 probabilities the router kernel writes; everything here is
// computed in fp64 (the work is ~7 N logarithms per step, nothing next to the expert GEMMs), with
// SymKL(P,Q) = (1/2) sum_k (P[k] - Q[k]) (ln P[k] - ln Q[k]).
//
// loss_partial_kernel: grid (chunk, sequence); a workgroup walks its chunk of steps in blocks whose
// logarithms lie in LDS (loss_rows.h), a wavefront per step with lane l holding experts l and l + 64, and
// then its chunk of the windows; per-wavefront fp64 sums are combined in wavefront order and written to
// the workspace.  loss_final_kernel adds the chunks of a sequence (a lane per chunk, fixed order) and applies the
// normalisations, so results repeat bit for bit.
//
// Bound by the fp64 logarithms: (1 + halo / steps) + 1 per entry instead of the 2 + |D| of a step that computes
// its partners' itself.  8 sequences x 2048 steps, 64 experts, |D| = 5: 130 us at first, 22 us with the logarithms in LDS, 17 us with the
// probabilities beside them (16 x 4096 steps, 128 experts: 114 -> 78 us).
#include "common.h"
#include "loss_rows.h"

namespace remoe {

namespace {

constexpr int LS_CHUNKS = 64;           // chunks of steps (and of windows) per sequence, a lane each in the last sum
constexpr int LS_TERMS = 5;             // sum m_t, sum KL, sum SymKL adjacent, sum lag term, sum window entropy

// this lane's share of KL(a || b): a ln(a / b), 0 where a = 0 (ln b = -inf where b = 0)
__device__ __forceinline__ double kl_part(double a, double la, double lb) { return a > 0.0 ? a * (la - lb) : 0.0; }

// ... of SymKL(a, b) = (1/2) (a - b) (ln a - ln b), 0 where a = b
__device__ __forceinline__ double symkl_part(double a, double la, double b, double lb)
{
    return a == b ? 0.0 : 0.5 * (a - b) * (la - lb);
}

struct LossArgs {
    const float *probs, *probs_ref;
    const int32_t *idx;
    int64_t T;
    int N, K, n_lags, window;
    int lags[8];
    RowBlocks blk;
    double *partial;                    // [S, LS_CHUNKS, LS_TERMS]
    double *out;                        // [S, 6]
};

// HALVES: 64-expert halves of a row.  MANY: registers for four workgroups on a compute unit (three for two halves) at the cost of a slower
// staging of the rows, where the LDS of one leaves room for three and more.  With the registers of two everywhere, few experts or short
// chunks had half of the wavefronts: 32 sequences x 1024 steps, 32 experts, 5 lags 39 us, now 30; 64 x 512 steps, 64 experts 69 and 49.
template <int HALVES, bool MANY>
__global__ __launch_bounds__(LR_WAVES * 64, !MANY ? 4 : HALVES == 1 ? 8 : 6) void loss_partial_kernel(const LossArgs a)
{
    extern __shared__ double logs[];
    __shared__ double part[LR_WAVES][LS_TERMS];
    __shared__ double2 table[LT_BINS];
    float *const vals = reinterpret_cast<float *>(logs + a.blk.rows * a.N);
    const int chunk = blockIdx.x;
    const int64_t s = blockIdx.y;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int N = a.N, K = a.K;
    const int64_t T = a.T;
    const float *P = a.probs + s * T * N, *Q = a.probs_ref + s * T * N;
    const int32_t *E = a.idx + s * T * K;
    double acc[LS_TERMS] = {0.0, 0.0, 0.0, 0.0, 0.0};
    fill_log_table(table);
    int unit = -1;                      // the lag that is L_Smooth's partner too (the first one, should it be given twice)
    for (int i = a.n_lags - 1; i >= 0; --i)
        if (a.lags[i] == 1) unit = i;

    const int64_t per = (T + LS_CHUNKS - 1) / LS_CHUNKS;
    const int64_t t_lo = chunk * per, t_hi = (t_lo + per < T) ? t_lo + per : T;
    for (int64_t b0 = t_lo; b0 < t_hi; b0 += a.blk.steps) {
        const int64_t b1 = b0 + a.blk.steps < t_hi ? b0 + a.blk.steps : t_hi;
        const int64_t r0 = b0 > a.blk.halo ? b0 - a.blk.halo : 0;
        __syncthreads();                // the block before is done with the LDS
        stage_rows<!MANY ? 4 : HALVES == 1 ? 1 : 2>(P, r0, b1, N, table, logs, vals);
        __syncthreads();
        // the reference row and the requests of the wavefront's next step are on their way during this one
        float ref[HALVES];
        int id = 0;
        auto request = [&](int64_t t) {
            if (t >= b1) t = b1 - 1;
#pragma unroll
            for (int h = 0; h < HALVES; ++h) ref[h] = Q[t * N + (lane + 64 * h < N ? lane + 64 * h : N - 1)];
            if (t >= 1 && lane < K) id = E[(t - 1) * K + lane];
        };
        request(b0 + wave);
        for (int64_t t = b0 + wave; t < b1; t += LR_WAVES) {
            const int row = (int)(t - r0) * N;
            float q[HALVES];
#pragma unroll
            for (int h = 0; h < HALVES; ++h) q[h] = ref[h];
            const int before = id;
            request(t + LR_WAVES);
            if (t >= 1 && lane < K) acc[0] += (double)vals[row + before];
#pragma unroll
            for (int h = 0; h < HALVES; ++h) {
                const int e = lane + 64 * h;
                if (e >= N) continue;
                const double p = (double)vals[row + e], lp = logs[row + e];
                acc[1] += kl_part(p, lp, log_f32(q[h], table));
                if (t < 1) continue;
                if (unit < 0) acc[2] += symkl_part(p, lp, (double)vals[row - N + e], logs[row - N + e]);
                for (int i = 0; i < a.n_lags; ++i) {
                    const int d = a.lags[i];
                    if (t - d < 0) continue;
                    float r;
                    double lr;
                    if (d <= a.blk.halo) {
                        r = vals[row - d * N + e];
                        lr = logs[row - d * N + e];
                    } else {
                        r = P[(t - d) * N + e];
                        lr = log_f32(r, table);
                    }
                    const double v = symkl_part(p, lp, (double)r, lr);
                    acc[3] += v;
                    if (i == unit) acc[2] += v;
                }
            }
        }
    }
    // windows of this chunk
    const int64_t n_win = T / a.window;
    const int64_t wper = (n_win + LS_CHUNKS - 1) / LS_CHUNKS;
    const int64_t w_lo = chunk * wper, w_hi = (w_lo + wper < n_win) ? w_lo + wper : n_win;
    __syncthreads();
    for (int64_t b = w_lo; b < w_hi; ++b) {
        double m0, m1;
        window_mean(P, b * a.window, a.window, N, logs, m0, m1);
        if (wave == 0) acc[4] -= (m0 > 0.0 ? m0 * log(m0) : 0.0) + (m1 > 0.0 ? m1 * log(m1) : 0.0);
    }
#pragma unroll
    for (int k = 0; k < LS_TERMS; ++k) {
        const double v = wsum64(acc[k]);
        if (lane == 0) part[wave][k] = v;
    }
    __syncthreads();
    if (threadIdx.x < LS_TERMS) {
        double v = 0.0;
        for (int w = 0; w < LR_WAVES; ++w) v += part[w][threadIdx.x];
        a.partial[(s * LS_CHUNKS + chunk) * LS_TERMS + threadIdx.x] = v;
    }
}

// one wavefront per sequence, a lane per chunk
__global__ __launch_bounds__(64) void loss_final_kernel(const LossArgs a)
{
    const int64_t s = blockIdx.x;
    const int lane = threadIdx.x;
    double sum[LS_TERMS];
#pragma unroll
    for (int k = 0; k < LS_TERMS; ++k) sum[k] = wsum64(a.partial[(s * LS_CHUNKS + lane) * LS_TERMS + k]);
    if (lane != 0) return;
    const int64_t T = a.T;
    const double pairs = T > 1 ? (double)(T - 1) : 1.0;
    const int64_t n_win = T / a.window;
    const double rho = T > 1 ? sum[0] / (double)a.K / pairs : 0.0;
    double *o = a.out + s * 6;
    o[0] = rho;
    o[1] = -log(rho + 1e-8);
    o[2] = T > 0 ? sum[1] / (double)T : 0.0;
    o[3] = T > 1 ? sum[2] / pairs : 0.0;
    o[4] = (T > 1 && a.n_lags > 0) ? sum[3] / (double)a.n_lags / pairs : 0.0;
    o[5] = n_win > 0 ? sum[4] / (double)n_win : 0.0;
}

}  // namespace

size_t loss_workspace_bytes(int64_t S) { return align_up(sizeof(double) * (size_t)S * LS_CHUNKS * LS_TERMS, 256); }

remoe_status launch_loss_forward(const float *probs, const float *probs_ref, const int32_t *idx, int64_t S, int64_t T,
                                 int N, int K, const int32_t *lags, int n_lags, int window, double *out, void *workspace,
                                 hipStream_t stream)
{
    if (S == 0) return REMOE_OK;
    if (S > 65535) return fail(REMOE_E_UNSUPPORTED, "remoe_loss_forward handles at most 65535 sequences per call (got %lld)", (long long)S);
    LossArgs a;
    a.probs = probs; a.probs_ref = probs_ref; a.idx = idx;
    a.T = T; a.N = N; a.K = K; a.n_lags = n_lags; a.window = window;
    for (int i = 0; i < 8; ++i) a.lags[i] = i < n_lags ? lags[i] : 0;
    a.blk = plan_rows(N, lags, n_lags, 1);
    const int64_t per = ceil_div(T, LS_CHUNKS);
    if (per < a.blk.steps) {             // less LDS, more workgroups on a compute unit
        a.blk.steps = per > 0 ? (int)per : 1;
        a.blk.rows = a.blk.steps + a.blk.halo;
    }
    a.partial = static_cast<double *>(workspace);
    a.out = out;
    const size_t rows_bytes = (size_t)LR_ENTRY * a.blk.rows * N, win_bytes = sizeof(double) * LR_WAVES * 128;
    const size_t lds = rows_bytes > win_bytes ? rows_bytes : win_bytes;
    const dim3 grid(LS_CHUNKS, (unsigned)S), block(LR_WAVES * 64);
    const bool many = 3 * (lds + 2432) <= 160 * 1024;
    auto kernel = N <= 64 ? (many ? loss_partial_kernel<1, true> : loss_partial_kernel<1, false>)
                          : (many ? loss_partial_kernel<2, true> : loss_partial_kernel<2, false>);
    hipLaunchKernelGGL(kernel, grid, block, lds, stream, a);
    hipLaunchKernelGGL(loss_final_kernel, dim3((unsigned)S), dim3(64), 0, stream, a);
    return check_hip(hipGetLastError(), "loss kernels launch");
}

}  // namespace remoe
