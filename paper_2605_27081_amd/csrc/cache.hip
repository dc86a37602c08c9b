// The rest of the paper's expert-cache simulator on routing traces, and routing-balance statistics.
//
// launch_cache_policy: per-layer expert cache of capacity C under LRU, FIFO, LFU or Belady's MIN
// (App. E.2 "Cache state": the update rule depends on the policy, the hit / miss definitions do
// not; App. F.1 evaluates Belady under the same per-request resets).  Per step it reports the
// unique misses |U_t \ C_t| and the token hits against the resident set BEFORE the step, and |U_t|
// (App. E.2, "Per-step hits and misses"); per trace the totals that give #uMiss and uHR.
// The LRU cache is a function of the last requests alone and is found for every step in parallel (trace.hip).  The other policies
// carry state from step to step, so cache_policy_kernel walks a trace in order: one wavefront per trace, the resident set
// a 128-bit mask in wave-uniform registers, lane l holding the retention keys of experts l and
// l + 64.  After a step every requested expert is held; while more than C are held, the one with the
// smallest key among those the step did not request is dropped.  Keys (larger = kept longer), ending in the
// order of the ids:
//   FIFO   step of last fetch, id
//   LFU    requests so far, step of last use, id
//   Belady steps_total - step of next request, 127 - id: the next request farthest ahead goes first
// The next requests of Belady are looked up in masks of the steps that request an expert, a batch of 64 steps at a time: by
// the walk itself for a trace of one batch, else by next_use_kernel, from the last batch to the first.
//
// step_summary_kernel / step_percentile_kernel: per-step sums of a miss table over the MoE layers,
// their histogram and P50 / P95 / P99 (App. E.2, "Per-step (edge) reporting").
//
// balance_kernel: expert loads of a trace, experts used, normalised routing entropy and the
// coefficient of variation of the loads (the quantities Sec. 5.2 tracks to show that routing stays
// balanced).
#include "common.h"
#include "topk.h"

namespace remoe {

namespace {

constexpr int CP_BATCH = 64;            // steps staged in LDS at a time
constexpr uint32_t CP_NONE = 0xFFFFFFFFu;

// rows [t0, t0 + n) of a [T, K] int32 table -> LDS, coalesced
__device__ __forceinline__ void stage_rows(const int32_t *__restrict__ table, int64_t t0, int n, int K, int32_t *lds)
{
    const int lane = threadIdx.x & 63;
    for (int q = lane; q < n * K; q += 64) lds[q] = table[t0 * K + q];
}

// Belady: in a batch of n staged rows, first step after row t that requests expert ids[t, j] again -> out (may be ids itself).  when[e] is
// the set of rows that request e; behind the batch the answer is later(e).  One wavefront.
template <typename Later>
__device__ __forceinline__ void next_uses(const int32_t *ids, int n, int K, int N, int64_t t0, unsigned long long *when, int32_t *out, Later later)
{
    const int lane = threadIdx.x & 63;
    when[lane] = 0ull;
    when[lane + 64] = 0ull;
    __syncthreads();
    if (lane < n) {
        for (int j = 0; j < K; ++j) {
            const int e = ids[lane * K + j];
            if ((uint32_t)e < (uint32_t)N) atomicOr(&when[e], 1ull << lane);
        }
    }
    __syncthreads();
    if (lane < n) {
        for (int j = 0; j < K; ++j) {
            const int e = ids[lane * K + j];
            int32_t next = later(-1);
            if ((uint32_t)e < (uint32_t)N) {
                const unsigned long long ahead = when[e] >> lane >> 1;
                next = ahead ? (int32_t)(t0 + lane) + __ffsll((long long)ahead) : later(e);
            }
            out[lane * K + j] = next;
        }
    }
    __syncthreads();
}

// nxt[t, j] = first step after t that requests expert idx[t, j] again, or T (never).  seen[e]: earliest request of expert e among the
// batches already done.
__global__ __launch_bounds__(64) void next_use_kernel(const int32_t *__restrict__ idx, int64_t T, int K, int N,
                                                      int32_t *__restrict__ nxt)
{
    extern __shared__ int32_t ids[];           // a batch of rows, replaced by their next requests
    __shared__ int32_t seen[128];
    __shared__ unsigned long long when[128];
    const int64_t s = blockIdx.x;
    const int lane = threadIdx.x;
    const int32_t *tr = idx + s * T * K;
    int32_t *no = nxt + s * T * K;
    seen[lane] = (int32_t)T;
    seen[lane + 64] = (int32_t)T;
    const int32_t never = (int32_t)T;
    for (int64_t hi = T; hi > 0; hi -= CP_BATCH) {
        const int64_t t0 = hi >= CP_BATCH ? hi - CP_BATCH : 0;
        const int n = (int)(hi - t0);
        stage_rows(tr, t0, n, K, ids);
        next_uses(ids, n, K, N, t0, when, ids, [&](int e) { return e < 0 ? never : seen[e]; });
        for (int e = lane; e < 128; e += 64)
            if (when[e]) seen[e] = (int32_t)t0 + __ffsll((long long)when[e]) - 1;
        for (int q = lane; q < n * K; q += 64) no[t0 * K + q] = ids[q];
        __syncthreads();
    }
}

// lane `l` of a per-lane register (l wave-uniform)
__device__ __forceinline__ uint32_t get_lane(uint32_t reg, int l)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return (uint32_t)__builtin_amdgcn_readlane((int)reg, l);
#else
    (void)l;
    return reg;
#endif
}
__device__ __forceinline__ bool bit_of(unsigned long long lo, unsigned long long hi, int e)
{
    return (((e < 64 ? lo : hi) >> (e & 63)) & 1ull) != 0ull;
}

// a wave-uniform mask as a condition per lane
__device__ __forceinline__ bool mask_lane(unsigned long long m)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_inverse_ballot_w64(m);
#else
    return m & 1ull;
#endif
}

__device__ __forceinline__ unsigned long long ballot64(bool b)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_ballot_w64(b);
#else
    return b;
#endif
}

// the n lowest (HIGH: highest) members of a set of more than n
template <bool HIGH>
__device__ __forceinline__ void first_members(unsigned long long &lo, unsigned long long &hi, int n)
{
    unsigned long long out_lo = 0ull, out_hi = 0ull;
    for (; n > 0; --n) {
        unsigned long long &from = HIGH ? (hi ? hi : lo) : (lo ? lo : hi), &to = &from == &lo ? out_lo : out_hi;
        const unsigned long long one = HIGH ? 1ull << (63 - __clzll((long long)from)) : from & (0ull - from);
        to |= one;
        from ^= one;
    }
    lo = out_lo;
    hi = out_hi;
}

// The walk is sequential per trace and bound by the instructions its wavefronts issue, so the step is
// kept short: the sets (resident, requested, evictable) are masks in wave-uniform registers and all set
// arithmetic is scalar; only the retention keys are per lane, and the upper half of both exists only
// for more than 64 experts (WIDE).  A batch of 64 steps is staged in LDS (as much of it as K asks for: with room
// for 64 ids a step, 10 wavefronts fitted a compute unit) and lane l first builds the request mask of step
// l (one pass, all steps at once); the walk then fetches a step's mask with two or four lane reads.
// Victims leave in groups of equal key, found by one wavefront minimum per group (a pointer over the steps, for
// FIFO, took four times as long); only the group that is not needed whole is gone through by id.
// 3328 traces x 64 steps, 64 experts, top-6, capacity 12 (us): FIFO 31, LFU 32, Belady 32 (43 with its next requests walked back
// step by step in a launch of its own), LRU 9 (30 as a walk like these).
template <int POLICY, bool WIDE>
__global__ __launch_bounds__(64) void cache_policy_kernel(const int32_t *__restrict__ idx, int64_t T, int K, int N, int C,
                                                          unsigned long long expert_bytes,
                                                          const int32_t *__restrict__ nxt,
                                                          uint8_t *__restrict__ out_miss, uint8_t *__restrict__ out_uniq,
                                                          uint8_t *__restrict__ out_hit_tok,
                                                          unsigned long long *__restrict__ out_total_miss,
                                                          unsigned long long *__restrict__ out_total_uniq,
                                                          unsigned long long *__restrict__ out_bytes)
{
    static_assert(POLICY == REMOE_CACHE_FIFO || POLICY == REMOE_CACHE_LFU || POLICY == REMOE_CACHE_BELADY, "LRU keeps no keys here");
    extern __shared__ int32_t stage[];
    int32_t *ids = stage, *nus = stage + CP_BATCH * K;
    __shared__ uint32_t kb[(POLICY == REMOE_CACHE_BELADY) ? 128 : 1];
    __shared__ unsigned long long when[(POLICY == REMOE_CACHE_BELADY) ? 128 : 1];
    const int64_t s = blockIdx.x;
    const int lane = threadIdx.x;
    const int32_t *tr = idx + s * T * K;
    unsigned long long res_lo = 0ull, res_hi = 0ull;          // resident experts 0..63, 64..127 (wave-uniform)
    int held = 0;                                             // how many
    uint32_t key0 = 0, key1 = 0;                              // keys of experts lane, lane + 64
    uint32_t age0 = 0, age1 = 0;                              // LFU: step of last use, among equal keys
    unsigned long long lane_miss = 0, lane_uniq = 0;
    for (int64_t t0 = 0; t0 < T; t0 += CP_BATCH) {
        const int n = (int)((T - t0 < CP_BATCH) ? T - t0 : CP_BATCH);
        stage_rows(tr, t0, n, K, ids);
        if (POLICY == REMOE_CACHE_BELADY && T > CP_BATCH) stage_rows(nxt + s * T * K, t0, n, K, nus);
        __syncthreads();
        if (POLICY == REMOE_CACHE_BELADY && T <= CP_BATCH) {
            const int32_t never = (int32_t)T;
            next_uses(ids, n, K, N, 0, when, nus, [&](int) { return never; });
        }
        // request mask of step t0 + lane
        unsigned long long m_lo = 0ull, m_hi = 0ull;
        int valid = 0;
        if (lane < n) {
            for (int j = 0; j < K; ++j) {
                const int e = ids[lane * K + j];
                if (e >= 0 && e < N) {
                    ++valid;
                    if (!WIDE || e < 64) m_lo |= 1ull << (e & 63);
                    else m_hi |= 1ull << (e - 64);
                }
            }
        }
        const uint32_t m0 = (uint32_t)m_lo, m1 = (uint32_t)(m_lo >> 32), m2 = (uint32_t)m_hi, m3 = (uint32_t)(m_hi >> 32);
        const uint32_t uniq = (uint32_t)(__popcll(m_lo) + (WIDE ? __popcll(m_hi) : 0));
        const unsigned long long repeats = ballot64((int)uniq != valid);      // steps that name an expert twice
        uint32_t o_miss = 0, o_hit = 0;                       // results of step t0 + lane
        for (int tt = 0; tt < n; ++tt) {
            const uint32_t stamp = (uint32_t)(t0 + tt) + 1u;
            const unsigned long long req_lo = ((unsigned long long)get_lane(m1, tt) << 32) | get_lane(m0, tt);
            const unsigned long long req_hi = WIDE ? ((unsigned long long)get_lane(m3, tt) << 32) | get_lane(m2, tt) : 0ull;
            int miss = __popcll(req_lo & ~res_lo);
            if (WIDE) miss += __popcll(req_hi & ~res_hi);
            // token hits count a repeated id every time: lane j looks at slot j
            if ((repeats >> tt) & 1ull) {
                const int ej = lane < K ? ids[tt * K + lane] : -1;
                const int hits = __popcll(ballot64(ej >= 0 && ej < N && bit_of(res_lo, res_hi, ej)));
                if (lane == tt) o_hit = (uint32_t)hits;
            }
            if (lane == tt) o_miss = (uint32_t)miss;
            // serve the step: every requested expert is held now; refresh its key
            if (POLICY == REMOE_CACHE_FIFO) {
                if (mask_lane(req_lo & ~res_lo)) key0 = stamp;
                if (WIDE && mask_lane(req_hi & ~res_hi)) key1 = stamp;
            }
            if (POLICY == REMOE_CACHE_LFU) {
                if (mask_lane(req_lo)) { ++key0; age0 = stamp; }
                if (WIDE && mask_lane(req_hi)) { ++key1; age1 = stamp; }
            }
            if (POLICY == REMOE_CACHE_BELADY) {
                // lane j posts the key of slot j's expert, the lanes that own a requested expert pick theirs
                // up (one wavefront: its LDS accesses are served in program order; a repeated id posts the
                // same key twice)
                const int ej = lane < K ? ids[tt * K + lane] : -1;
                if (ej >= 0 && ej < N) kb[ej] = (uint32_t)T - (uint32_t)nus[tt * K + lane];
                if (mask_lane(req_lo)) key0 = kb[lane];
                if (WIDE && mask_lane(req_hi)) key1 = kb[lane + 64];
            }
            // Victims come from the held experts this step did not request: an expert served in a step
            // stays until the step is over (App. A, step atomicity and admission: E_t is part of the
            // next resident set whenever C >= K).  Only a step with more distinct requests than C
            // leaves none of those, and then the ranking runs over the requested ones.
            unsigned long long free_lo = res_lo & ~req_lo, free_hi = res_hi & ~req_hi;
            res_lo |= req_lo;
            res_hi |= req_hi;
            held += miss;
            while (held > C) {
                if ((free_lo | free_hi) == 0ull) {
                    free_lo = res_lo;
                    free_hi = res_hi;
                }
                const uint32_t b0 = mask_lane(free_lo) ? key0 : CP_NONE, b1 = WIDE && mask_lane(free_hi) ? key1 : CP_NONE;
                const uint32_t least = wave_min_u32(WIDE && b1 < b0 ? b1 : b0);
                unsigned long long g_lo = ballot64(key0 == least) & free_lo, g_hi = WIDE ? ballot64(key1 == least) & free_hi : 0ull;
                int n_g = __popcll(g_lo) + (WIDE ? __popcll(g_hi) : 0);
                const int drop = held - C;
                if (POLICY == REMOE_CACHE_LFU && n_g > drop) {
                    const uint32_t a0 = mask_lane(g_lo) ? age0 : CP_NONE, a1 = WIDE && mask_lane(g_hi) ? age1 : CP_NONE;
                    const uint32_t least_age = wave_min_u32(WIDE && a1 < a0 ? a1 : a0);
                    g_lo &= ballot64(age0 == least_age);
                    if (WIDE) g_hi &= ballot64(age1 == least_age);
                    n_g = __popcll(g_lo) + (WIDE ? __popcll(g_hi) : 0);
                }
                if (n_g > drop) {
                    first_members<POLICY == REMOE_CACHE_BELADY>(g_lo, g_hi, drop);
                    n_g = drop;
                }
                res_lo &= ~g_lo;
                free_lo &= ~g_lo;
                res_hi &= ~g_hi;
                free_hi &= ~g_hi;
                held -= n_g;
            }
        }
        if (lane < n) {
            out_miss[s * T + t0 + lane] = (uint8_t)o_miss;
            out_uniq[s * T + t0 + lane] = (uint8_t)uniq;
            out_hit_tok[s * T + t0 + lane] = (uint8_t)((repeats >> lane) & 1ull ? o_hit : uniq - o_miss);
            lane_miss += o_miss;
            lane_uniq += uniq;
        }
        __syncthreads();       // the staged rows are replaced next
    }
    for (int d = 32; d > 0; d >>= 1) {
        lane_miss += __shfl_xor(lane_miss, d, 64);
        lane_uniq += __shfl_xor(lane_uniq, d, 64);
    }
    if (lane == 0) {
        out_total_miss[s] = lane_miss;
        out_total_uniq[s] = lane_uniq;
        out_bytes[s] = lane_miss * expert_bytes;
    }
}

// ---- per-step sums over layers, histogram, percentiles -----------------------------------------------
constexpr int SS_MAX_HIST = 4097;       // sums up to 64 layers x 64 experts

__global__ void zero_u64_kernel(unsigned long long *p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = 0ull;
}

// V neighbouring steps per thread (4 when the table's rows allow 4-byte loads), the bytes summed two and two
// in 16-bit halves (at most 257 layers of at most 255).
template <int V>
__global__ __launch_bounds__(256) void step_summary_kernel(const uint8_t *__restrict__ miss, int64_t L, int64_t n,
                                                           uint16_t *__restrict__ out_all,
                                                           unsigned long long *__restrict__ hist, int hist_len)
{
    __shared__ uint32_t lh[SS_MAX_HIST];
    for (int v = threadIdx.x; v < hist_len; v += blockDim.x) lh[v] = 0u;
    __syncthreads();
    for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * V; i < n; i += (int64_t)gridDim.x * blockDim.x * V) {
        uint32_t even = 0, odd = 0;
#pragma unroll 8
        for (int64_t l = 0; l < L; ++l) {
            const uint32_t w = V == 4 ? *reinterpret_cast<const uint32_t *>(miss + l * n + i) : (uint32_t)miss[l * n + i];
            even += w & 0x00FF00FFu;
            odd += (w >> 8) & 0x00FF00FFu;
        }
        const uint32_t a[4] = {even & 0xFFFFu, odd & 0xFFFFu, even >> 16, odd >> 16};
#pragma unroll
        for (int j = 0; j < V; ++j) {
            out_all[i + j] = (uint16_t)a[j];
            atomicAdd(&lh[(int)a[j] < hist_len ? a[j] : (uint32_t)(hist_len - 1)], 1u);   // sums beyond the table share its last bin
        }
    }
    __syncthreads();
    for (int v = threadIdx.x; v < hist_len; v += blockDim.x)
        if (lh[v]) atomicAdd(&hist[v], (unsigned long long)lh[v]);   // integer sums: exact in any order
}

// percentile p = smallest v whose cumulative count reaches p percent of the n steps.  One wavefront: lane l
// sums its share of the bins, the shares are scanned, and the lane in whose share the count is reached finds
// the bin (a single thread walking the table took 23 us for 385 bins).
__global__ __launch_bounds__(64) void step_percentile_kernel(const unsigned long long *__restrict__ hist, int hist_len, unsigned long long n,
                                                             int32_t *__restrict__ out_pct)
{
    const int lane = threadIdx.x;
    const int per = (hist_len + 63) / 64, lo = lane * per, hi = lo + per < hist_len ? lo + per : hist_len;
    unsigned long long mine = 0;
    for (int v = lo; v < hi; ++v) mine += hist[v];
    unsigned long long upto = mine;                  // inclusive scan over the lanes
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned long long o = __shfl_up(upto, off, 64);
        if (lane >= off) upto += o;
    }
    const unsigned long long pcts[3] = {50ull, 95ull, 99ull};
    if (lane < 3 && n == 0) out_pct[lane] = -1;
    if (n == 0) return;
    for (int k = 0; k < 3; ++k) {
        const unsigned long long target = pcts[k] * n;
        if (100ull * upto < target || 100ull * (upto - mine) >= target) continue;
        unsigned long long cum = upto - mine;
        for (int v = lo; v < hi; ++v) {
            cum += hist[v];
            if (100ull * cum >= target) { out_pct[k] = v; break; }
        }
    }
}

// ---- expert-load balance of a trace -------------------------------------------------------------------
__device__ __forceinline__ double wave_sum_f64(double v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const unsigned long long b = (unsigned long long)__double_as_longlong(v);
        const unsigned lo = __shfl_xor((unsigned)(b & 0xFFFFFFFFull), off, 64);
        const unsigned hi = __shfl_xor((unsigned)(b >> 32), off, 64);
        v += __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
    }
    return v;
}

__global__ __launch_bounds__(256) void balance_kernel(const int32_t *__restrict__ idx, int64_t T, int K, int N,
                                                      uint32_t *__restrict__ out_load, int32_t *__restrict__ out_used,
                                                      double *__restrict__ out_entropy, double *__restrict__ out_cv)
{
    __shared__ uint32_t load[128], bins[4][128];      // a histogram per wavefront: fewer lanes meet in one bin
    const int64_t s = blockIdx.x;
    for (int q = threadIdx.x; q < 4 * 128; q += 256) (&bins[0][0])[q] = 0u;
    __syncthreads();
    const int32_t *tr = idx + s * T * K;
    uint32_t *mine = bins[threadIdx.x >> 6];
    auto add = [&](int e) { if ((uint32_t)e < (uint32_t)N) atomicAdd(&mine[e], 1u); };
    const int64_t n = T * K, n4 = (reinterpret_cast<uintptr_t>(tr) & 15) == 0 ? n / 4 : 0;
#pragma unroll 2
    for (int64_t q = threadIdx.x; q < n4; q += 256) {
        const int4 v = reinterpret_cast<const int4 *>(tr)[q];
        add(v.x);
        add(v.y);
        add(v.z);
        add(v.w);
    }
    for (int64_t q = n4 * 4 + threadIdx.x; q < n; q += 256) add(tr[q]);
    __syncthreads();
    if (threadIdx.x < 128) load[threadIdx.x] = (bins[0][threadIdx.x] + bins[1][threadIdx.x]) + (bins[2][threadIdx.x] + bins[3][threadIdx.x]);
    __syncthreads();
    if (threadIdx.x < N) out_load[s * N + threadIdx.x] = load[threadIdx.x];
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        const double total = (double)T * (double)K;
        const double m = total / (double)N;
        double h = 0.0, var = 0.0;
        int used = 0;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int e = lane + 64 * half;
            if (e < N) {
                const double c = (double)load[e];
                if (load[e] > 0u) {
                    const double p = c / total;
                    h -= p * log(p);
                }
                var += (c - m) * (c - m);
            }
            used += __popcll(__ballot(e < N && load[e] > 0u));
        }
        h = wave_sum_f64(h);
        var = wave_sum_f64(var);
        if (lane == 0) {
            out_used[s] = used;
            out_entropy[s] = (total > 0.0 && N > 1) ? h / log((double)N) : 0.0;
            out_cv[s] = (total > 0.0) ? sqrt(var / (double)N) / m : 0.0;
        }
    }
}

}  // namespace

size_t cache_workspace_bytes(int64_t S, int64_t T, int K, int policy)
{
    return policy == REMOE_CACHE_BELADY ? align_up(sizeof(int32_t) * (size_t)S * (size_t)T * (size_t)K, 256) : 0;
}

remoe_status launch_cache_policy(const int32_t *idx, int64_t S, int64_t T, int K, int N, int C, int policy,
                                 uint64_t expert_bytes, uint8_t *miss, uint8_t *uniq, uint8_t *hit_tok,
                                 uint64_t *total_miss, uint64_t *total_uniq, uint64_t *bytes, void *workspace,
                                 hipStream_t stream)
{
    if (S == 0) return REMOE_OK;
    const dim3 grid((unsigned)S), block(64);
    unsigned long long *tm = reinterpret_cast<unsigned long long *>(total_miss);
    unsigned long long *tu = reinterpret_cast<unsigned long long *>(total_uniq);
    unsigned long long *tb = reinterpret_cast<unsigned long long *>(bytes);
    int32_t *nxt = static_cast<int32_t *>(workspace);
    const size_t rows = sizeof(int32_t) * CP_BATCH * K;
    auto run = [&](auto kernel, size_t lds) {
        hipLaunchKernelGGL(kernel, grid, block, lds, stream, idx, T, K, N, C, expert_bytes, nxt, miss, uniq, hit_tok, tm, tu, tb);
    };
    const bool wide = N > 64;
    switch (policy) {
    case REMOE_CACHE_LRU:
        return launch_lru_detail(idx, S, T, K, N, C, expert_bytes, miss, uniq, hit_tok, total_miss, total_uniq, bytes, stream);
    case REMOE_CACHE_FIFO:
        run(wide ? cache_policy_kernel<REMOE_CACHE_FIFO, true> : cache_policy_kernel<REMOE_CACHE_FIFO, false>, rows);
        break;
    case REMOE_CACHE_LFU:
        run(wide ? cache_policy_kernel<REMOE_CACHE_LFU, true> : cache_policy_kernel<REMOE_CACHE_LFU, false>, rows);
        break;
    case REMOE_CACHE_BELADY:
        if (T > CP_BATCH) hipLaunchKernelGGL(next_use_kernel, grid, block, rows, stream, idx, T, K, N, nxt);
        run(wide ? cache_policy_kernel<REMOE_CACHE_BELADY, true> : cache_policy_kernel<REMOE_CACHE_BELADY, false>, 2 * rows);
        break;
    default:
        return fail(REMOE_E_INVALID_ARG, "unknown cache policy %d", policy);
    }
    return check_hip(hipGetLastError(), "cache_policy_kernel launch");
}

int step_summary_max_hist() { return SS_MAX_HIST; }

remoe_status launch_step_summary(const uint8_t *miss, int64_t L, int64_t S, int64_t T, uint16_t *out_all,
                                 uint64_t *hist, int hist_len, int32_t *pct, hipStream_t stream)
{
    const int64_t n = S * T;
    unsigned long long *h = reinterpret_cast<unsigned long long *>(hist);
    hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(256), 0, stream, h, (int64_t)hist_len);
    if (n > 0) {
        const bool wide = (n & 3) == 0 && ((reinterpret_cast<uintptr_t>(miss) & 3) == 0);
        int64_t blocks = ceil_div(n, wide ? 1024 : 256);
        if (blocks > 2048) blocks = 2048;
        if (wide) hipLaunchKernelGGL(step_summary_kernel<4>, dim3((unsigned)blocks), dim3(256), 0, stream, miss, L, n, out_all, h, hist_len);
        else hipLaunchKernelGGL(step_summary_kernel<1>, dim3((unsigned)blocks), dim3(256), 0, stream, miss, L, n, out_all, h, hist_len);
    }
    hipLaunchKernelGGL(step_percentile_kernel, dim3(1), dim3(64), 0, stream, h, hist_len, (unsigned long long)n, pct);
    return check_hip(hipGetLastError(), "step_summary launch");
}

remoe_status launch_balance(const int32_t *idx, int64_t S, int64_t T, int K, int N, uint32_t *load, int32_t *used,
                            double *entropy, double *cv, hipStream_t stream)
{
    if (S == 0) return REMOE_OK;
    hipLaunchKernelGGL(balance_kernel, dim3((unsigned)S), dim3(256), 0, stream, idx, T, K, N, load, used, entropy, cv);
    return check_hip(hipGetLastError(), "balance_kernel launch");
}

}  // namespace remoe
