// Routing-trace statistics on expert-set bitmasks: adjacent-step overlap and LRU cache misses.
//
// trace_reuse_kernel: |E_t ∩ E_{t-1}|, the numerator of IR_t (Eq. 1).  One workgroup per trace
// (a (sequence, layer) pair); a lane turns one step into a 128-bit mask, gets its neighbour's mask
// for the step before and counts the bits of their AND.
//
// lru_walk_kernel: the per-layer LRU expert cache of the paper's simulator (App. A cache model,
// App. E.2 unique-miss accounting), one thread per step (see below).
#include "common.h"
#include "trace_mask.h"

namespace remoe {

namespace {

// A wavefront walks its own run of consecutive steps 64 at a time, so a step's predecessor is in the
// neighbouring lane (lane 0: in the last lane of the pass before) and every id is read once.  Bound by
// reading the trace: 768 traces x 4096 steps x 8 ids (101 MB) 90 us before, 23 us now.
__global__ void trace_reuse_kernel(const int32_t *__restrict__ idx, int64_t T, int K, int N, uint8_t *__restrict__ ov,
                                   uint64_t *__restrict__ sum)
{
    const int64_t s = blockIdx.x;
    const int32_t *tr = idx + s * T * K;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const bool wide = rows_are_wide(tr, K);
    const int64_t run = ((T + waves - 1) / waves + 63) & ~(int64_t)63;
    const int64_t t_lo = wave * run, t_hi = t_lo + run < T ? t_lo + run : T;
    unsigned long long local = 0;
    if (t_lo < t_hi) {
        Mask last = t_lo > 0 ? step_mask(tr + (t_lo - 1) * K, K, N, wide) : Mask{};
        for (int64_t t0 = t_lo; t0 < t_hi; t0 += 64) {
            const int64_t t = t0 + lane;
            const bool live = t < t_hi;
            const Mask m = step_mask(tr + (live ? t : t_hi - 1) * K, K, N, wide);
            int o = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t up = __shfl_up(m.w[q], 1, 64);
                o += __popc(m.w[q] & (lane ? up : last.w[q]));
            }
            if (t == 0) o = 0;
            if (live) {
                ov[s * T + t] = (uint8_t)o;
                local += (unsigned long long)o;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) last.w[q] = __shfl(m.w[q], 63, 64);
        }
    }
    // workgroup reduction of the per-thread sums (integer: exact and order independent)
    __shared__ unsigned long long part[16];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) local += __shfl_xor(local, off, 64);
    if (lane == 0) part[wave] = local;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long v = 0;
        for (int w = 0; w < waves; ++w) v += part[w];
        sum[s] = v;
    }
}

// ---- LRU misses, every step in parallel
//
// With recency keys (step, id) the cache before step t holds the C distinct experts of largest
// key.  Walking back from step t-1 and collecting unseen experts, each step's from the highest id
// down, visits the experts in exactly that key order, so the first C collected are the resident
// set; the walk also ends as soon as every expert of step t has been collected (all hits) or the
// trace, and then the caller's prior state, is exhausted.  Each step of a trace is therefore an
// independent piece of work: one thread per step, LRU_CHUNK consecutive steps per pass of a workgroup,
// with the 128-bit masks of those steps and of the LRU_HALO before them staged in LDS.
//
// A step adds at most K experts, so the first floor(C / K) steps are merged without looking.  Lanes end their
// walks at different steps, so what happens only at the end of a walk (cutting the step in which the cache
// fills up) waits until the whole wavefront is out of the loop.  The masks are put together in LDS, a lane
// per id (one LDS OR instead of a dozen vector instructions), and the last LRU_HALO of a pass serve the next.
// 768 traces x 4096 steps, top-8, C = 32: 120 us before, 62 us now.
constexpr int LRU_CHUNK = 512;   // steps per pass (threads per workgroup)
constexpr int LRU_HALO = 256;    // earlier steps whose masks are staged as well

__global__ __launch_bounds__(256) void lru_zero_kernel(uint64_t *__restrict__ total, uint64_t *__restrict__ bytes, int64_t S)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < S) { total[i] = 0; bytes[i] = 0; }
}

// Workgroup (s, part): chunks [part * chunks_per_wg, ...) of trace s.  `whole`: one workgroup per trace, which
// stores the totals; otherwise the workgroups add to totals that a kernel in front has cleared.
__global__ __launch_bounds__(LRU_CHUNK) void lru_walk_kernel(const int32_t *__restrict__ idx, int64_t T, int K,
                                                             int N, int C, unsigned long long expert_bytes,
                                                             const uint32_t *__restrict__ state, int sure_steps, int parts, int64_t chunks_per_wg,
                                                             uint8_t *__restrict__ miss_out,
                                                             unsigned long long *__restrict__ total_out,
                                                             unsigned long long *__restrict__ bytes_out)
{
    __shared__ Mask masks[LRU_CHUNK + LRU_HALO];
    __shared__ uint32_t prev_key[128];
    __shared__ uint8_t prev_order[128];   // experts of the prior state, most recent first
    __shared__ int n_prev;
    __shared__ unsigned long long wg_miss;

    const int64_t s = blockIdx.x / parts;
    const int tid = threadIdx.x;
    const int32_t *tr = idx + s * T * K;
    const bool wide = rows_are_wide(tr, K);
    if (tid == 0) { n_prev = 0; wg_miss = 0; }
    if (state && tid < 128) {
        const uint32_t l = (tid < N) ? state[s * N + tid] : 0u;
        prev_key[tid] = l ? ((l << 7) | (uint32_t)tid) : 0u;
    }
    __syncthreads();
    if (state && tid < 128) {
        const uint32_t k = prev_key[tid];
        if (k) {
            int above = 0;
            for (int e = 0; e < 128; ++e) above += prev_key[e] > k;
            prev_order[above] = (uint8_t)tid;   // nonzero keys are distinct: the ranks are a permutation
            atomicAdd(&n_prev, 1);
        }
    }
    unsigned long long total = 0;
    const int64_t c_lo = (int64_t)(blockIdx.x % parts) * chunks_per_wg;
    // masks[LRU_HALO + j] is step t0 + j; `first` is the first staged one
    auto stage = [&](int64_t t_from, int n, int at) {
        for (int i = tid; i < n; i += LRU_CHUNK) masks[at + i] = Mask{};
        __syncthreads();
        const int32_t *src = tr + t_from * K;
        auto put = [&](int row, int e) {
            if ((uint32_t)e < (uint32_t)N) atomicOr(&masks[at + row].w[e >> 5], 1u << (e & 31));
        };
        if (wide) {
            const int per_row = K >> 2;
            for (int q = tid; q < n * per_row; q += LRU_CHUNK) {
                const int4 v = reinterpret_cast<const int4 *>(src)[q];
                const int row = q / per_row;
                put(row, v.x);
                put(row, v.y);
                put(row, v.z);
                put(row, v.w);
            }
        } else {
            for (int q = tid; q < n * K; q += LRU_CHUNK) put(q / K, src[q]);
        }
        __syncthreads();
    };
    for (int64_t c = c_lo; c < c_lo + chunks_per_wg; ++c) {
        const int64_t t0 = c * LRU_CHUNK;
        if (t0 >= T) break;
        const int back = t0 < LRU_HALO ? (int)t0 : LRU_HALO;
        const int first = LRU_HALO - back;
        if (c > c_lo) {
            __syncthreads();               // the masks of the pass before are no longer read
            if (tid < LRU_HALO) masks[tid] = masks[LRU_CHUNK + tid];
            __syncthreads();
        } else {
            stage(t0 - back, back, first);
        }
        stage(t0, (int)(T - t0 < LRU_CHUNK ? T - t0 : LRU_CHUNK), LRU_HALO);
        const int64_t t = t0 + tid;
        int miss = 0;
        if (t < T) {
            const Mask want = masks[LRU_HALO + tid];
            Mask seen{}, m{};
            int i = LRU_HALO + tid - 1;    // next step to collect
            // the first steps fit whatever they hold
            for (int stop = i - sure_steps < first - 1 ? first - 1 : i - sure_steps; i > stop; --i) seen |= masks[i];
            int held = count(seen);
            bool open = held < C && any(without(want, seen));
            while (open && i >= first) {
                m = masks[i];
                --i;
                Mask all = seen;
                all |= m;
                held = count(all);
                open = held < C && any(without(want, all));
                if (held <= C) seen = all;
            }
            int64_t u = t0 + (i - LRU_HALO);
            while (open && u >= 0) {       // past the staged steps
                m = step_mask(tr + u * K, K, N, wide);
                --u;
                Mask all = seen;
                all |= m;
                held = count(all);
                open = held < C && any(without(want, all));
                if (held <= C) seen = all;
            }
            if (held > C) {                // the cut falls inside step m: its lowest ids were touched first and are out
                Mask fresh = without(m, seen);
                for (int over = held - C; over > 0; --over) drop_lowest(fresh);
                seen |= fresh;
            }
            if (state && u < 0) {
                int cnt = count(seen);
                const int np = n_prev;
                for (int j = 0; j < np && cnt < C && any(without(want, seen)); ++j) {
                    const Mask bit = single(prev_order[j]);
                    if (any(without(bit, seen))) {
                        seen |= bit;
                        ++cnt;
                    }
                }
            }
            miss = count(without(want, seen));
            miss_out[s * T + t] = (uint8_t)miss;
        }
        total += (unsigned long long)miss;
    }
    // integer sums: exact and independent of the order in which they are added
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) total += __shfl_xor(total, off, 64);
    if ((tid & 63) == 0 && total) atomicAdd(&wg_miss, total);
    __syncthreads();
    if (tid == 0) {
        if (parts == 1) {
            total_out[s] = wg_miss;
            bytes_out[s] = wg_miss * expert_bytes;
        } else if (wg_miss) {
            atomicAdd(&total_out[s], wg_miss);
            atomicAdd(&bytes_out[s], wg_miss * expert_bytes);
        }
    }
}

// state[e] = (global step of e's last use) + 1 after the call; one workgroup per trace
__global__ __launch_bounds__(256) void lru_state_kernel(const int32_t *__restrict__ idx, int64_t T, int K,
                                                        int N, int64_t step0, uint32_t *__restrict__ state)
{
    __shared__ uint32_t last[128];
    const int64_t s = blockIdx.x;
    const int tid = threadIdx.x;
    if (tid < 128) last[tid] = (tid < N) ? state[s * N + tid] : 0u;
    __syncthreads();
    const int32_t *tr = idx + s * T * K;
    for (int64_t t = tid; t < T; t += blockDim.x) {
        for (int j = 0; j < K; ++j) {
            const int e = tr[t * K + j];
            if (e >= 0 && e < N) atomicMax(&last[e], (uint32_t)(step0 + t + 1));
        }
    }
    __syncthreads();
    if (tid < N) state[s * N + tid] = last[tid];
}

}  // namespace

remoe_status launch_trace_reuse(const int32_t *idx, int64_t S, int64_t T, int K, int N,
                                uint8_t *ov, uint64_t *sum, hipStream_t stream)
{
    if (S == 0) return REMOE_OK;
    // few traces: more wavefronts for each, as long as every wavefront has a pass of 64 steps
    int64_t waves = S >= 1024 ? 4 : ceil_div(4096, S);
    if (waves > ceil_div(T, 64)) waves = ceil_div(T, 64);
    waves = waves < 1 ? 1 : waves > 16 ? 16 : waves;
    hipLaunchKernelGGL(trace_reuse_kernel, dim3((unsigned)S), dim3((unsigned)(64 * waves)), 0, stream, idx, T, K, N, ov, sum);
    return check_hip(hipGetLastError(), "trace_reuse_kernel launch");
}

remoe_status launch_lru(const int32_t *idx, int64_t S, int64_t T, int K, int N, int C,
                        uint64_t expert_bytes, int64_t step0, uint32_t *state, uint8_t *miss,
                        uint64_t *total, uint64_t *bytes, hipStream_t stream)
{
    if (S == 0) return REMOE_OK;
    const int64_t n_chunks = ceil_div(T, LRU_CHUNK);
    // a workgroup takes a whole trace where the traces alone fill the chip (no clearing launch, no global atomics)
    const int64_t parts = S >= 512 || n_chunks <= 1 ? 1 : n_chunks;
    if (parts > 1 || T == 0) {
        hipLaunchKernelGGL(lru_zero_kernel, dim3((unsigned)ceil_div(S, 256)), dim3(256), 0, stream, total, bytes, S);
        REMOE_HIP_TRY(hipGetLastError());
    }
    if (T == 0) return REMOE_OK;
    if (S * parts >= ((int64_t)1 << 31))
        return fail(REMOE_E_UNSUPPORTED, "lru_simulate: %lld traces x %lld steps exceed one launch", (long long)S, (long long)T);
    hipLaunchKernelGGL(lru_walk_kernel, dim3((unsigned)(S * parts)), dim3(LRU_CHUNK), 0, stream, idx, T, K, N, C,
                       (unsigned long long)expert_bytes, state, (int)(C / K < LRU_HALO ? C / K : LRU_HALO), (int)parts, ceil_div(n_chunks, parts), miss,
                       reinterpret_cast<unsigned long long *>(total), reinterpret_cast<unsigned long long *>(bytes));
    REMOE_HIP_TRY(hipGetLastError());
    if (state) {   // after every walk has read the prior state
        hipLaunchKernelGGL(lru_state_kernel, dim3((unsigned)S), dim3(256), 0, stream, idx, T, K, N, step0, state);
        REMOE_HIP_TRY(hipGetLastError());
    }
    return REMOE_OK;
}

}  // namespace remoe
