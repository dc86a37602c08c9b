// Routing-trace statistics on expert-set bitmasks: adjacent-step overlap and LRU cache misses.
//
// trace_reuse_kernel: |E_t ∩ E_{t-1}|, the numerator of IR_t (Eq. 1).  One workgroup per trace
// (a (sequence, layer) pair); a lane turns one step into a 128-bit mask, gets its neighbour's mask
// for the step before and counts the bits of their AND.
//
// lru_walk_kernel: the per-layer LRU expert cache of the paper's simulator (App. A cache model,
// App. E.2 unique-miss accounting), one thread per step (see below).
#include <type_traits>

#include "common.h"
#include "lds_copy.h"
#include "trace_mask.h"

namespace remoe {

namespace {

// A wavefront walks its own run of consecutive steps 64 at a time, so a step's predecessor is in the
// neighbouring lane (lane 0: in the last lane of the pass before) and every id is read once.  Bound by
// the instructions that put a step's set together: 768 traces x 4096 steps x 8 ids (101 MB) 90 us at first, 21 us now.
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
// independent piece of work: one thread per step, up to LRU_CHUNK consecutive steps per pass of a workgroup.
//
// The experts of the steps (i - 2^j, i] are kept in LDS for j = 0 .. LEVELS - 1, for the steps of the pass and LRU_HALO before
// them, so that a walk takes 8 (4) steps at a time while they fit and then 4, 2 and 1: the lanes of a wavefront, whose walks
// have different lengths, go through the same few look-ups.  One step at a time, they wait for the longest walk: 768 traces x
// 4096 steps, 128 experts, top-8, C = 32 60 us, now 47; C = 64 166 and 59.  A step adds at most K experts,
// so the first floor(C / K) steps are merged without looking.  The masks are put together in LDS, a lane
// per id (one LDS OR instead of a dozen vector instructions), and the last rows of a pass serve the next.
//
// Walks that are not done where the staged steps begin go on without walking: there an expert is in the cache if fewer than C are more
// recent than it, and those are the ones seen so far and the ones used after it before the staged steps.  The workgroup keeps the last use
// of every expert before the staged steps, brought up to date for the passes that ask for it.  (A lane that read on through the
// trace a step at a time kept its workgroup waiting wherever an expert is rare or the capacity close to the experts in use: AR(1) of 0.9,
// some experts more popular, 64 experts, top-4, C = 48 820 us, now 114; 128 experts, top-8, C = 64, popularity more uneven 10.9 ms,
// now 0.20, and 0.65 for a cache that is walked step by step.)
constexpr int LRU_CHUNK = 512;   // steps per pass (threads per workgroup) of a trace that has as many
constexpr int LRU_HALO = 128;    // leaves room for three workgroups on a compute unit; 256: 768 x 4096 steps as above 115 and 231 us
constexpr uint32_t LRU_OWN = 1u << 31;      // keys of this call's steps (below 2^24) are larger than any of the prior state

__global__ __launch_bounds__(256) void lru_zero_kernel(uint64_t *__restrict__ total, uint64_t *__restrict__ uniq, uint64_t *__restrict__ bytes, int64_t S)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < S) {
        total[i] = 0;
        if (uniq) uniq[i] = 0;
        bytes[i] = 0;
    }
}

struct LruOut {
    uint8_t *miss, *uniq, *hit_tok;                  // uniq, hit_tok: DETAIL
    unsigned long long *total, *total_uniq, *bytes;
};

// Workgroup (s, part): chunks [part * chunks_per_wg, ...) of trace s, blockDim.x steps each.  One part: one workgroup per trace, which
// stores the totals; otherwise the workgroups add to totals that a kernel in front has cleared.
// halo: steps before a chunk that are staged as well.  DETAIL: distinct requests and token hits are reported too.  PRIOR: the traces
// go on from the caller's state.
template <int W, int LEVELS, bool DETAIL, bool PRIOR>
__global__ __launch_bounds__(LRU_CHUNK) void lru_walk_kernel(const int32_t *__restrict__ idx, int64_t T, int K,
                                                             int N, int C, unsigned long long expert_bytes,
                                                             const uint32_t *__restrict__ prior, int sure_steps, int halo, int parts,
                                                             int64_t chunks_per_wg, LruOut out)
{
    const uint32_t *const state = PRIOR ? prior : nullptr;
    extern __shared__ __align__(16) uint32_t lds_sets[];
    __shared__ uint32_t far_key[128];     // last use in front of the staged steps: LRU_OWN | step << 7 | e, in the prior state (step + 1) << 7 | e
    __shared__ Set<W> above[32 * W];      // the experts of larger far_key
    __shared__ int far_pass;              // the latest pass in which a walk went past the staged steps
    __shared__ unsigned long long wg_miss, wg_uniq;

    const int64_t s = blockIdx.x / parts;
    const int tid = threadIdx.x, chunk = blockDim.x, rows = chunk + halo;
    Set<W> *const sets = reinterpret_cast<Set<W> *>(lds_sets);           // [level][rows]; row halo + j is step t0 + j
    const int32_t *tr = idx + s * T * K;
    const bool wide = rows_are_wide(tr, K);
    if (tid == 0) { far_pass = 0; wg_miss = 0; wg_uniq = 0; }
    auto prior_key = [&](int e) {
        const uint32_t l = e < N ? state[s * N + e] : 0u;
        return l ? (l << 7 | (uint32_t)e) & ~LRU_OWN : 0u;
    };
    const bool one_pass = T <= chunk;         // only the prior state is in front of it
    for (int e = tid; e < 128; e += chunk) far_key[e] = PRIOR && one_pass ? prior_key(e) : 0u;
    unsigned long long total = 0, total_uniq = 0;
    const int64_t c_lo = (int64_t)(blockIdx.x % parts) * chunks_per_wg;
    // steps [t_from, t_from + n) -> rows [at, at + n), which are empty unless `clear`; `first` is the first row that is staged
    auto stage = [&](int64_t t_from, int n, int at, int first, bool clear) {
        if (clear) {
            for (int i = tid; i < n; i += chunk) sets[at + i] = Set<W>{};
            __syncthreads();
        }
        const int32_t *src = tr + t_from * K;
        auto put = [&](int row, int e) {
            if ((uint32_t)e < (uint32_t)N) atomicOr(&sets[at + row].w[e >> 5], 1u << (e & 31));
        };
        if (wide) {
            const int per_row = K >> 2;
            for (int q = tid; q < n * per_row; q += chunk) {
                const int4 v = reinterpret_cast<const int4 *>(src)[q];
                const int row = q / per_row;
                put(row, v.x);
                put(row, v.y);
                put(row, v.z);
                put(row, v.w);
            }
        } else {
            for (int q = tid; q < n * K; q += chunk) put(q / K, src[q]);
        }
        __syncthreads();
#pragma unroll
        for (int j = 1; j < LEVELS; ++j) {
            for (int i = at + tid; i < at + n; i += chunk) {
                if (i - (1 << j) + 1 < first) continue;
                Set<W> v = sets[(j - 1) * rows + i];
                v |= sets[(j - 1) * rows + i - (1 << (j - 1))];
                sets[j * rows + i] = v;
            }
            __syncthreads();
        }
    };
    auto report = [&](int64_t t, const Set<W> &want, const Set<W> &seen) __attribute__((always_inline)) {
        const int miss = count(without(want, seen));
        out.miss[s * T + t] = (uint8_t)miss;
        total += (unsigned long long)miss;
        if (DETAIL) {
            const int uniq = count(want);
            int hits = 0;              // a repeated id counts every time
            for (int j = 0; j < K; ++j) {
                const int e = tr[t * K + j];
                hits += (uint32_t)e < (uint32_t)N && holds(seen, e) ? 1 : 0;
            }
            out.uniq[s * T + t] = (uint8_t)uniq;
            out.hit_tok[s * T + t] = (uint8_t)hits;
            total_uniq += (unsigned long long)uniq;
        }
    };
    // far_key and above for the steps in front of `hi` (growing): those since the last call, then further back until C experts are known
    // (more can not matter), and behind the start of the trace the prior state
    int64_t far_lo = PRIOR && one_pass ? 0 : -1, far_hi = 0;           // steps in far_key
    auto look_back = [&](int64_t hi) __attribute__((always_inline)) {
        const bool prior_to_come = state && far_lo != 0;
        if (far_lo < 0) far_lo = far_hi = hi;
        while (hi > 0) {
            const bool ahead = far_hi < hi;
            const int64_t from = ahead ? far_hi : far_lo > LRU_CHUNK ? far_lo - LRU_CHUNK : 0;
            const int64_t to = !ahead ? far_lo : far_hi + LRU_CHUNK < hi ? far_hi + LRU_CHUNK : hi;
            const int32_t *src = tr + from * K;
#pragma unroll 1
            for (int q = tid; q < (int)(to - from) * K; q += chunk) {
                const int e = src[q];
                const uint32_t key = LRU_OWN | (uint32_t)(from + q / K) << 7 | (uint32_t)e;
                if ((uint32_t)e < (uint32_t)N && far_key[e] < key) atomicMax(&far_key[e], key);
            }
            if (ahead) far_hi = to;
            else far_lo = from;
            __syncthreads();
            const int known = __popcll(__ballot(far_key[tid & 63] != 0u)) + __popcll(__ballot(far_key[(tid & 63) + 64] != 0u));
            __syncthreads();
            if (far_hi == hi && (known >= C || known >= N || far_lo == 0)) break;
        }
        if (prior_to_come && far_lo == 0) {
            for (int e = tid; e < N; e += chunk)
                if (far_key[e] == 0u) far_key[e] = prior_key(e);
            __syncthreads();
        }
#pragma unroll 1
        for (int q = tid; q < 32 * W * W; q += chunk) {
            const int e = q & (32 * W - 1), word = q / (32 * W);
            const uint32_t k = far_key[e];
            uint32_t bits = 0u;
#pragma unroll 8
            for (int x = 0; x < 32; ++x) bits |= far_key[32 * word + x] > k ? 1u << x : 0u;
            above[e].w[word] = bits;
        }
        __syncthreads();
    };
    for (int64_t c = c_lo; c < c_lo + chunks_per_wg; ++c) {
        const int64_t t0 = c * chunk;
        if (t0 >= T) break;
        const int back = t0 < halo ? (int)t0 : halo;
        const int first = halo - back;
        if (c > c_lo) __syncthreads();     // the halo is there, the other rows are empty
        else if (back > 0) stage(t0 - back, back, first, first, true);
        stage(t0, (int)(T - t0 < chunk ? T - t0 : chunk), halo, first, c == c_lo);
        const int64_t t = t0 + tid;
        Set<W> want{}, seen{};
        bool far = false;                  // the walk is through the staged steps and not done
        if (t < T) {
            want = sets[halo + tid];
            int i = halo + tid - 1;        // next step to collect
            // the first steps fit whatever they hold
            int sure = sure_steps < i - first + 1 ? sure_steps : i - first + 1;
#pragma unroll
            for (int j = LEVELS - 1; j >= 0; --j) {
                while (sure >= (1 << j)) {
                    seen |= sets[j * rows + i];
                    i -= 1 << j;
                    sure -= 1 << j;
                }
            }
            bool open = count(seen) < C && any(without(want, seen));
            Set<W> m{};                    // the step in which the cache fills up
            int over = 0;                  // members that do not fit (LEVELS > 1: counted at the cut)
            if constexpr (LEVELS == 1) {
                int n = 0;
                while (open && i >= first) {
                    m = sets[i];
                    --i;
                    Set<W> all = seen;
                    all |= m;
                    n = count(all);
                    open = n < C && any(without(want, all));
                    if (n <= C) seen = all;
                }
                over = n - C;
            } else {
                // takes the 2^j steps up to i if the lane wants them and they fit (without a branch: the lanes differ)
                auto take = [&](int j, int at, bool wanted) {
                    Set<W> all = seen;
                    all |= sets[j * rows + at];
                    const int n = count(all);
                    const bool fits = wanted & (n <= C);
#pragma unroll
                    for (int q = 0; q < W; ++q) seen.w[q] = fits ? all.w[q] : seen.w[q];
                    i -= fits ? 1 << j : 0;
                    open = open & !(fits & ((n == C) | !any(without(want, all))));
                    return fits;
                };
                constexpr int TOP = 1 << (LEVELS - 1);
                for (bool more = open & (i - TOP + 1 >= first); more;)
                    more = take(LEVELS - 1, i, true) & open & (i - TOP + 1 >= first);
#pragma unroll
                for (int j = LEVELS - 2; j >= 0; --j) take(j, i > 0 ? i : 0, open & (i - (1 << j) + 1 >= first));
                if (open && i >= first) m = sets[i];
            }
            // the cut falls inside step m: its lowest ids were touched first and are out
            if (LEVELS == 1 ? over > 0 : any(m)) {
                Set<W> fresh = without(m, seen);
                if (LEVELS == 1) drop_one_by_one(fresh, over);
                else drop_lowest(fresh, count(seen) + count(fresh) - C);
                seen |= fresh;
            }
            far = open && i < first && (t0 > back || state);
            report(t, want, seen);         // (taken back where far: one branch less for the others)
        }
        if (__ballot(far)) far_pass = (int)(c - c_lo) + 1;
        if (!PRIOR && one_pass) break;     // nothing is in front of it
        lds_barrier();                     // the rows of this pass are no longer read (its results may still be on their way)
        const int last_far = far_pass;
        if (c + 1 < c_lo + chunks_per_wg) {
            const int row = halo + tid;
            if (row >= chunk) {
#pragma unroll
                for (int j = 0; j < LEVELS; ++j) sets[j * rows + row - chunk] = sets[j * rows + row];
            }
            sets[row] = Set<W>{};
        }
        if (last_far == (int)(c - c_lo) + 1) {
            look_back(t0 - back);
            if (far) {
                total -= (unsigned long long)count(without(want, seen));
                if (DETAIL) total_uniq -= (unsigned long long)count(want);
                // an expert is in the cache if fewer than C are more recent: those of the staged steps, and those above it in front of them
                const Set<W> left = without(want, seen), staged = seen;
#pragma unroll
                for (int q = 0; q < W; ++q) {
                    for (uint32_t bits = left.w[q]; bits; bits &= bits - 1u) {
                        const int e = 32 * q + __ffs((int)bits) - 1;
                        Set<W> newer = above[e];
                        newer |= staged;
                        if (far_key[e] != 0u && count(newer) < C) seen |= single<W>(e);
                    }
                }
                report(t, want, seen);
            }
        }
    }
    // integer sums: exact and independent of the order in which they are added
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        total += __shfl_xor(total, off, 64);
        if (DETAIL) total_uniq += __shfl_xor(total_uniq, off, 64);
    }
    if ((tid & 63) == 0) {
        if (total) atomicAdd(&wg_miss, total);
        if (DETAIL && total_uniq) atomicAdd(&wg_uniq, total_uniq);
    }
    __syncthreads();
    if (tid == 0) {
        if (parts == 1) {
            out.total[s] = wg_miss;
            out.bytes[s] = wg_miss * expert_bytes;
            if (DETAIL) out.total_uniq[s] = wg_uniq;
        } else {
            if (wg_miss) {
                atomicAdd(&out.total[s], wg_miss);
                atomicAdd(&out.bytes[s], wg_miss * expert_bytes);
            }
            if (DETAIL && wg_uniq) atomicAdd(&out.total_uniq[s], wg_uniq);
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
    // few traces: more wavefronts for each, as long as every wavefront has a pass of 64 steps; six to a SIMD where the traces are long
    // (4 / 6 / 8 to a SIMD: 768 x 4096 steps, top-8 21.9 / 20.9 / 22.5 us, top-6 25.6 / 23.0 / 27.2; 300 x 1000 steps 5.1 / 6.6 / -)
    int64_t waves = ceil_div(T >= 2048 ? 6144 : 4096, S);
    if (waves < 4) waves = 4;
    if (waves > ceil_div(T, 64)) waves = ceil_div(T, 64);
    waves = waves < 1 ? 1 : waves > 16 ? 16 : waves;
    hipLaunchKernelGGL(trace_reuse_kernel, dim3((unsigned)S), dim3((unsigned)(64 * waves)), 0, stream, idx, T, K, N, ov, sum);
    return check_hip(hipGetLastError(), "trace_reuse_kernel launch");
}

static remoe_status launch_lru_walk(const int32_t *idx, int64_t S, int64_t T, int K, int N, int C, uint64_t expert_bytes, const uint32_t *state,
                                    const LruOut &out, hipStream_t stream)
{
    // (a few steps that go on from a state, as in decoding, leave most threads without a step, but they put above together: 48 traces of
    // one step, 128 experts, 13.0 us with 64 threads)
    const int64_t least = state && T > 0 ? 256 : 0;
    const int chunk = T < LRU_CHUNK ? (int)align_up((size_t)(T > least ? T : least), 64) : LRU_CHUNK;
    const int64_t n_chunks = chunk > 0 ? ceil_div(T, chunk) : 0;
    // a workgroup takes a whole trace where the traces alone fill the chip (no clearing launch, no global atomics)
    const int64_t parts = S >= 512 || n_chunks <= 1 ? 1 : n_chunks;
    if (parts > 1 || T == 0) {
        hipLaunchKernelGGL(lru_zero_kernel, dim3((unsigned)ceil_div(S, 256)), dim3(256), 0, stream, reinterpret_cast<uint64_t *>(out.total),
                           reinterpret_cast<uint64_t *>(out.total_uniq), reinterpret_cast<uint64_t *>(out.bytes), S);
        REMOE_HIP_TRY(hipGetLastError());
    }
    if (T == 0) return REMOE_OK;
    const int halo = n_chunks <= 1 ? 0 : LRU_HALO;
    // Tables cost a pass over the staged steps for each level.  768 x 4096 steps, 128 experts (us with 1 / 2 / 3 / 4 / 5 levels): top-8,
    // C = 8 23 / 26 / 28 / 31 / 35, 16 38 / 41 / 41 / 44 / 49, 24 48 / 46 / 44 / 46 / 49, 32 59 / 54 / 47 / 46 / 49, 48 97 / 74 / 57 / 51 / 52,
    // top-2, C = 64 680 / 405 / 220 / 167 / 172; 64 experts, top-6: C = 12 45 / 43 / 43 / 45 / 48, 24 69 / 55 / 50 / 47 / 49.
    const int words = N > 64 ? 4 : 2, levels = T < 16 || C <= (words == 4 ? 2 : 1) * K ? 1 : C <= 3 * K ? 3 : 4;
    const size_t lds = (size_t)levels * (chunk + halo) * words * 4;
    const int sure = (int)(C / K < chunk + halo ? C / K : chunk + halo);
    auto pick = [&](auto w, auto l) {
        constexpr int W = decltype(w)::value, L = decltype(l)::value;
        return out.uniq ? lru_walk_kernel<W, L, true, false> : state ? lru_walk_kernel<W, L, false, true> : lru_walk_kernel<W, L, false, false>;
    };
    const std::integral_constant<int, 1> one;
    const std::integral_constant<int, 2> two;
    const std::integral_constant<int, 3> three;
    const std::integral_constant<int, 4> four;
    auto kernel = words == 4 ? (levels == 1 ? pick(four, one) : levels == 3 ? pick(four, three) : pick(four, four))
                             : (levels == 1 ? pick(two, one) : levels == 3 ? pick(two, three) : pick(two, four));
    const int64_t most = (((int64_t)1 << 31) / chunk) / parts;           // traces of a launch, whose threads are counted in 32 bits
    for (int64_t s0 = 0; s0 < S; s0 += most) {
        LruOut o = out;
        o.miss += s0 * T;
        o.total += s0;
        o.bytes += s0;
        if (out.uniq) {
            o.uniq += s0 * T;
            o.hit_tok += s0 * T;
            o.total_uniq += s0;
        }
        hipLaunchKernelGGL(kernel, dim3((unsigned)((S - s0 < most ? S - s0 : most) * parts)), dim3((unsigned)chunk), lds, stream, idx + s0 * T * K, T, K, N, C,
                           (unsigned long long)expert_bytes, state ? state + s0 * N : nullptr, sure, halo, (int)parts, ceil_div(n_chunks, parts), o);
        REMOE_HIP_TRY(hipGetLastError());
    }
    return REMOE_OK;
}

remoe_status launch_lru(const int32_t *idx, int64_t S, int64_t T, int K, int N, int C,
                        uint64_t expert_bytes, int64_t step0, uint32_t *state, uint8_t *miss,
                        uint64_t *total, uint64_t *bytes, hipStream_t stream)
{
    if (S == 0) return REMOE_OK;
    LruOut out{};
    out.miss = miss;
    out.total = reinterpret_cast<unsigned long long *>(total);
    out.bytes = reinterpret_cast<unsigned long long *>(bytes);
    const remoe_status st = launch_lru_walk(idx, S, T, K, N, C, expert_bytes, state, out, stream);
    if (st != REMOE_OK || T == 0) return st;
    if (state) {   // after every walk has read the prior state
        hipLaunchKernelGGL(lru_state_kernel, dim3((unsigned)S), dim3(256), 0, stream, idx, T, K, N, step0, state);
        REMOE_HIP_TRY(hipGetLastError());
    }
    return REMOE_OK;
}

remoe_status launch_lru_detail(const int32_t *idx, int64_t S, int64_t T, int K, int N, int C, uint64_t expert_bytes, uint8_t *miss, uint8_t *uniq,
                               uint8_t *hit_tok, uint64_t *total_miss, uint64_t *total_uniq, uint64_t *bytes, hipStream_t stream)
{
    if (S == 0) return REMOE_OK;
    const LruOut out{miss, uniq, hit_tok, reinterpret_cast<unsigned long long *>(total_miss), reinterpret_cast<unsigned long long *>(total_uniq),
                     reinterpret_cast<unsigned long long *>(bytes)};
    return launch_lru_walk(idx, S, T, K, N, C, expert_bytes, nullptr, out, stream);
}

}  // namespace remoe
