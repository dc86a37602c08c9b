// Cache-aware rerouting at inference time (App. G): experts resident in the LRU cache get a bonus on
// their pre-top-k score, so each step's routing depends on the cache the earlier steps left.
//
// Score of expert e at step t: P_t[e] * factor if e is resident before the step, else P_t[e] (factor =
// exp(beta): the same order as adding beta to the resident experts' logits); ties to the lower id; gate
// weights are the unmodified probabilities of the chosen experts (divided by their sum when renorm).
//
// What bounds it is the chain from step to step of a trace, so everything that does not need the cache
// is taken out of that chain, and the chain is cut:
//   reroute_rank_kernel    every step on its own, one wavefront each: an expert has two scores, resident or
//                          not, and the order of all 2 N of them (score, then id) does not depend on the
//                          cache.  The first P entries of that order are kept, a byte each.
//   reroute_walk_kernel    the steps in order.  Lane r holds entry r: it is in force if the expert's
//                          residency is the entry's, and the first K entries in force are the step's experts
//                          in their final order: one comparison, one ballot and a lane count instead of K
//                          wavefront maxima.  A step whose first P entries hold fewer than K in force (or
//                          that has no list) takes the K maxima from the probabilities instead.
//                          A trace is walked by up to 16 wavefronts at once, each on its own stretch from a
//                          guessed cache: a cold one warmed on the steps before the stretch.  A
//                          stretch counts only if its first state is the last state of the stretch before
//                          it, key for key; those that fail are walked again from that state until all
//                          agree, so the result is that of the single walk whatever the guesses were.
//   reroute_weights_kernel ids and gate weights from the entries the walk marked.
// The lists and marks of a step live where its ids and weights will be (8 K bytes), so that no
// scratch memory is needed: entries r < 4 K in the id row, the marks (one bit per entry) in front of the
// weight row and the other entries behind them.
//
// 16 traces x 4096 steps, 128 experts, top-8, C = 4: 7.5 ms as one walk of K maxima per step and wavefront,
// 0.19 ms now (lists 37, walk 140, weights 15 us; the
// walk is bound by the instructions its 16 wavefronts issue: 1.8 us a step before, 0.45 us now with 16 steps at once).
#include "common.h"
#include "topk.h"

namespace remoe {

namespace {

constexpr int RR_WAVES = 16;            // stretches of a trace walked at once
constexpr int RR_MIN_STEPS = 32;        // a shorter stretch is not worth its warm-up
constexpr int RR_BATCH = 16;            // steps whose lists are staged in LDS at a time
constexpr int RR_MAX_ENTRIES = 63;      // see reroute_rank_kernel

struct RowLayout {
    int K, marks, entries;              // marks: bytes in front of the weight row
    __host__ __device__ RowLayout(int N, int K_) : K(K_), marks(K_ < 8 ? K_ : 8)
    {
        entries = 8 * K - marks;
        if (entries > 2 * N) entries = 2 * N;
        if (entries > RR_MAX_ENTRIES) entries = RR_MAX_ENTRIES;
    }
    // byte of entry r < entries in row `row`
    __device__ uint8_t *entry(int32_t *idx, float *w, int64_t row, int r) const
    {
        return r < 4 * K ? reinterpret_cast<uint8_t *>(idx + row * K) + r
                         : reinterpret_cast<uint8_t *>(w + row * K) + marks + (r - 4 * K);
    }
    __device__ uint8_t *mark(float *w, int64_t row) const { return reinterpret_cast<uint8_t *>(w + row * K); }
};

// value of lane ^ J
template <int J>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v)
{
#if defined(__HIP_DEVICE_COMPILE__)
    if (J == 1) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);      // quad_perm [1,0,3,2]
    if (J == 2) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);      // quad_perm [2,3,0,1]
    if (J == 4) {                                                                                    // 7 - l, then 3 - l
        const int m = __builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);
        return (uint32_t)__builtin_amdgcn_update_dpp(0, m, 0x1B, 0xF, 0xF, true);
    }
    if (J == 8) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, true);     // row_ror:8
    if (J == 16) return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x401F);
    return (uint32_t)__shfl_xor((int)v, J, 64);
#else
    return v;
#endif
}

typedef unsigned long long u64;

__device__ __forceinline__ u64 ballot(bool b)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_ballot_w64(b);
#else
    return b;
#endif
}

template <int J>
__device__ __forceinline__ u64 lane_xor64(u64 v)
{
    return ((u64)lane_xor<J>((uint32_t)(v >> 32)) << 32) | lane_xor<J>((uint32_t)v);
}

template <int J>
__device__ __forceinline__ u64 keep(u64 v, bool larger)
{
    const u64 o = lane_xor64<J>(v);
    return ((v > o) == larger) ? v : o;
}

// merge of a bitonic sequence of 2 J lanes, larger values to the lanes `down` says
template <int J>
__device__ __forceinline__ u64 merge(u64 v, int lane, bool down)
{
    v = keep<J>(v, ((lane & J) == 0) == down);
    if constexpr (J > 1) v = merge<J / 2>(v, lane, down);
    return v;
}

// 64 lanes sorted, descending if `down`
__device__ __forceinline__ u64 sort64(u64 v, int lane, bool down)
{
    v = merge<1>(v, lane, ((lane & 2) == 0) == down);
    v = merge<2>(v, lane, ((lane & 4) == 0) == down);
    v = merge<4>(v, lane, ((lane & 8) == 0) == down);
    v = merge<8>(v, lane, ((lane & 16) == 0) == down);
    v = merge<16>(v, lane, ((lane & 32) == 0) == down);
    return merge<32>(v, lane, down);
}

// Entry of the list: expert in the low seven bits, bit 7 = the score it has as a resident.  Two equal first
// entries say that the row has no list: probabilities that are negative or no numbers, bonuses that
// overflow (more of those tie than the 64 kept), or bonuses that rounding makes equal in an order other than that
// of the ids (the boosted list is taken to be in the order of the plain one).  The last of the 64 boosted scores kept could tie with one that was not, hence 63 entries.
template <bool WIDE>
__global__ __launch_bounds__(256) void reroute_rank_kernel(const float *__restrict__ probs, int64_t rows, int N, float factor, RowLayout lay,
                                                           int32_t *out_idx, float *out_w)
{
    const int lane = threadIdx.x & 63;
    const int64_t stride = (int64_t)gridDim.x * 4;
    for (int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); row < rows; row += stride) {
        const float *p = probs + row * N;
        const uint32_t q0 = lane < N ? __float_as_uint(p[lane]) : 0u;
        const uint32_t q1 = WIDE && lane + 64 < N ? __float_as_uint(p[lane + 64]) : 0u;
        bool bad = q0 > 0x7F800000u || q1 > 0x7F800000u;          // negative or NaN
        // key: score, then lower id first; 0 where there is no expert
        u64 a = lane < N ? ((u64)q0 << 32) | (uint32_t)((128 - lane) << 1) : 0ull;
        a = sort64(a, lane, true);
        if (WIDE) {
            u64 b = lane + 64 < N ? ((u64)q1 << 32) | (uint32_t)((64 - lane) << 1) : 0ull;
            b = sort64(b, lane, false);
            a = merge<32>(a > b ? a : b, lane, true);
        }
        const float boosted = __uint_as_float((uint32_t)(a >> 32)) * factor;
        const u64 b = a ? ((u64)__float_as_uint(boosted) << 32) | (uint32_t)a | 1u : 0ull;
        const u64 after = ((u64)(uint32_t)__shfl_down((int)(uint32_t)(b >> 32), 1, 64) << 32) |
                          (uint32_t)__shfl_down((int)(uint32_t)b, 1, 64);
        bad = bad || (lane < 63 && after > b) || __float_as_uint(boosted) >= 0x7F800000u;
        const u64 rev = ((u64)(uint32_t)__shfl_xor((int)(uint32_t)(b >> 32), 63, 64) << 32) |
                        (uint32_t)__shfl_xor((int)(uint32_t)b, 63, 64);
        const u64 m = merge<32>(a > rev ? a : rev, lane, true);
        const uint32_t lo = (uint32_t)m;
        uint32_t entry = (128u - (lo >> 1)) | ((lo & 1u) << 7);
        if (ballot(bad)) entry = 0u;
        if (lane < lay.entries) *lay.entry(out_idx, out_w, row, lane) = (uint8_t)entry;
    }
}

struct WalkState {
    uint32_t cut;                       // experts whose key is at least this are resident
    int held;                           // how many
};

// a value that is the same in every lane, in a scalar register
__device__ __forceinline__ int uniform(int v)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_readfirstlane(v);
#else
    return v;
#endif
}

// set bits of the mask in front of this lane's
__device__ __forceinline__ int below(u64 mask)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
#else
    (void)mask;
    return 0;
#endif
}

// The n-th expert (from 0) of a set with more than n: in0 says whether expert `lane` is in it, in1 expert `lane` + 64.
__device__ __forceinline__ int nth(bool in0, bool in1, int n)
{
    const u64 g0 = ballot(in0), g1 = ballot(in1);
    const int n0 = __popcll(g0);
    if (n < n0) return __ffsll((long long)ballot(in0 & (below(g0) == n))) - 1;
    return 63 + __ffsll((long long)ballot(in1 & (n0 + below(g1) == n)));
}

// One stretch [t0, t1) of a trace from the state in (keys, st).  keys[e] = (step of last use + 1) << 7 | e, 0 =
// never used; slots 128 + lane take the writes of lanes without an expert.  STORE: marks, misses and
// the ids of steps without a list are written.  FULL: K >= C.  Returns the misses that this lane counted.
template <bool WIDE, bool FULL, bool STORE>
__device__ __forceinline__ uint32_t walk(const float *__restrict__ probs, int64_t s, int64_t T, int64_t t0, int64_t t1, int N, int C, float factor,
                    const RowLayout lay, int32_t *out_idx, float *out_w, uint8_t *out_miss, uint32_t *keys,
                    uint8_t *lists, WalkState &st)
{
    const int lane = threadIdx.x & 63, K = lay.K;
    const bool has = lane < lay.entries;
    uint32_t cut = st.cut;
    int held = st.held;
    uint32_t lane_misses = 0;
    uint32_t next[RR_BATCH];            // the lists of the next batch, a byte per lane and step
    typedef const __attribute__((address_space(1))) uint8_t *global_bytes;
    global_bytes list = (global_bytes)lay.entry(out_idx, out_w, s * T + t0, has ? lane : 0);
    int left = has ? (int)(t1 - t0) : 0;
    auto fetch = [&] {
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("" : "+v"(list));  // sixteen addresses held in front of the loop would be spilled
#endif
#pragma unroll
        for (int a = 0; a < RR_BATCH; ++a) {
            next[a] = a < left ? *list : 0u;
            list += 4 * K;
        }
        left -= RR_BATCH;
    };
    fetch();
    uint32_t k0 = keys[lane], k1 = WIDE ? keys[lane + 64] : 0u;
    for (int64_t tb = t0; tb < t1; tb += RR_BATCH) {
#pragma unroll
        for (int a = 0; a < RR_BATCH; ++a) lists[a * 64 + lane] = (uint8_t)next[a];
        asm volatile("" ::: "memory");
        const int n = (int)(t1 - tb < RR_BATCH ? t1 - tb : RR_BATCH);
        fetch();
        // bit a: step tb + a has no list
        const uint32_t no_list = (uint32_t)ballot(lane < RR_BATCH && lists[lane * 64] == lists[lane * 64 + 1]);
        uint32_t b = lists[lane];
        uint32_t kr = keys[b & 127u];
        uint32_t o_lo = 0, o_hi = 0, o_miss = 0;              // marks and misses of step tb + lane
        for (int a = 0; a < n; ++a) {
            const uint32_t t1u = (uint32_t)(tb + a) + 1u, stamp = t1u << 7;
            const uint32_t b_next = lists[(a + 1) * 64 + lane];        // behind the last step: not used
            const bool boost = b > 127u;
            const bool live = has & ((kr >= cut) == boost);
            const u64 live_mask = ballot(live);
            const bool chosen = live & (below(live_mask) < K);
            u64 sel = ballot(chosen);
            uint32_t e = b & 127u, slot = chosen ? e : 128u + (uint32_t)lane;
            int n_sel = K, miss = __popcll(sel & ~ballot(boost));
            if (((no_list >> a) & 1u) | (__popcll(live_mask) < K)) {
                // K rounds of wavefront maximum over the boosted scores; an expert that is out, taken or never there, is a NaN:
                // no maximum takes it and nothing equals it, not even where the scores that are left are -inf
                const float *pr = probs + (s * T + tb + a) * N;
                const float OUT = __builtin_nanf("");
                const float p0 = lane < N ? pr[lane] : 0.f, p1 = WIDE && lane + 64 < N ? pr[lane + 64] : 0.f;
                const u64 res_lo = ballot(k0 >= cut), res_hi = WIDE ? ballot(k1 >= cut) : 0ull;
                float m0 = lane < N ? (k0 >= cut ? p0 * factor : p0) : OUT;
                float m1 = WIDE && lane + 64 < N ? (k1 >= cut ? p1 * factor : p1) : OUT;
                u64 sel_lo = 0ull, sel_hi = 0ull;
                for (int j = 0; j < K; ++j) {
                    const float m = wave_max(WIDE ? fmaxf(m0, m1) : m0);
                    const u64 b0 = ballot(m0 == m), b1 = WIDE ? ballot(m1 == m) : 0ull;
                    // (where only NaNs are left nothing equals the maximum, and one expert stands for them)
                    const int x = b0 ? __ffsll((long long)b0) - 1 : b1 ? 63 + __ffsll((long long)b1) : N < 64 ? N - 1 : 63;
                    if (lane == j) e = (uint32_t)x;
                    if (x == lane) m0 = OUT;
                    if (x == lane + 64) m1 = OUT;
                    if (x < 64) sel_lo |= 1ull << x;
                    else sel_hi |= 1ull << (x - 64);
                }
                sel = 0ull;
                slot = lane < K ? e : 128u + (uint32_t)lane;
                n_sel = __popcll(sel_lo) + __popcll(sel_hi);
                miss = __popcll(sel_lo & ~res_lo) + __popcll(sel_hi & ~res_hi);
                if (STORE) {
                    // two equal entries, then the ids; a row without marks is one of these
                    uint8_t *row = lay.entry(out_idx, out_w, s * T + tb + a, 0);
                    if (lane < 2) row[lane] = 0;
                    if (lane < K) row[2 + lane] = (uint8_t)e;
                }
            }
            // one wavefront: its LDS accesses are served in program order
            keys[slot] = stamp | e;
            asm volatile("" ::: "memory");
            kr = keys[b_next & 127u];
            k0 = keys[lane];
            if (WIDE) k1 = keys[lane + 64];
            b = b_next;
            if (lane == a) {
                o_lo = (uint32_t)sel;
                o_hi = (uint32_t)(sel >> 32);
                o_miss = (uint32_t)miss;
            }
            // The least recent go first, within a step the lower ids: whole steps while they fit, then the
            // lowest ids of one.  Where the step alone fills the cache, everything older goes.
            if (FULL && n_sel >= C) {
                held = C;
                cut = stamp;
                if (n_sel > C) cut |= (uint32_t)nth(k0 >= stamp, WIDE & (k1 >= stamp), n_sel - C);
            } else {
                held += miss;
                int drop = held - C;
                if (drop > 0) {
                    held = C;
                    uint32_t step = cut >> 7;
                    do {
                        const bool in0 = (k0 >= cut) & ((k0 >> 7) == step), in1 = WIDE & (k1 >= cut) & ((k1 >> 7) == step);
                        const int n_g = __popcll(ballot(in0)) + (WIDE ? __popcll(ballot(in1)) : 0);
                        if (n_g <= drop) {
                            drop -= n_g;
                            cut = ++step << 7;
                        } else {
                            cut = (step << 7) | (uint32_t)nth(in0, in1, drop);
                            drop = 0;
                        }
                    } while (drop > 0 && step <= t1u);
                }
            }
        }
        lane_misses += o_miss;
        if (STORE && lane < n) {
            uint8_t *mk = lay.mark(out_w, s * T + tb + lane);
            const u64 marks = ((u64)o_hi << 32) | o_lo;
            for (int q = 0; q < lay.marks; ++q) mk[q] = (uint8_t)(marks >> (8 * q));
            out_miss[s * T + tb + lane] = (uint8_t)o_miss;
        }
    }
    st.cut = cut;
    st.held = held;
    return lane_misses;
}

template <bool WIDE, bool FULL>
__global__ __launch_bounds__(64 * RR_WAVES) void reroute_walk_kernel(const float *__restrict__ probs, int64_t T, int N, int C, float factor,
                                                                     RowLayout lay, int64_t stretch, int64_t warm, int32_t *out_idx,
                                                                     float *out_w, uint8_t *out_miss, u64 *__restrict__ out_total_miss)
{
    __shared__ uint32_t keys[RR_WAVES][192];
    __shared__ uint32_t first[RR_WAVES][128];                 // state the stretch was walked from, 0 = not resident
    __shared__ uint8_t lists[RR_WAVES][(RR_BATCH + 1) * 64];
    __shared__ uint32_t cuts[RR_WAVES];
    __shared__ int helds[RR_WAVES];
    __shared__ uint32_t misses[RR_WAVES];
    const int64_t s = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = uniform((int)threadIdx.x >> 6), waves = blockDim.x >> 6;
    const int64_t t0 = wave * stretch < T ? wave * stretch : T, t1 = t0 + stretch < T ? t0 + stretch : T;

    keys[wave][lane] = 0u;
    keys[wave][lane + 64] = 0u;
    const int64_t from = t0 > warm ? t0 - warm : 0;
    WalkState st{(uint32_t)(from + 1) << 7, 0};
    if (wave > 0 && t0 < t1) {
        walk<WIDE, FULL, false>(probs, s, T, from, t0, N, C, factor, lay, out_idx, out_w, out_miss, keys[wave], lists[wave], st);
    }
    __syncthreads();                    // the walks below may replace the list of a step that has none
    bool again = true;
    for (int pass = 0; pass <= waves; ++pass) {
        if (again) {
            for (int e = lane; e < 128; e += 64) {
                const uint32_t k = keys[wave][e] >= st.cut ? keys[wave][e] : 0u;
                keys[wave][e] = k;
                first[wave][e] = k;
            }
            const uint32_t m = walk<WIDE, FULL, true>(probs, s, T, t0, t1, N, C, factor, lay, out_idx, out_w, out_miss, keys[wave], lists[wave], st);
            uint32_t sum = m;
            for (int d = 32; d > 0; d >>= 1) sum += (uint32_t)__shfl_xor((int)sum, d, 64);
            if (lane == 0) {
                cuts[wave] = st.cut;
                helds[wave] = st.held;
                misses[wave] = sum;
            }
        }
        __syncthreads();
        // does the stretch start where the one before it ended?
        again = false;
        uint32_t k[2] = {0u, 0u};
        if (wave > 0 && t0 < t1) {
            const uint32_t c = (uint32_t)uniform((int)cuts[wave - 1]);
            bool differ = false;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t v = keys[wave - 1][lane + 64 * h];
                k[h] = v >= c ? v : 0u;
                differ = differ || k[h] != first[wave][lane + 64 * h];
            }
            again = ballot(differ) != 0ull;
            if (again) st = WalkState{c, uniform(helds[wave - 1])};
        }
        if (!__syncthreads_or(again ? 1 : 0)) break;
        if (again) {
            keys[wave][lane] = k[0];
            keys[wave][lane + 64] = k[1];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        u64 sum = 0;
        for (int q = 0; q < waves; ++q) sum += misses[q];
        out_total_miss[s] = sum;
    }
}

// one wavefront per step; the sum of the chosen probabilities is taken in the order of their places
__global__ __launch_bounds__(256) void reroute_weights_kernel(const float *__restrict__ probs, int64_t rows, int N, int renorm, RowLayout lay,
                                                              int32_t *out_idx, float *out_w)
{
    const int lane = threadIdx.x & 63, K = lay.K;
    const int64_t stride = (int64_t)gridDim.x * 4;
    for (int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); row < rows; row += stride) {
        const uint8_t *mk = lay.mark(out_w, row);
        const bool mine = lane < lay.entries && ((mk[lane >> 3] >> (lane & 7)) & 1) != 0;
        int e = 0;
        if (lane < lay.entries) e = *lay.entry(out_idx, out_w, row, lane) & 127;
        int id = lane < K ? lay.entry(out_idx, out_w, row, 0)[lane + 2] : 0;     // a step that had no list
        const u64 marks = ballot(mine);
        if (marks) {
#if defined(__HIP_DEVICE_COMPILE__)
            id = __builtin_amdgcn_ds_permute((mine ? below(marks) : 63) << 2, e);
#endif
        }
        const float p = lane < K && id < N ? probs[row * N + id] : 0.f;
        const float wgt = renorm ? p / wave_sum(p) : p;
        if (lane < K) {
            out_idx[row * K + lane] = id;
            out_w[row * K + lane] = wgt;
        }
    }
}

}  // namespace

remoe_status launch_reroute(const float *probs, int64_t S, int64_t T, int N, int K, int C, float factor, int renorm,
                            int32_t *idx, float *w, uint8_t *miss, uint64_t *total_miss, hipStream_t stream)
{
    if (S == 0) return REMOE_OK;
    const RowLayout lay(N, K);
    const int64_t rows = S * T;
    const int64_t row_blocks = ceil_div(rows, 4) < 8192 ? ceil_div(rows, 4) : 8192;
    // stretches of at least RR_MIN_STEPS, whole batches; the guessed state has forgotten the steps before the
    // warm-up after a few times the steps that fill the cache
    int64_t stretch = ceil_div(T, RR_WAVES);
    if (stretch < RR_MIN_STEPS) stretch = RR_MIN_STEPS;
    stretch = ceil_div(stretch, RR_BATCH) * RR_BATCH;
    const int waves = T > 0 ? (int)ceil_div(T, stretch) : 1;
    int64_t warm = RR_BATCH * ceil_div(16 + 12 * (int64_t)(C < N ? C : N) / K, RR_BATCH);
    if (warm > stretch) warm = stretch;
    u64 *total = reinterpret_cast<u64 *>(total_miss);
    if (rows > 0) {
        auto rank = N > 64 ? reroute_rank_kernel<true> : reroute_rank_kernel<false>;
        hipLaunchKernelGGL(rank, dim3((unsigned)row_blocks), dim3(256), 0, stream, probs, rows, N, factor, lay, idx, w);
    }
    auto walk_kernel = N > 64 ? (K >= C ? reroute_walk_kernel<true, true> : reroute_walk_kernel<true, false>)
                              : (K >= C ? reroute_walk_kernel<false, true> : reroute_walk_kernel<false, false>);
    hipLaunchKernelGGL(walk_kernel, dim3((unsigned)S), dim3(64 * waves), 0, stream, probs, T, N, C, factor, lay, stretch, warm, idx, w, miss, total);
    if (rows > 0) hipLaunchKernelGGL(reroute_weights_kernel, dim3((unsigned)row_blocks), dim3(256), 0, stream, probs, rows, N, renorm, lay, idx, w);
    return check_hip(hipGetLastError(), "reroute launch");
}

}  // namespace remoe
