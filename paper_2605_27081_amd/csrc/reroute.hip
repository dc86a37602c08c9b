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
//                          A trace is walked by up to 56 wavefronts at once, each on its own stretch from a
//                          guessed cache: a cold one warmed on the steps before the stretch.
//   reroute_check_kernel   every stretch but the first again, from the cache that the choices of the steps before it
//                          leave, until the cache holds only experts used inside the stretch: if every choice up to
//                          there is the one made from the guess, so are all that follow.  A stretch that fails sets its
//                          bit in the trace's word.
//                          The trace's last workgroup mends what failed: up to 16 wavefronts walk again at once, each as far as
//                          anything changes or to where the next one started, until no start differs from what arrives
//                          there, so the result is that of the single walk whatever the guesses were.  It then sums the misses.
//   reroute_group_kernel   short traces and those whose guesses are not likely to settle: up to 16 stretches in one workgroup,
//                          which compares their states in LDS.
//   reroute_weights_kernel ids and gate weights from the entries the walk marked.
// The lists and marks of a step live where its ids and weights will be (8 K bytes), so that no
// scratch memory is needed: entries r < 4 K in the id row, the marks (one bit per entry, K but at most 8 bytes) in front of
// the weight row and the other entries behind them.  There are fewer entries than bits, so the last bit of the marks is
// free: where it is set the step's K ids stand for the marks, a byte each in their place (K <= 8) or at the end of the
// weight row.  The bits of the stretches that failed are kept in the trace's total.  Lists are only written by the first kernel and marks only by the stretch's own
// wavefront, so that a wavefront may warm up on the lists of the stretch before while that one is walked.
//
// 16 traces x 4096 steps, 128 experts, top-8, C = 4: 7.5 ms as one walk of K maxima per step and wavefront, 0.19 ms with
// 16 stretches of a trace in one workgroup (walk 140 us, bound by the instructions that 16 wavefronts issue on one
// compute unit), 0.102 ms with 52 stretches of 80 steps over the chip: lists 37, walk 42 (one wavefront per SIMD, bound by
// the latency of a step), check 14, weights 12 us.  With C = 32, a bonus of 4 and scores more alike from step to step (AR(1) of
// 0.9) about 23 of 51 stretches fail: 0.31 ms; mended by one wavefront, one stretch after the other, 1.1 ms, and 0.44 ms in one workgroup.
#include <type_traits>

#include "common.h"
#include "topk.h"

namespace remoe {

namespace {

constexpr int RR_GROUP = 16;            // stretches of a trace that one workgroup walks at once
constexpr int RR_GROUP_STEPS = 512;     // see launch_reroute
constexpr int RR_STRETCHES = 56;        // of a trace, walked by several: a bit each in the trace's word, whose last eight bits
                                        // count the workgroups that have checked theirs
constexpr int RR_BLOCK_WAVES = 4;
constexpr int RR_MIN_STEPS = 32;        // a shorter stretch is not worth its warm-up
constexpr int RR_BATCH = 16;            // steps whose lists are staged in LDS at a time
constexpr int RR_MAX_ENTRIES = 63;      // see reroute_rank_kernel

struct RowLayout {
    int K, marks, entries;              // marks: bytes in front of the weight row
    __host__ __device__ RowLayout(int N, int K_) : K(K_), marks(K_ < 8 ? K_ : 8)
    {
        entries = K > 8 ? 7 * K - marks : 8 * K - marks;       // more than 8 ids have a place of their own
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
    __device__ bool is_ids(unsigned long long m) const { return (m >> (8 * marks - 1)) & 1ull; }
    // byte of id j of a row of ids, K > 8
    __device__ uint8_t *id(float *w, int64_t row, int j) const { return reinterpret_cast<uint8_t *>(w + row * K) + 3 * K + j; }
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

// The marks of a row (weights are four-byte aligned, not more).
__device__ __forceinline__ u64 load_marks(const RowLayout &lay, float *w, int64_t row)
{
    const uint8_t *mk = lay.mark(w, row);
    const uint32_t *words = reinterpret_cast<const uint32_t *>(mk);
    if (lay.marks == 8) return ((u64)words[1] << 32) | words[0];
    if (lay.marks == 4) return words[0];
    u64 m = 0ull;
    for (int q = 0; q < lay.marks; ++q) m |= (u64)mk[q] << (8 * q);
    return m;
}

// The cut behind which `drop` > 0 fewer of the experts from `cut` on are: whole steps while they fit, then the lowest ids of one.
// `last`: no key is of a later step.
template <bool WIDE>
__device__ __forceinline__ uint32_t evict(uint32_t k0, uint32_t k1, uint32_t cut, int drop, uint32_t last)
{
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
    } while (drop > 0 && step <= last);
    return cut;
}

struct WalkEnd {
    int64_t t;                          // first step not walked
    uint32_t misses;                    // counted by this lane
    bool differ;                        // CHECK: some choice was not the stored one
    bool settled;                       // CHECK: the stored choices stand from here to the end of the stretch
};

// Steps [t0, t1) of a trace, t0 and stretch multiples of RR_BATCH, from the state in (keys, st).  keys[e] = (step of last
// use + 1) << 7 | e, 0 = never used; slots 128 + lane take the writes of lanes without an expert.
// STORE: marks and misses are written.  CHECK: they are compared with the stored ones first, and the walk ends
// behind a batch when the cache is full and all that is resident was last used since the last difference and since the start of
// the current stretch: the walk that stored the choices then held the same, and from there on they stand.  (The cut says
// less: it moves with evictions only, and a cache that has stopped missing would never be seen to be renewed.)
// Without STORE it also ends at a difference.  FULL: K >= C.
template <bool WIDE, bool FULL, bool STORE, bool CHECK>
__device__ __forceinline__ WalkEnd walk(const float *__restrict__ probs, int64_t s, int64_t T, int64_t t0, int64_t t1, int64_t stretch, int N, int C,
                    float factor, const RowLayout lay, const int32_t *out_idx, float *out_w, uint8_t *out_miss, uint32_t *keys,
                    uint8_t *lists, WalkState &st)
{
    const int lane = threadIdx.x & 63, K = lay.K;
    const bool has = lane < lay.entries;
    uint32_t cut = st.cut;
    int held = st.held;
    int64_t same_from = t0, stretch_end = t0 - t0 % stretch + stretch;
    bool differ = false;
    uint32_t lane_misses = 0;
    uint32_t next[RR_BATCH];            // the lists of the next batch, a byte per lane and step
    typedef const __attribute__((address_space(1))) uint8_t *global_bytes;
    global_bytes list = (global_bytes)lay.entry(const_cast<int32_t *>(out_idx), out_w, s * T + t0, has ? lane : 0);
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
        u64 stored = 0ull;                                    // CHECK: marks and misses of step tb + lane
        uint32_t stored_miss = 0;
        if (CHECK && lane < n) {
            stored = load_marks(lay, out_w, s * T + tb + lane);
            stored_miss = out_miss[s * T + tb + lane];
        }
        // bit a: step tb + a has no list
        const uint32_t no_list = (uint32_t)ballot(lane < RR_BATCH && lists[lane * 64] == lists[lane * 64 + 1]);
        uint32_t b = lists[lane];
        uint32_t kr = keys[b & 127u];
        uint32_t ids_differ = 0;                              // CHECK, K > 8: bit a in any lane
        uint32_t o_lo = 0, o_hi = 0, o_miss = 0;              // marks (or ids) and misses of step tb + lane
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
                if (K <= 8) {
                    for (int j = 0; j < K; ++j) sel |= (u64)(uint32_t)__shfl((int)e, j, 64) << (8 * j);
                } else if (lane < K) {
                    uint8_t *id = lay.id(out_w, s * T + tb + a, lane);
                    if (CHECK && *id != (uint8_t)e) ids_differ |= 1u << a;
                    if (STORE) *id = (uint8_t)e;
                }
                sel |= 1ull << (8 * lay.marks - 1);
                slot = lane < K ? e : 128u + (uint32_t)lane;
                n_sel = __popcll(sel_lo) + __popcll(sel_hi);
                miss = __popcll(sel_lo & ~res_lo) + __popcll(sel_hi & ~res_hi);
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
                if (held > C) {
                    cut = evict<WIDE>(k0, k1, cut, held - C, t1u);
                    held = C;
                }
            }
        }
        lane_misses += o_miss;
        const u64 marks = ((u64)o_hi << 32) | o_lo;
        const int64_t row = s * T + tb + lane;
        if (CHECK) {
            u64 others = ballot(lane < n && (stored != marks || stored_miss != o_miss));
            if (K > 8) {
                for (int a = 0; a < n; ++a)
                    if (ballot((ids_differ >> a) & 1u)) others |= 1ull << a;
            }
            if (tb >= stretch_end) {
                same_from = stretch_end;
                stretch_end += stretch;
            }
            if (others) {
                differ = true;
                same_from = tb + 64 - __clzll((long long)others);
            }
        }
        if (STORE && lane < n) {
            uint8_t *mk = lay.mark(out_w, row);
            for (int q = 0; q < lay.marks; ++q) mk[q] = (uint8_t)(marks >> (8 * q));
            out_miss[row] = (uint8_t)o_miss;
        }
        if (CHECK) {
            bool settled = false;
            if (held == C) {
                const uint32_t r0 = k0 >= cut ? k0 : ~0u, r1 = WIDE && k1 >= cut ? k1 : ~0u;
                settled = (int64_t)(wave_min_u32(r1 < r0 ? r1 : r0) >> 7) > same_from;
            }
            if (settled || (differ && !STORE)) {
                st = WalkState{cut, held};
                return WalkEnd{tb + n, lane_misses, differ, settled};
            }
        }
    }
    st.cut = cut;
    st.held = held;
    return WalkEnd{t1, lane_misses, differ, false};
}

// The state in front of step t from the choices stored for the steps before it: walking back, the first C experts met,
// within a step the higher ids first.  Four steps at a time are entered without looking (the latest use of an expert is its
// largest key) before the experts are counted; the next batch is requested once the first four did not do.
template <bool WIDE>
__device__ __forceinline__ WalkState state_before(int64_t s, int64_t T, int64_t t, int C, const RowLayout lay, const int32_t *out_idx, float *out_w,
                                                  uint32_t *keys)
{
    const int lane = threadIdx.x & 63, K = lay.K;
    const bool has = lane < lay.entries;
    keys[lane] = 0u;
    keys[lane + 64] = 0u;
    uint32_t next[RR_BATCH];
    u64 next_marks = 0ull;
    auto fetch = [&](int64_t tb) {
#pragma unroll
        for (int a = 0; a < RR_BATCH; ++a)
            next[a] = has && a < tb ? *lay.entry(const_cast<int32_t *>(out_idx), out_w, s * T + tb - 1 - a, lane) : 0u;
        next_marks = lane < RR_BATCH && lane < tb ? load_marks(lay, out_w, s * T + tb - 1 - lane) : 0ull;
    };
    fetch(t);
    int count = 0;
    for (int64_t tb = t; tb > 0; tb -= RR_BATCH) {
        uint32_t entry[RR_BATCH];
#pragma unroll
        for (int a = 0; a < RR_BATCH; ++a) entry[a] = next[a];
        const u64 marks = next_marks;
#pragma unroll
        for (int q = 0; q < RR_BATCH; q += 4) {
#pragma unroll
            for (int a = q; a < q + 4; ++a) {                              // (no marks in front of the trace: nothing is chosen there)
                const u64 m = ((u64)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(marks >> 32), a) << 32) |
                              (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)marks, a);
                uint32_t e = entry[a];
                bool chosen = (m >> lane) & 1ull;
                if (lay.is_ids(m)) {
                    e = K <= 8 ? (uint32_t)(m >> (8 * (lane & 7))) : lane < K ? *lay.id(out_w, s * T + tb - 1 - a, lane) : 0u;
                    chosen = lane < K;
                }
                e &= 127u;
                if (chosen) atomicMax(&keys[e], ((uint32_t)(tb - a) << 7) | e);       // step tb - 1 - a, plus one
            }
            asm volatile("" ::: "memory");
            const uint32_t k0 = keys[lane], k1 = WIDE ? keys[lane + 64] : 0u;
            const int now = __popcll(ballot(k0 != 0u)) + (WIDE ? __popcll(ballot(k1 != 0u)) : 0);
            if (now < C) {
                count = now;
                if (q == 0) fetch(tb - RR_BATCH);
                continue;
            }
            for (uint32_t step = (uint32_t)(tb - q);; --step) {               // the last of the four in which the cache is full
                const bool in0 = (k0 >> 7) == step, in1 = WIDE & ((k1 >> 7) == step);
                count += __popcll(ballot(in0)) + (WIDE ? __popcll(ballot(in1)) : 0);
                if (count >= C) return WalkState{(step << 7) | (count > C ? (uint32_t)nth(in0, in1, count - C) : 0u), C};
            }
        }
    }
    return WalkState{1u << 7, count};
}

// A whole trace in one workgroup, its stretches compared by their states: first state against last state of the one before, key for
// key; those that differ are walked again from that state until all agree.
template <bool WIDE, bool FULL>
__global__ __launch_bounds__(64 * RR_GROUP) void reroute_group_kernel(const float *__restrict__ probs, int64_t T, int N, int C, float factor,
                                                                     RowLayout lay, int64_t stretch, int64_t warm, const int32_t *out_idx,
                                                                     float *out_w, uint8_t *out_miss, u64 *__restrict__ out_total_miss)
{
    __shared__ uint32_t keys[RR_GROUP][192];
    __shared__ uint32_t first[RR_GROUP][128];                 // state the stretch was walked from, 0 = not resident
    __shared__ uint8_t lists[RR_GROUP][(RR_BATCH + 1) * 64];
    __shared__ uint32_t cuts[RR_GROUP];
    __shared__ int helds[RR_GROUP];
    __shared__ uint32_t misses[RR_GROUP];
    const int64_t s = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = uniform((int)threadIdx.x >> 6), waves = blockDim.x >> 6;
    const int64_t t0 = wave * stretch < T ? wave * stretch : T, t1 = t0 + stretch < T ? t0 + stretch : T;

    keys[wave][lane] = 0u;
    keys[wave][lane + 64] = 0u;
    const int64_t from = t0 > warm ? t0 - warm : 0;
    WalkState st{(uint32_t)(from + 1) << 7, 0};
    if (wave > 0 && t0 < t1) {
        walk<WIDE, FULL, false, false>(probs, s, T, from, t0, stretch, N, C, factor, lay, out_idx, out_w, out_miss, keys[wave], lists[wave], st);
    }
    bool again = true;
    for (int pass = 0; pass <= waves; ++pass) {
        if (again) {
            for (int e = lane; e < 128; e += 64) {
                const uint32_t k = keys[wave][e] >= st.cut ? keys[wave][e] : 0u;
                keys[wave][e] = k;
                first[wave][e] = k;
            }
            uint32_t sum = walk<WIDE, FULL, true, false>(probs, s, T, t0, t1, stretch, N, C, factor, lay, out_idx, out_w, out_miss, keys[wave], lists[wave], st).misses;
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

template <bool WIDE, bool FULL>
__global__ __launch_bounds__(64 * RR_BLOCK_WAVES) void reroute_walk_kernel(const float *__restrict__ probs, int64_t T, int N, int C, float factor,
                                                                           RowLayout lay, int64_t stretch, int64_t warm, const int32_t *out_idx,
                                                                           float *out_w, uint8_t *out_miss, u64 *__restrict__ out_total_miss)
{
    __shared__ uint32_t keys[RR_BLOCK_WAVES][192];
    __shared__ uint8_t lists[RR_BLOCK_WAVES][(RR_BATCH + 1) * 64];
    const int lane = threadIdx.x & 63, wave = uniform((int)threadIdx.x >> 6);
    const int64_t s = blockIdx.y, t0 = ((int64_t)blockIdx.x * RR_BLOCK_WAVES + wave) * stretch, t1 = t0 + stretch < T ? t0 + stretch : T;
    if (t0 == 0 && lane == 0) out_total_miss[s] = 0ull;               // no stretch has failed so far
    if (t0 >= T) return;
    keys[wave][lane] = 0u;
    keys[wave][lane + 64] = 0u;
    const int64_t from = t0 > warm ? t0 - warm : 0;
    WalkState st{(uint32_t)(from + 1) << 7, 0};
    if (t0 > 0) {
        walk<WIDE, FULL, false, false>(probs, s, T, from, t0, stretch, N, C, factor, lay, out_idx, out_w, out_miss, keys[wave], lists[wave], st);
        for (int e = lane; e < 128; e += 64) keys[wave][e] = keys[wave][e] >= st.cut ? keys[wave][e] : 0u;
    }
    walk<WIDE, FULL, true, false>(probs, s, T, t0, t1, stretch, N, C, factor, lay, out_idx, out_w, out_miss, keys[wave], lists[wave], st);
}

// The first `checkers` wavefronts of a workgroup check a stretch each; the workgroup that is the last of its trace to be done mends and
// sums.  (Marks and misses are only read until then, and the bits of the stretches that failed arrive with the count.)
// Mending: up to 16 wavefronts, each from a stretch that failed to where the next one's first is, all at once from the states that the
// stored choices leave in front of theirs; where a wavefront does not settle, the next one's state is compared with the one it
// arrives at, and those that differ walk again, until none does.  A wavefront that settles has left the state behind it as it was.
template <bool WIDE, bool FULL>
__global__ __launch_bounds__(64 * RR_GROUP) void reroute_check_kernel(const float *__restrict__ probs, int64_t T, int N, int C, float factor,
                                                                      RowLayout lay, int64_t stretch, int checkers, const int32_t *out_idx,
                                                                      float *out_w, uint8_t *out_miss, u64 *__restrict__ out_total_miss)
{
    __shared__ uint32_t keys[RR_GROUP][192];
    __shared__ uint32_t first[RR_GROUP][128];                 // state the wavefront walked from, 0 = not resident
    __shared__ uint8_t lists[RR_GROUP][(RR_BATCH + 1) * 64];
    __shared__ uint32_t cuts[RR_GROUP];
    __shared__ int helds[RR_GROUP];
    __shared__ bool arrived[RR_GROUP];                        // at its last step, without having settled
    __shared__ u64 part[RR_GROUP], word;
    const int lane = threadIdx.x & 63, wave = uniform((int)threadIdx.x >> 6);
    const int which = 1 + (int)blockIdx.x * checkers + wave;
    const int64_t s = blockIdx.y;
    bool differ = false;
    if (wave < checkers && which * stretch < T) {
        const int64_t t0 = which * stretch, t1 = t0 + stretch < T ? t0 + stretch : T;
        WalkState st = state_before<WIDE>(s, T, t0, C, lay, out_idx, out_w, keys[wave]);
        differ = walk<WIDE, FULL, false, true>(probs, s, T, t0, t1, stretch, N, C, factor, lay, out_idx, out_w, out_miss, keys[wave], lists[wave], st).differ;
    }
    if (lane == 0) part[wave] = differ ? 1ull << which : 0ull;
    __syncthreads();
    if (threadIdx.x == 0) {
        u64 mine = 1ull << 56;
        for (int q = 0; q < RR_GROUP; ++q) mine |= part[q];
        word = mine + atomicAdd(&out_total_miss[s], mine);
    }
    __syncthreads();
    if ((word >> 56) != gridDim.x) return;
    const u64 failed = word & ((1ull << 56) - 1ull);
    if (failed) {
        const int n_failed = __popcll(failed), waves = n_failed < RR_GROUP ? n_failed : RR_GROUP;
        // where wavefront w starts: at a failed stretch each, or, if there are more of them, evenly over the rest of the trace
        auto start = [&](int w) {
            if (w >= waves) return T;
            u64 m = failed;
            for (int q = n_failed <= RR_GROUP ? w : 0; q > 0; --q) m &= m - 1ull;
            const int64_t t = (int64_t)(__ffsll((long long)m) - 1) * stretch;
            return n_failed <= RR_GROUP ? t : t + (T - t) / RR_BATCH * w / RR_GROUP * RR_BATCH;
        };
        const bool takes_part = wave < waves;
        const int64_t t0 = start(wave), t1 = start(wave + 1);
        WalkState st{0u, 0};
        if (takes_part) {
            st = state_before<WIDE>(s, T, t0, C, lay, out_idx, out_w, keys[wave]);
            for (int e = lane; e < 128; e += 64) first[wave][e] = keys[wave][e] >= st.cut ? keys[wave][e] : 0u;
        }
        bool again = takes_part;
        for (int pass = 0; pass <= waves; ++pass) {
            __syncthreads();                                  // nobody reads what the wavefronts write now
            bool open = again;
            for (int64_t t = t0; again;) {
                const WalkEnd end = walk<WIDE, FULL, true, true>(probs, s, T, t, t1, stretch, N, C, factor, lay, out_idx, out_w, out_miss, keys[wave], lists[wave], st);
                open = !end.settled;
                if (open || pass > 0) break;
                // every stretch that it entered is done; its own steps fill the cache in front of the next that failed
                u64 left = failed & (~0ull << (uniform((int)((end.t - 1) / stretch)) + 1));
                if (!left) break;
                t = (int64_t)uniform(__ffsll((long long)left) - 1) * stretch;
                if (t >= t1) break;
                st = state_before<WIDE>(s, T, t, C, lay, out_idx, out_w, keys[wave]);
            }
            if (lane == 0) {
                cuts[wave] = st.cut;
                helds[wave] = st.held;
                arrived[wave] = open;
            }
            __syncthreads();
            again = false;
            uint32_t k[2] = {0u, 0u};
            if (takes_part && wave > 0 && arrived[wave - 1]) {
                const uint32_t c = (uint32_t)uniform((int)cuts[wave - 1]);
                bool other = false;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint32_t v = keys[wave - 1][lane + 64 * h];
                    k[h] = v >= c ? v : 0u;
                    other = other || k[h] != first[wave][lane + 64 * h];
                }
                again = ballot(other) != 0ull;
                if (again) st = WalkState{c, uniform(helds[wave - 1])};
            }
            if (!__syncthreads_or(again ? 1 : 0)) break;
            if (again) {
#pragma unroll
                for (int h = 0; h < 2; ++h) keys[wave][lane + 64 * h] = first[wave][lane + 64 * h] = k[h];
            }
        }
    }
    __syncthreads();
    u64 sum = 0;
    for (int64_t t = threadIdx.x; t < T; t += 64 * RR_GROUP) sum += out_miss[s * T + t];
    for (int d = 32; d > 0; d >>= 1) sum += (u64)__shfl_xor((unsigned long long)sum, d, 64);
    if (lane == 0) part[wave] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        sum = 0;
        for (int q = 0; q < RR_GROUP; ++q) sum += part[q];
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
        const u64 m = load_marks(lay, out_w, row);
        const bool ids = lay.is_ids(m);
        int e = 0, id = (int)(m >> (8 * (lane & 7))) & 127;
        if (lane < lay.entries) e = *lay.entry(out_idx, out_w, row, lane) & 127;
        if (K > 8 && lane < K) id = *lay.id(out_w, row, lane) & 127;
        if (!ids) {
#if defined(__HIP_DEVICE_COMPILE__)
            id = __builtin_amdgcn_ds_permute(((m >> lane) & 1ull ? below(m) : 63) << 2, e);
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
    if (C > N) C = N;                   // nothing is evicted either way, and a cache of N can be seen to be full
    const RowLayout lay(N, K);
    const int64_t rows = S * T;
    const int64_t row_blocks = ceil_div(rows, 4) < 8192 ? ceil_div(rows, 4) : 8192;
    // The guessed state has forgotten the steps before the warm-up after a few times the steps that fill the cache.
    // Stretches are whole batches and not shorter than that, so that the warm-up at most doubles the work.
    const int64_t warm = RR_BATCH * ceil_div(16 + 12 * (int64_t)C / K, RR_BATCH);
    // One workgroup per trace (16 stretches, one launch, states compared in LDS) against several (up to 56 stretches, a second launch
    // that walks part of every stretch again to check it), whole calls of 128 experts in us, S traces x T steps, K, C:
    //   16 x 256, 8, 4     35 / 43       16 x 1024, 8, 4    64 / 52      60 x 4096, 8, 4    295 / 230
    //   16 x 512, 8, 4     44 / 46       16 x 640, 8, 4     51 / 48      16 x 4096, 4, 32   248 / 164
    //   16 x 1024, 4, 32  110 / 127      16 x 2048, 4, 32  155 / 140     60 x 2048, 8, 64   262 / 248
    //   16 x 4096, 2, 64  487 / 549      16 x 4096, 2, 32  271 / 234     60 x 4096, 2, 60   580 / 653
    // (bonus 1.5, rho 0.8).  A warm-up longer than a sixteenth of the trace leaves too few stretches for the second way to gain.
    // Where guesses do not settle, as with a strong bonus and a cache of more than half of the experts, both walk most of the trace again
    // several times, 16 wavefronts at once, and the second way has walked it once more before.  1900 calls of 16 traces of AR(1) scores
    // (16 to 128 experts, C = 4 to 64, bonus 1 to 4, rho 0.5 to 0.9), time of the second way against the first, geometric mean and worst:
    //   bonus 2.5 or 4, C > N / 2, up to 64 warm-ups  0.98, 1.41 (two of five calls lose)     the same, longer traces  0.54, 0.88
    //   bonus 2.5 or 4, C <= N / 2  0.68, 1.32 (one of 25 loses)                              bonus 1 or 1.5, any C < N  0.66, 1.28 (one of 70)
    // A cache of all experts settles when the last of them has been used: 1.0 to 1.3, and the states are what has to be compared.
    const bool sticky = factor > 2.0f && 2 * C > N;
    const bool group = T <= RR_GROUP_STEPS || T <= RR_GROUP * warm * (sticky ? 4 : 1) || C == N;
    int64_t stretch = ceil_div(T, group ? RR_GROUP : RR_STRETCHES);
    if (stretch < RR_MIN_STEPS) stretch = RR_MIN_STEPS;
    if (stretch < warm && !group) stretch = warm;
    stretch = ceil_div(stretch, RR_BATCH) * RR_BATCH;
    const int64_t n_stretch = ceil_div(T, stretch);
    // few checking wavefronts in a workgroup (the others wait to mend) as long as the workgroups, one to a compute unit, run at once
    int checkers = 4;
    while (checkers < RR_GROUP && S * ceil_div(n_stretch - 1, checkers) > 256) checkers *= 2;
    u64 *total = reinterpret_cast<u64 *>(total_miss);
    if (rows > 0) {
        auto rank = N > 64 ? reroute_rank_kernel<true> : reroute_rank_kernel<false>;
        hipLaunchKernelGGL(rank, dim3((unsigned)row_blocks), dim3(256), 0, stream, probs, rows, N, factor, lay, idx, w);
    }
    auto walk_all = [&](auto wide, auto full) {
        constexpr bool W = decltype(wide)::value, F = decltype(full)::value;
        if (group || n_stretch == 1) {
            const int waves = T > 0 ? (int)n_stretch : 1;
            hipLaunchKernelGGL((reroute_group_kernel<W, F>), dim3((unsigned)S), dim3(64 * waves), 0, stream, probs, T, N, C, factor, lay, stretch,
                               warm < stretch ? warm : stretch, idx, w, miss, total);
            return;
        }
        for (int64_t s0 = 0; s0 < S; s0 += 65535) {               // traces in the grid's second dimension
            const unsigned n_s = (unsigned)(S - s0 < 65535 ? S - s0 : 65535);
            const float *p = probs + s0 * T * N;
            int32_t *i = idx + s0 * T * K;
            float *v = w + s0 * T * K;
            uint8_t *m = miss + s0 * T;
            hipLaunchKernelGGL((reroute_walk_kernel<W, F>), dim3((unsigned)ceil_div(n_stretch, RR_BLOCK_WAVES), n_s), dim3(64 * RR_BLOCK_WAVES), 0, stream,
                               p, T, N, C, factor, lay, stretch, warm, i, v, m, total + s0);
            hipLaunchKernelGGL((reroute_check_kernel<W, F>), dim3((unsigned)ceil_div(n_stretch - 1, checkers), n_s), dim3(64 * RR_GROUP), 0, stream,
                               p, T, N, C, factor, lay, stretch, checkers, i, v, m, total + s0);
        }
    };
    const std::true_type yes;
    const std::false_type no;
    if (N > 64) K >= C ? walk_all(yes, yes) : walk_all(yes, no);
    else K >= C ? walk_all(no, yes) : walk_all(no, no);
    if (rows > 0) hipLaunchKernelGGL(reroute_weights_kernel, dim3((unsigned)row_blocks), dim3(256), 0, stream, probs, rows, N, renorm, lay, idx, w);
    return check_hip(hipGetLastError(), "reroute launch");
}

}  // namespace remoe
