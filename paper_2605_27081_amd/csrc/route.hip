// Router kernel: fp32-accurate logits on the matrix cores, then the top-k and softmax in the same workgroup.
//
// Computes the paper's routing step (Sec. 3.1): P_t = Softmax(h_t^T theta_gate), E_t = Top-K(P_t).
// One workgroup of 4 wavefronts owns a block of tokens and all N_r <= 128 experts.  The experts are cut
// into NE tiles of 32 (NE = 1, 2 or 4); wavefront w computes expert tile w % NE for MT tiles of 32
// tokens, the 4 / NE wavefronts of one expert tile taking different tokens, so a workgroup owns
// 32 * MT * 4 / NE tokens and every token's full logit row ends in one workgroup.  (Layers of few tokens spread the work
// further: route_few_kernel below.)
//
// Logits.  The gate weights are fp32 and the logits must carry fp32 accuracy (near ties decide
// which experts run).  For fp32 hidden states the products run on v_mfma_f32_32x32x2_f32.  For bf16
// hidden states every x is already exact in bf16, and each fp32 weight is split on the fly into three
// bf16 pieces w = hi + mid + lo (each the round-to-nearest of what the previous ones left, 24+
// significand bits in all), so x*hi, x*mid and x*lo are exact fp32 products and three
// v_mfma_f32_32x32x16_bf16 with fp32 accumulation replace sixteen fp32 MFMA steps.
//
// Data path.  Slices of 32 k-values of the gate matrix and of the tokens move global -> LDS directly, in
// full lines, into a ring of 3 or 4 stages (no staging registers, one barrier per slice).  A wavefront reads
// its expert tile's fp32 weights and its token rows one slice ahead of the MFMAs and splits the weights in
// registers.  What bounds it: the split, 44 vector instructions per 3 MT MFMAs, repeated by every workgroup.
// (Loading each lane's weights straight into the operand registers needs no LDS for them, but the 64 lanes of
// such a load touch 32 rows: 34 us against 27 us for 32 tokens, 112 against 101 us for 65,536.)  Before, the
// split pieces went through LDS, between two barriers: 72 us and 113 us, with an insertion top-k by two
// lanes per token.
//
// Top-k.  The logits are parked in LDS, one padded row per token.  Eight neighbouring lanes share a
// token, each holding NE * 4 consecutive experts in registers.  K rounds (one more when the margin is
// asked for) each take the maximum over the eight lanes and the lowest id that holds it, and strike
// that id out; lane j keeps the winner of round j and writes it.
#include "common.h"
#include "lds_copy.h"

namespace remoe {

namespace {

constexpr int RT_BLOCK = 256;          // threads
constexpr int RT_BK = 32;              // k-values per slice
constexpr int RT_LANES = 8;            // lanes per token in the top-k
constexpr int RT_PARTS = 8;            // shares of an fp32 reduction at most

// 128-byte rows (fp32 values) are 8 chunks of 16 bytes; chunk c of row r lives in row slot r ^ ((r >> 3) & 1)
// at chunk position c ^ (r & 7): 16 consecutive rows of one logical chunk cover all banks once.
__device__ __forceinline__ int slot_f32(int r, int c) { return ((r ^ ((r >> 3) & 1)) << 3) + (c ^ (r & 7)); }
// 64-byte rows (bf16 tokens) are 4 chunks; chunk c of row r sits at chunk position c ^ ((r >> 2) & 3)
__device__ __forceinline__ int slot_bf16(int r, int c) { return r * 4 + (c ^ ((r >> 2) & 3)); }

// round-to-nearest-even bf16 pieces of two neighbouring fp32 weights: w = hi + mid + lo up to 2^-24
// relative, each piece packed the way the MFMA operand holds it (first weight in the low half); three
// packed conversions (v_cvt_pk_bf16_f32) for the pair
__device__ __forceinline__ void split3_pair(float w0, float w1, uint32_t &hi, uint32_t &mid, uint32_t &lo)
{
    hi = pack_bf16x2(w0, w1);
    const float r0 = w0 - __uint_as_float(hi << 16), r1 = w1 - __uint_as_float(hi & 0xFFFF0000u);
    mid = pack_bf16x2(r0, r1);
    const float q0 = r0 - __uint_as_float(mid << 16), q1 = r1 - __uint_as_float(mid & 0xFFFF0000u);
    lo = pack_bf16x2(q0, q1);
}

// Logit rows in LDS.  The lanes of a token read 16-byte pieces of their own NE * 4 consecutive experts;
// 4 floats of padding behind every 32 experts (and none behind a row of 32) spread the eight lanes of a
// token and of its neighbours over the banks.
template <int NE> struct LogitLayout {
    static constexpr int STRIDE = NE * 36 + (NE == 1 ? 0 : 4);
    __device__ static __forceinline__ int at(int row, int col) { return row * STRIDE + col + 4 * (col >> 5); }
};

// Operands of one slice in registers: read from the stage (xs: token rows, wst: the 32 rows of this
// wavefront's expert tile) one slice ahead of the MFMAs that use them.
template <int MT, typename XT> struct Frags;

template <int MT> struct Frags<MT, bf16_t> {
    floatx4_t w[4];            // this lane's eight k values of k-step ks: 16 ks + 8 lh + {0..7}
    bf16x8_t a[2][MT];
    __device__ __forceinline__ void read(const u32x4_t *xs, const u32x4_t *wst, int row0, int li, int lh)
    {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
            for (int i = 0; i < 2; ++i) w[2 * ks + i] = *reinterpret_cast<const floatx4_t *>(&wst[slot_f32(li, 4 * ks + 2 * lh + i)]);
#pragma unroll
            for (int m = 0; m < MT; ++m) a[ks][m] = *reinterpret_cast<const bf16x8_t *>(&xs[slot_bf16(row0 + m * 32 + li, 2 * ks + lh)]);
        }
    }
    __device__ __forceinline__ void mfma(floatx16_t (&acc)[MT]) const
    {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            u32x4_t piece[3];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const floatx4_t w4 = w[2 * ks + (q >> 1)];
                uint32_t hi, mid, lo;
                split3_pair(w4[2 * (q & 1)], w4[2 * (q & 1) + 1], hi, mid, lo);
                piece[0][q] = hi;
                piece[1][q] = mid;
                piece[2][q] = lo;
            }
#pragma unroll
            for (int pc = 0; pc < 3; ++pc)
#pragma unroll
                for (int m = 0; m < MT; ++m)
                    acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][m], __builtin_bit_cast(bf16x8_t, piece[pc]), acc[m], 0, 0, 0);
        }
    }
};

template <int MT> struct Frags<MT, float> {
    floatx4_t w[4];            // this lane's four k values of group q: 8 q + 4 lh + {0..3} = chunk 2 q + lh
    floatx4_t a[4][MT];
    __device__ __forceinline__ void read(const u32x4_t *xs, const u32x4_t *wst, int row0, int li, int lh)
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            w[q] = *reinterpret_cast<const floatx4_t *>(&wst[slot_f32(li, 2 * q + lh)]);
#pragma unroll
            for (int m = 0; m < MT; ++m) a[q][m] = *reinterpret_cast<const floatx4_t *>(&xs[slot_f32(row0 + m * 32 + li, 2 * q + lh)]);
        }
    }
    __device__ __forceinline__ void mfma(floatx16_t (&acc)[MT]) const
    {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int m = 0; m < MT; ++m) acc[m] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q][m][s], w[q][s], acc[m], 0, 0, 0);
    }
};

// reductions over the eight lanes of a token (quad permutes, then the mirror of the half row)
#if defined(__HIP_DEVICE_COMPILE__)
#define RT_DPP(v, ctrl) __builtin_amdgcn_mov_dpp((v), ctrl, 0xF, 0xF, true)
#else
#define RT_DPP(v, ctrl) (v)
#endif
#define RT_DPP_F(v, ctrl) __int_as_float(RT_DPP(__float_as_int(v), ctrl))
__device__ __forceinline__ float max8(float v)
{
    v = fmaxf(v, RT_DPP_F(v, 0xB1));
    v = fmaxf(v, RT_DPP_F(v, 0x4E));
    return fmaxf(v, RT_DPP_F(v, 0x141));
}
__device__ __forceinline__ float sum8(float v)
{
    v += RT_DPP_F(v, 0xB1);
    v += RT_DPP_F(v, 0x4E);
    return v + RT_DPP_F(v, 0x141);
}
__device__ __forceinline__ int min8(int v)
{
    int o = RT_DPP(v, 0xB1);
    v = o < v ? o : v;
    o = RT_DPP(v, 0x4E);
    v = o < v ? o : v;
    o = RT_DPP(v, 0x141);
    return o < v ? o : v;
}

// Top-k, softmax weights, margin and probabilities of one token whose logit row lies in LDS; the eight
// lanes sub = 0..7 of a token call this together.
template <int NE>
__device__ __forceinline__ void route_topk(const float *row, int sub, int64_t t, bool live, int N, int K, int renorm,
                                           int32_t *__restrict__ out_idx, float *__restrict__ out_w,
                                           float *__restrict__ out_margin, float *__restrict__ out_probs)
{
    constexpr int E = NE * 4;              // experts of one lane
    const float NEG_INF = -__builtin_inff();
    const int e0 = sub * E;
    const float *mine = row + e0 + 4 * (e0 >> 5);
    float val[E];
#pragma unroll
    for (int j = 0; j < E; j += 4) {
        const floatx4_t v4 = *reinterpret_cast<const floatx4_t *>(mine + j);
#pragma unroll
        for (int i = 0; i < 4; ++i) val[j + i] = (e0 + j + i < N) ? v4[i] : NEG_INF;
    }
    float m = val[0];
#pragma unroll
    for (int j = 1; j < E; ++j) m = fmaxf(m, val[j]);
    const float zmax = max8(m);
    // softmax denominator over all N experts, maximum subtracted
    float part = 0.f;
#pragma unroll
    for (int j = 0; j < E; ++j) part += __expf(val[j] - zmax);
    const float den = sum8(part);

    // an expert that is out, taken or never there, is a NaN: a maximum passes it over and nothing equals it, not even
    // where the logits that are left are -inf
    const float OUT = __builtin_nanf("");
#pragma unroll
    for (int j = 0; j < E; ++j) val[j] = e0 + j < N ? val[j] : OUT;
    float my_v = NEG_INF, zk = zmax, zk1 = NEG_INF;
    int my_e = 0;
    const int rounds = (out_margin && K < N) ? K + 1 : K;
    float top = zmax;
    for (int r = 0; r < rounds; ++r) {
        int id = 0x7FFFFFFF;
#pragma unroll
        for (int j = E - 1; j >= 0; --j) id = (val[j] == top) ? e0 + j : id;    // the lowest id that holds the maximum
        id = min8(id);
        if (r == sub) { my_v = top; my_e = id; }
        if (r == K - 1) zk = top;
        if (r == K) zk1 = top;
        const int gone = id - e0;
        m = NEG_INF;
#pragma unroll
        for (int j = 0; j < E; ++j) {
            val[j] = (j == gone) ? OUT : val[j];
            m = fmaxf(m, val[j]);
        }
        top = max8(m);
    }
    const float p = sub < K ? __expf(my_v - zmax) : 0.f;
    const float sel = sum8(p);
    if (!live) return;
    if (sub < K) {
        out_idx[t * K + sub] = my_e < N ? my_e : N - 1;      // (a row of NaNs names no expert; ids stay in range)
        out_w[t * K + sub] = p * (1.0f / (renorm ? sel : den));
    }
    if (out_margin && sub == 0) out_margin[t] = (K < N) ? zk - zk1 : __builtin_inff();
    if (out_probs) {
        const float rden = 1.0f / den;
        float *o = out_probs + t * N + e0;
        const bool wide = (N & 3) == 0 && (reinterpret_cast<uintptr_t>(out_probs) & 15) == 0;
#pragma unroll
        for (int j = 0; j < E; j += 4) {
            const floatx4_t v4 = *reinterpret_cast<const floatx4_t *>(mine + j);
            floatx4_t p4;
#pragma unroll
            for (int i = 0; i < 4; ++i) p4[i] = __expf(v4[i] - zmax) * rden;
            if (wide) {
                if (e0 + j < N) *reinterpret_cast<floatx4_t *>(o + j) = p4;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (e0 + j + i < N) o[j + i] = p4[i];
            }
        }
    }
}

// fp32 hidden states: a logit is the sum of shares of per_part slices each (an even number), added in order, which
// keeps the sums' rounding small at large H.  PART: workgroup (b, s) takes share s only and stores its sums, a row of
// NE * 32 per token, to partial[s]; route_rank_kernel adds the shares and ranks them.
template <int NE, int MT, bool PART, typename XT>
__global__ __launch_bounds__(RT_BLOCK, 2) void route_kernel(const XT *__restrict__ x, int64_t T, int H,
                                                            const float *__restrict__ wr, int N, int K, int renorm,
                                                            int32_t *__restrict__ out_idx, float *__restrict__ out_w,
                                                            float *__restrict__ out_margin, float *__restrict__ out_probs,
                                                            float *__restrict__ partial, int per_part)
{
    typedef LogitLayout<NE> LL;
    constexpr bool BF16 = sizeof(XT) == 2;
    constexpr int TOKENS = 32 * MT * (4 / NE);
    constexpr int W_U4 = NE * 32 * 8;                               // 16-byte units of the weight stage
    constexpr int X_U4 = TOKENS * (BF16 ? 4 : 8);                   // ... of the token stage
    constexpr int STAGE = W_U4 + X_U4;
    constexpr int STAGES = STAGE * 16 > 20480 ? 3 : 4;
    constexpr int LOGIT_U4 = TOKENS * LL::STRIDE / 4;
    constexpr int W_COPIES = NE;                                    // copy instructions (1 KB each) per wavefront and slice
    constexpr int X_TOTAL = X_U4 / 64, X_COPIES = X_TOTAL >= 4 ? X_TOTAL / 4 : 1;
    constexpr int COPIES = W_COPIES + X_COPIES;
    __shared__ u32x4_t smem[STAGES * STAGE > LOGIT_U4 ? STAGES * STAGE : LOGIT_U4];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 31;              // row / column inside a 32x32 MFMA tile
    const int lh = lane >> 5;
    const int et = wave % NE;              // expert tile
    const int row0 = (wave / NE) * MT * 32;
    const int64_t t0 = (int64_t)blockIdx.x * TOKENS;

    // What this lane fetches for its landing places: copy i of a wavefront fills the 64 chunks behind
    // group * 64.  Expert rows past N and tokens past T repeat the last one (masked or not stored later).
    uint32_t w_off[W_COPIES], x_off[X_COPIES];
#pragma unroll
    for (int i = 0; i < W_COPIES; ++i) {
        const int rs = (wave * W_COPIES + i) * 8 + (lane >> 3), r = rs ^ ((rs >> 3) & 1), c = (lane & 7) ^ (r & 7);
        w_off[i] = (uint32_t)(((r < N ? r : N - 1) * H + c * 4) * 4);
    }
    const int64_t left = T - t0;
#pragma unroll
    for (int i = 0; i < X_COPIES; ++i) {
        const int grp = (X_TOTAL >= 4 ? wave * X_COPIES + i : wave % X_TOTAL);      // fewer than 4 groups: fetched twice
        int r, c;
        if (BF16) {
            r = grp * 16 + (lane >> 2);
            c = (lane & 3) ^ ((r >> 2) & 3);
        } else {
            const int rs = grp * 8 + (lane >> 3);
            r = rs ^ ((rs >> 3) & 1);
            c = (lane & 7) ^ (r & 7);
        }
        x_off[i] = (uint32_t)((r < left ? r : (int)left - 1) * H * (int)sizeof(XT) + c * 16);
    }
    const char *w_base = reinterpret_cast<const char *>(wr), *x_base = reinterpret_cast<const char *>(x + t0 * H);
    const int slices = H / RT_BK, first = PART ? (int)blockIdx.y * per_part : 0;
    const int nk = PART ? (slices - first < per_part ? slices - first : per_part) : slices;
    // slice j of the share -> stage `st` (past the end: the last slice again, so that the count of
    // outstanding copies never varies)
#define RT_COPY(j, st)                                                                                            \
    {                                                                                                             \
        const int j_ = first + ((j) < nk ? (j) : nk - 1);                                                         \
        const char *wb_ = w_base + (int64_t)j_ * RT_BK * 4, *xb_ = x_base + (int64_t)j_ * RT_BK * (int)sizeof(XT); \
        _Pragma("unroll") for (int i = 0; i < W_COPIES; ++i)                                                      \
            copy16_to_lds(wb_, w_off[i], (st) + (wave * W_COPIES + i) * 64);                                      \
        _Pragma("unroll") for (int i = 0; i < X_COPIES; ++i)                                                      \
            copy16_to_lds(xb_, x_off[i], (st) + W_U4 + (X_TOTAL >= 4 ? wave * X_COPIES + i : wave % X_TOTAL) * 64); \
    }

    constexpr bool SUMS = !PART && !BF16;      // several shares in this workgroup
    floatx16_t acc[MT], sum[SUMS ? MT : 1];
#pragma unroll
    for (int n = 0; n < MT; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            acc[n][r] = 0.f;
            if (SUMS) sum[n][r] = 0.f;
        }

#pragma unroll
    for (int j = 0; j < STAGES - 1; ++j) RT_COPY(j, smem + j * STAGE)
    int cur = 0, fill = STAGES - 1;        // stage of slice kt, stage that slice kt + STAGES - 1 goes to
    // Slice kt has landed (this wavefront's part, then everyone's), and everyone has read slice kt - 1, whose
    // stage is refilled; slice kt is read into one register set while the other, slice kt - 1, is multiplied.
#define RT_NEXT(kt, set)                                                                                          \
    {                                                                                                             \
        wait_vmem<(STAGES - 2) * COPIES>();                                                                       \
        lds_barrier();                                                                                            \
        RT_COPY((kt) + STAGES - 1, smem + fill * STAGE)                                                           \
        const u32x4_t *st_ = smem + cur * STAGE;                                                                  \
        set.read(st_ + W_U4, st_ + et * 256, row0, li, lh);                                                       \
        __builtin_amdgcn_sched_barrier(0);                                                                        \
        cur = cur + 1 == STAGES ? 0 : cur + 1;                                                                    \
        fill = fill + 1 == STAGES ? 0 : fill + 1;                                                                 \
    }
    Frags<MT, XT> fa, fb;
    RT_NEXT(0, fa)
    int kt = 1;
    for (int end = SUMS ? per_part : nk;; end += per_part) {       // slices [.., end) are the current share
        const int stop = end < nk - 1 ? end : nk - 1;
        for (; kt < stop; kt += 2) {
            RT_NEXT(kt, fb)
            fa.mfma(acc);
            RT_NEXT(kt + 1, fa)
            fb.mfma(acc);
        }
        if constexpr (SUMS) {
            if (kt > end) {
#pragma unroll
                for (int n = 0; n < MT; ++n)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        sum[n][r] += acc[n][r];
                        acc[n][r] = 0.f;
                    }
            }
        }
        if (!SUMS || kt >= nk - 1) break;
    }
    if (kt < nk) {
        RT_NEXT(kt, fb)
        fa.mfma(acc);
        fb.mfma(acc);
    } else {
        fa.mfma(acc);
    }
#undef RT_NEXT
#undef RT_COPY
    wait_vmem<0>();
    if constexpr (PART) {
        float *out = partial + ((int64_t)blockIdx.y * T + t0) * (NE * 32) + et * 32 + li;
#pragma unroll
        for (int n = 0; n < MT; ++n)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int tl = row0 + n * 32 + (r >> 2) * 8 + lh * 4 + (r & 3);
                if (tl < left) out[tl * (NE * 32)] = acc[n][r];
            }
        return;
    }
    lds_barrier();

    // park the logits (every copy has landed, every stage has been read)
    float *Ls = reinterpret_cast<float *>(smem);
#pragma unroll
    for (int n = 0; n < MT; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            Ls[LL::at(row0 + n * 32 + (r >> 2) * 8 + lh * 4 + (r & 3), et * 32 + li)] = SUMS ? sum[n][r] + acc[n][r] : acc[n][r];
    __syncthreads();
#pragma unroll 1
    for (int g = 0; g < TOKENS; g += RT_BLOCK / RT_LANES) {
        const int tl = g + tid / RT_LANES;
        route_topk<NE>(Ls + tl * LL::STRIDE, tid % RT_LANES, t0 + tl, t0 + tl < T, N, K, renorm, out_idx, out_w, out_margin, out_probs);
    }
}

// ---- few tokens ----------------------------------------------------------------------------------------
// route_kernel leaves most of the chip idle for a few hundred tokens: a workgroup fetches the whole gate matrix through
// its one compute unit, and each of its wavefronts splits the weights of its expert tile in front of the MFMAs that
// need them, 1000 cycles a slice of which the MFMAs are 200.  Here a workgroup owns 32 tokens and one tile of 32
// experts: eight wavefronts split the weights, four rows each, into LDS, one copies the tokens, and one does nothing
// but read operands and multiply, in steps of 64 k-values, two to a barrier.  It issues the MFMAs that route_kernel
// issues for this token and expert tile, in the same order on the same operands, so the logits are the same bits from
// either kernel: moe_forward routes as moe_route does, and a token the same way in a batch of any size.
// (Cutting the reduction itself into shares is 3 us faster and changes the sums.)  The logits go to memory;
// route_rank_kernel ranks them.
// What bounds it: the chain of 3 H / 16 dependent MFMAs, 36 cycles each (5.7 us at H = 2048).  Wavefronts w, w + 4 and w + 8
// share a SIMD: the multiplying one has its SIMD to itself but for the copies (beside two splitters it took 2 us
// more), and 8 and 11 end at once.  16 tokens, 128 experts, H = 2048, caches flushed: 27 us for route_kernel, 11 here
// and 5 for the ranking.
constexpr int RF_BK = 64;
constexpr int RF_THREADS = 12 * 64;
constexpr int RF_AHEAD = 8;            // steps of weights on their way (64 KB), stages of the tokens
constexpr int RF_X = 32 * 8, RF_PIECE = 32 * 8;                      // 16-byte units of a step's tokens, of one piece of its weights

// the operands of a step
struct StepFrags {
    u32x4_t x[4], piece[4][3];
    __device__ __forceinline__ void read(const u32x4_t *xs, const u32x4_t *ps, int i, int li, int lh)
    {
        const int ks = i / 3, pc = i % 3;
        if (pc == 0) x[ks] = xs[slot_f32(li, 2 * ks + lh)];        // 128-byte rows, whatever they hold
        piece[ks][pc] = ps[pc * RF_PIECE + slot_f32(li, 2 * ks + lh)];
    }
    __device__ __forceinline__ void mfma(floatx16_t &acc, int i) const
    {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, x[i / 3]), __builtin_bit_cast(bf16x8_t, piece[i / 3][i % 3]), acc,
                                                      0, 0, 0);
    }
};

// logits[t, pitch]: workgroup (b, e) writes columns 32 e .. 32 e + 31 of tokens 32 b ..; H is a multiple of 2 RF_BK
__global__ __launch_bounds__(RF_THREADS) void route_few_kernel(const bf16_t *__restrict__ x, int64_t T, int H, const float *__restrict__ wr, int N,
                                                               float *__restrict__ logits, int pitch)
{
    __shared__ u32x4_t ring[RF_AHEAD][RF_X];
    __shared__ u32x4_t pieces[4][3 * RF_PIECE];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int64_t t0 = (int64_t)blockIdx.x * 32, left = T - t0;
    const int e0 = blockIdx.y * 32, n = H / RF_BK;
    if (wave == 8 || wave == 11) return;       // (a barrier waits for the wavefronts that have not ended)
    if (wave == 4) {
        // tokens past the end repeat the last one (not stored)
        uint32_t x_off[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int rs = i * 8 + (lane >> 3), r = rs ^ ((rs >> 3) & 1), c = (lane & 7) ^ (r & 7);
            x_off[i] = (uint32_t)((r < left ? r : (int)left - 1) * H * 2 + c * 16);
        }
        const char *x_base = reinterpret_cast<const char *>(x + t0 * H);
        // steps j and j + 1 -> their stages (past the end the last step again, to a stage that is not read any more)
        auto copy = [&](int j) __attribute__((always_inline)) {
#pragma unroll
            for (int d = 0; d < 2; ++d)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    copy16_to_lds(x_base + (int64_t)(j + d < n ? j + d : n - 1) * RF_BK * 2, x_off[i], ring[(j + d) & (RF_AHEAD - 1)] + i * 64);
        };
#pragma unroll
        for (int j = 0; j < RF_AHEAD - 4; j += 2) copy(j);
        for (int j = 0; j < n; j += 2) {
            copy(j + RF_AHEAD - 4);            // stages of steps j - 4 and j - 3, which have been read
            wait_vmem<(RF_AHEAD - 4) * 4>();
            lds_barrier();                     // the tokens of steps j and j + 1 are there
        }
        wait_vmem<0>();
        return;
    }
    if (wave != 0) {
        // this lane splits four weights of row r a step: half a chunk.  Rows past the end repeat the last expert (masked in
        // the ranking).  (Through LDS instead of straight into registers the weights took a third of its bandwidth.)
        const int r = (wave < 4 ? wave - 1 : wave < 8 ? wave - 2 : wave - 3) * 4 + (lane >> 4), place = slot_f32(r, (lane & 15) >> 1) * 2 + (lane & 1);
        const floatx4_t *src = reinterpret_cast<const floatx4_t *>(wr + (int64_t)(e0 + r < N ? e0 + r : N - 1) * H) + (lane & 15);
        floatx4_t w[RF_AHEAD];
        auto split = [&](int u) __attribute__((always_inline)) {
            uint32_t p0[3], p1[3];
            split3_pair(w[u][0], w[u][1], p0[0], p0[1], p0[2]);
            split3_pair(w[u][2], w[u][3], p1[0], p1[1], p1[2]);
#pragma unroll
            for (int pc = 0; pc < 3; ++pc)
                reinterpret_cast<uint2 *>(&pieces[u & 3][pc * RF_PIECE])[place] = make_uint2(p0[pc], p1[pc]);
        };
#pragma unroll
        for (int u = 0; u < RF_AHEAD; ++u) w[u] = src[(u < n ? u : n - 1) * (RF_BK / 4)];
        int j = 0;
        for (; j + RF_AHEAD <= n; j += RF_AHEAD) {
#pragma unroll
            for (int u = 0; u < RF_AHEAD; ++u) {
                split(u);
                const int next = j + u + RF_AHEAD;
                w[u] = src[(next < n ? next : n - 1) * (RF_BK / 4)];
                if (u & 1) {
                    lds_barrier();                     // steps j + u - 1 and j + u are ready, the two before them have been read
                    __builtin_amdgcn_sched_barrier(0); // (later steps' splits in front of it would wait for their loads)
                }
            }
        }
#pragma unroll
        for (int u = 0; u < RF_AHEAD - 1; ++u) {
            if (j + u < n) {
                split(u);
                if (u & 1) lds_barrier();
            }
        }
        return;
    }
    __builtin_amdgcn_s_setprio(3);
    const int li = lane & 31, lh = lane >> 5;
    floatx16_t acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    StepFrags fa, fb;
    // step j is read while the step before it is multiplied: the reads behind the first MFMAs (in front of them they
    // would keep them waiting), so that they have landed when the last one is issued
    auto step = [&](int j, bool barrier, const StepFrags &prev, StepFrags &next) __attribute__((always_inline)) {
        if (barrier) lds_barrier();            // this step and the next are there
        const u32x4_t *xs = ring[j & (RF_AHEAD - 1)], *ps = pieces[j & 3];
#pragma unroll
        for (int i = 0; i < 12; ++i) {
            if (j > 0) prev.mfma(acc, i);
            if (i < 6) {
                next.read(xs, ps, 2 * i, li, lh);
                next.read(xs, ps, 2 * i + 1, li, lh);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    step(0, true, fb, fa);
    for (int j = 1; j + 1 < n; j += 2) {                           // n is even
        step(j, false, fa, fb);
        step(j + 1, true, fb, fa);
    }
    step(n - 1, false, fa, fb);
#pragma unroll
    for (int i = 0; i < 12; ++i) fb.mfma(acc, i);
    float *out = logits + t0 * pitch + e0 + li;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int tl = (r >> 2) * 8 + lh * 4 + (r & 3);
        if (tl < left) out[tl * pitch] = acc[r];
    }
}

// ---- 33 to 64 experts, one block of tokens per compute unit ----------------------------------------------------
// route_kernel's four wavefronts split the weights for their own MFMAs, 1000 cycles a slice with nothing else on their SIMD.  Here
// eight wavefronts split the weights of both expert tiles into LDS, once for the block, in steps of 64 k-values, and copy the
// tokens; four, one per SIMD, only read operands and multiply, a tile of 32 tokens x 32 experts each.  The MFMAs
// of a tile are route_kernel's, in its order on its operands: the logits are the same bits.
// The copies of a splitter's step go out in front of its weight loads, and the wait in front of the barrier counts both.
// What bounds it: about 600 cycles a step, MFMAs (384), split, LDS writes and operand reads each close to that (any one of them left
// out gives 1-2 us, no more), and 7 us that a call of one step takes.
// H = 2048, 64 experts, moe_route, route_kernel / this (us): 16 tokens 26.4 / 16.0, 2048 tokens 26.7 / 17.2, 16384 tokens 30.3 / 22.8,
// caches flushed 28.0 / 20.0, 27.8 / 23.0, 40.4 / 37.4; 32768 tokens, two blocks each, 38 / 45.  128 experts: 8192 tokens 31.3 / 30.1, flushed
// 38.0 / 39.4 (a step's pieces are 48 KB there, two steps in all fit the LDS): left to route_kernel.
constexpr int RB_THREADS = 12 * 64, RB_SPLIT = 8;

__global__ __launch_bounds__(RB_THREADS) void route_block_kernel(const bf16_t *__restrict__ x, int64_t T, int H, const float *__restrict__ wr, int N,
                                                                 int K, int renorm, int32_t *__restrict__ out_idx, float *__restrict__ out_w,
                                                                 float *__restrict__ out_margin, float *__restrict__ out_probs)
{
    constexpr int NE = 2, TT = 4 / NE, TOKENS = 32 * TT;             // expert tiles, token tiles
    typedef LogitLayout<NE> LL;
    // Weights and tokens are requested DEPTH steps ahead.  In front of a step's split the compiler waits until no more loads are outstanding
    // than the weights it has asked for since, 10, and does not count the copies among them: three steps and a load stay on their way.
    constexpr int DEPTH = 6, STAGES = DEPTH + 2;                     // ...; stages of the tokens
    constexpr int COPIES = TT * 4 / RB_SPLIT;                        // copy instructions (1 KB each) per wavefront and step
    constexpr int X_U4 = TT * RF_X, P_U4 = NE * 3 * RF_PIECE;
    __shared__ u32x4_t smem[STAGES * X_U4 + 2 * P_U4];
    static_assert(sizeof(smem) >= sizeof(float) * TOKENS * LL::STRIDE, "the logits are parked in the stages");
    u32x4_t *const ring = smem, *const pieces = smem + STAGES * X_U4;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int64_t t0 = (int64_t)blockIdx.x * TOKENS, left = T - t0;
    const int n = H / RF_BK;
    float *Ls = reinterpret_cast<float *>(smem);
    if (wave >= 4) {
        const int s = wave - 4;
        uint32_t x_off[COPIES];
#pragma unroll
        for (int i = 0; i < COPIES; ++i) {
            const int q = s * COPIES + i, rs = (q & 3) * 8 + (lane >> 3), rt = rs ^ ((rs >> 3) & 1), c = (lane & 7) ^ (rt & 7), r = (q >> 2) * 32 + rt;
            x_off[i] = (uint32_t)((r < left ? r : (int)left - 1) * H * 2 + c * 16);      // tokens past the end repeat the last one
        }
        const char *x_base = reinterpret_cast<const char *>(x + t0 * H);
        // this lane splits four weights of NE rows a step (rows past the end repeat the last expert, masked in the ranking)
        const floatx4_t *src[NE];
        int place[NE];
#pragma unroll
        for (int f = 0; f < NE; ++f) {
            const int r = (s * NE + f) * 4 + (lane >> 4);
            src[f] = reinterpret_cast<const floatx4_t *>(wr + (int64_t)(r < N ? r : N - 1) * H) + (lane & 15);
            place[f] = ((r >> 5) * 3 * RF_PIECE + slot_f32(r & 31, (lane & 15) >> 1)) * 2 + (lane & 1);
        }
        floatx4_t w[DEPTH][NE];
        int fill = 0;
        // the tokens of step j -> the next stage, its weights -> w[u] (past the end the last step again)
        auto request = [&](int j, int u) __attribute__((always_inline)) {
            const int j_ = j < n ? j : n - 1;
#pragma unroll
            for (int i = 0; i < COPIES; ++i) copy16_to_lds(x_base + (int64_t)j_ * RF_BK * 2, x_off[i], ring + fill * X_U4 + (s * COPIES + i) * 64);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int f = 0; f < NE; ++f) w[u][f] = src[f][j_ * (RF_BK / 4)];
            fill = fill + 1 == STAGES ? 0 : fill + 1;
            __builtin_amdgcn_sched_barrier(0);
        };
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) request(u, u);
        auto step = [&](int j, int u) __attribute__((always_inline)) {
            uint2 *out = reinterpret_cast<uint2 *>(pieces + (j & 1) * P_U4);
#pragma unroll
            for (int f = 0; f < NE; ++f) {
                uint32_t p0[3], p1[3];
                split3_pair(w[u][f][0], w[u][f][1], p0[0], p0[1], p0[2]);
                split3_pair(w[u][f][2], w[u][f][3], p1[0], p1[1], p1[2]);
#pragma unroll
                for (int pc = 0; pc < 3; ++pc) out[pc * RF_PIECE * 2 + place[f]] = make_uint2(p0[pc], p1[pc]);
            }
            __builtin_amdgcn_sched_barrier(0);
            request(j + DEPTH, u);                   // tokens: into the stage of step j - 2
            wait_vmem<DEPTH * (NE + COPIES)>();      // (the step's copies are older than that)
            lds_barrier();                           // tokens and pieces of this step are there, those of the step before last have been read
            __builtin_amdgcn_sched_barrier(0);
        };
        int j = 0;
        for (; j + DEPTH <= n; j += DEPTH) {         // (a condition around every step and the compiler waits for all loads in flight)
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) step(j + u, u);
        }
#pragma unroll
        for (int u = 0; u < DEPTH - 1; ++u)
            if (j + u < n) step(j + u, u);
        wait_vmem<0>();
        lds_barrier();                             // everything has landed and has been read
    } else {
        __builtin_amdgcn_s_setprio(3);
        const int li = lane & 31, lh = lane >> 5, et = wave % NE, tt = wave / NE;
        floatx16_t acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        StepFrags fa, fb;
        int cur = 0;
        auto step = [&](int j, const StepFrags &prev, StepFrags &next) __attribute__((always_inline)) {
            lds_barrier();
            const u32x4_t *xs = ring + cur * X_U4 + tt * RF_X, *ps = pieces + (j & 1) * P_U4 + et * 3 * RF_PIECE;
            cur = cur + 1 == STAGES ? 0 : cur + 1;
#pragma unroll
            for (int i = 0; i < 12; ++i) {
                if (j > 0) prev.mfma(acc, i);
                if (i < 6) {
                    next.read(xs, ps, 2 * i, li, lh);
                    next.read(xs, ps, 2 * i + 1, li, lh);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        step(0, fb, fa);
        int j = 1;
        for (; j + 1 < n; j += 2) {
            step(j, fa, fb);
            step(j + 1, fb, fa);
        }
        if (j < n) {
            step(j, fa, fb);
#pragma unroll
            for (int i = 0; i < 12; ++i) fb.mfma(acc, i);
        } else {
#pragma unroll
            for (int i = 0; i < 12; ++i) fa.mfma(acc, i);
        }
        __builtin_amdgcn_s_setprio(0);
        lds_barrier();
#pragma unroll
        for (int r = 0; r < 16; ++r) Ls[LL::at(tt * 32 + (r >> 2) * 8 + lh * 4 + (r & 3), et * 32 + li)] = acc[r];
    }
    __syncthreads();
#pragma unroll 1
    for (int tl = threadIdx.x / RT_LANES; tl < TOKENS; tl += RB_THREADS / RT_LANES)
        route_topk<NE>(Ls + tl * LL::STRIDE, threadIdx.x % RT_LANES, t0 + tl, tl < left, N, K, renorm, out_idx, out_w, out_margin, out_probs);
}

// 32 tokens per workgroup, a row of NE * 32 logits each (columns past N hold anything), or `parts` shares of them, added
// in order
template <int NE>
__global__ __launch_bounds__(RT_BLOCK) void route_rank_kernel(const float *__restrict__ logits, int parts, int64_t T, int N, int K, int renorm,
                                                              int32_t *__restrict__ out_idx, float *__restrict__ out_w,
                                                              float *__restrict__ out_margin, float *__restrict__ out_probs)
{
    typedef LogitLayout<NE> LL;
    constexpr int TOKENS = RT_BLOCK / RT_LANES, ROW4 = NE * 8;        // 16-byte pieces of a row
    __shared__ floatx4_t smem[TOKENS * LL::STRIDE / 4];
    float *Ls = reinterpret_cast<float *>(smem);
    const int64_t t0 = (int64_t)blockIdx.x * TOKENS, left = T - t0;
#pragma unroll
    for (int q = (int)threadIdx.x; q < TOKENS * ROW4; q += RT_BLOCK) {
        const int tl = q / ROW4, c = q % ROW4;
        const int64_t t = t0 + (tl < left ? tl : left - 1);
        const floatx4_t *p = reinterpret_cast<const floatx4_t *>(logits) + t * ROW4 + c;
        floatx4_t sum = p[0];
        if (parts > 1) {
            floatx4_t v[RT_PARTS];
#pragma unroll
            for (int s = 1; s < RT_PARTS; ++s) v[s] = p[(s < parts ? s : 0) * T * ROW4];
#pragma unroll
            for (int s = 1; s < RT_PARTS; ++s)
                if (s < parts) sum += v[s];
        }
        *reinterpret_cast<floatx4_t *>(&Ls[LL::at(tl, 4 * c)]) = sum;
    }
    __syncthreads();
    const int tl = threadIdx.x / RT_LANES;
    route_topk<NE>(Ls + tl * LL::STRIDE, threadIdx.x % RT_LANES, t0 + tl, tl < left, N, K, renorm, out_idx, out_w, out_margin, out_probs);
}

// Tokens per workgroup.  A workgroup's time is one serial chain over the reduction whatever its width, and one
// wavefront per SIMD issues a vector instruction every 8 cycles at best, so as long as the blocks do not fill
// the chip the narrowest block is the fastest; beyond that a wider block splits the weights for more
// tokens at a time.  Hence the fewest token tiles that still give one workgroup per compute unit, up to what the
// LDS holds twice.  H = 2048, bf16, 1 / 2 / 4 token tiles: 128 experts, 4096 tokens 27 / 31 / 46 us, 16384 tokens
// 45 / 35 / 47, 65536 tokens 169 / 119 / 101; 64 experts, 16384 tokens 26 / 30 / 47, 65536 tokens 80 / 63 / 62.
// Few tokens (bf16, given scratch memory for the logits: launch_route's `logits`): one workgroup of route_few_kernel per
// compute unit (its registers hold no second one; 256, the constant, so that the size of the scratch is a function of its
// arguments alone).  Layer with the router as its largest part, caches flushed before each call, route_kernel / this
// (us): H = 2048, 128 experts, 16 tokens 75 / 62, 1021 tokens 114 / 105, 2048 tokens 144 / 142.  Below H = 1024 the second
// launch costs what the first one saves.
constexpr int RF_BLOCKS = 256;
int logit_pitch(int N) { return N <= 32 ? 32 : N <= 64 ? 64 : 128; }
int expert_tiles(int N) { return (int)ceil_div(N, 32); }
bool few_tokens(int64_t T, int H, int N) { return H >= 1024 && H % (2 * RF_BK) == 0 && ceil_div(T, 32) * expert_tiles(N) <= RF_BLOCKS; }

// fp32: where the reduction is cut depends on H alone, so the logits are the same bits for any batch and entry point.
// With scratch memory every share is a workgroup's of its own, up to two for each of the two that a compute unit
// holds; otherwise a workgroup takes the shares one after the other.  H = 2048, 128 experts, one after the other / each its
// own (us): 3000 tokens 356 / 338, 4096 tokens 503 / 494.
constexpr int RT_PART_BLOCKS = 1024;
int part_slices(int H)
{
    const int slices = H / RT_BK, most = H < 1024 ? 1 : slices / 8;
    return (int)ceil_div(slices, 2 * (most < RT_PARTS ? most : RT_PARTS)) * 2;
}
int part_count(int H) { return (int)ceil_div(H / RT_BK, part_slices(H)); }
bool one_share_each(int64_t T, int H, int N)
{
    return part_count(H) > 1 && ceil_div(T, 4096 / logit_pitch(N)) * part_count(H) <= RT_PART_BLOCKS;
}

template <int NE, typename XT>
remoe_status launch_tiles(const XT *x, int64_t T, int H, const float *wr, int N, int K, int renorm, int32_t *out_idx,
                          float *out_w, float *out_margin, float *out_probs, float *logits, hipStream_t stream)
{
    constexpr int UNIT = 32 * (4 / NE);    // tokens of a workgroup per token tile of a wavefront
    const dim3 block(RT_BLOCK);
#define RT_LAUNCH(MT)                                                                                              \
    hipLaunchKernelGGL((route_kernel<NE, MT, false, XT>), dim3((unsigned)ceil_div(T, UNIT * MT)), block, 0, stream, x, T, H, wr, N, K, \
                       renorm, out_idx, out_w, out_margin, out_probs, nullptr, per_part)
    constexpr bool BF16 = sizeof(XT) == 2;
    constexpr int MAX_MT = NE == 1 ? (BF16 ? 2 : 1) : (BF16 ? 4 : 2);
    const int parts = BF16 ? 1 : part_count(H), per_part = part_slices(H);
    bool ranked_apart = false;
    if constexpr (BF16) {
        if (logits && few_tokens(T, H, N)) {
            hipLaunchKernelGGL(route_few_kernel, dim3((unsigned)ceil_div(T, 32), (unsigned)expert_tiles(N)), dim3(RF_THREADS), 0, stream, x, T, H, wr, N,
                               logits, logit_pitch(N));
            ranked_apart = true;
        }
    } else if (logits && one_share_each(T, H, N)) {
        hipLaunchKernelGGL((route_kernel<NE, 1, true, XT>), dim3((unsigned)ceil_div(T, UNIT), (unsigned)parts), block, 0, stream, x, T, H, wr, N, K,
                           renorm, nullptr, nullptr, nullptr, nullptr, logits, per_part);
        ranked_apart = true;
    }
    if (ranked_apart) {
        hipLaunchKernelGGL(route_rank_kernel<NE>, dim3((unsigned)ceil_div(T, RT_BLOCK / RT_LANES)), block, 0, stream, logits, parts, T, N, K, renorm,
                           out_idx, out_w, out_margin, out_probs);
        return check_hip(hipGetLastError(), "route_rank_kernel launch");
    }
    int cus = 0;
    const remoe_status st = compute_units(&cus);
    if (st != REMOE_OK) return st;
    if constexpr (BF16 && NE == 2) {
        if (ceil_div(T, UNIT) <= cus && H % RF_BK == 0) {
            hipLaunchKernelGGL(route_block_kernel, dim3((unsigned)ceil_div(T, UNIT)), dim3(RB_THREADS), 0, stream, x, T, H, wr, N, K, renorm, out_idx,
                               out_w, out_margin, out_probs);
            return check_hip(hipGetLastError(), "route_block_kernel launch");
        }
    }
    const int64_t mt = ceil_div(T, (int64_t)UNIT * cus);
    if (mt > 2 && MAX_MT >= 4) RT_LAUNCH((MAX_MT >= 4 ? 4 : 1));
    else if (mt > 1 && MAX_MT >= 2) RT_LAUNCH((MAX_MT >= 2 ? 2 : 1));
    else RT_LAUNCH(1);
#undef RT_LAUNCH
    return check_hip(hipGetLastError(), "route_kernel launch");
}

template <typename XT>
remoe_status launch_typed(const XT *x, int64_t T, int H, const float *wr, int N, int K, int renorm,
                          int32_t *out_idx, float *out_w, float *out_margin, float *out_probs,
                          float *logits, hipStream_t stream)
{
    if (N <= 32) return launch_tiles<1, XT>(x, T, H, wr, N, K, renorm, out_idx, out_w, out_margin, out_probs, logits, stream);
    if (N <= 64) return launch_tiles<2, XT>(x, T, H, wr, N, K, renorm, out_idx, out_w, out_margin, out_probs, logits, stream);
    return launch_tiles<4, XT>(x, T, H, wr, N, K, renorm, out_idx, out_w, out_margin, out_probs, logits, stream);
}

}  // namespace

// What any batch of up to T tokens takes (so that more tokens never need less): 1 MB at most, 16 MB for fp32.
size_t route_scratch_bytes(int x_dtype, int64_t T, int H, int N)
{
    int64_t rows = 0, most = 0;
    if (x_dtype == REMOE_BF16 && few_tokens(1, H, N)) {
        rows = T;
        most = RF_BLOCKS / expert_tiles(N) * 32;
    }
    if (x_dtype == REMOE_F32 && one_share_each(1, H, N)) {
        rows = part_count(H) * T;
        most = (int64_t)RT_PART_BLOCKS * (4096 / logit_pitch(N));
    }
    return sizeof(float) * (size_t)(rows < most ? rows : most) * logit_pitch(N);
}

remoe_status launch_route(const void *x, int x_dtype, int64_t T, int H, const float *w_router,
                          int N, int K, int renorm, int32_t *out_idx, float *out_w,
                          float *out_margin, float *out_probs, float *logits, hipStream_t stream)
{
    if (T == 0) return REMOE_OK;
    if (x_dtype == REMOE_F32)
        return launch_typed<float>(static_cast<const float *>(x), T, H, w_router, N, K, renorm,
                                   out_idx, out_w, out_margin, out_probs, logits, stream);
    return launch_typed<bf16_t>(static_cast<const bf16_t *>(x), T, H, w_router, N, K, renorm,
                                out_idx, out_w, out_margin, out_probs, logits, stream);
}

}  // namespace remoe
