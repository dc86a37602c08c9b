// Router kernel: fp32-accurate logits on the matrix cores, then the top-k and softmax in the same workgroup.
//
// Computes the paper's routing step (Sec. 3.1): P_t = Softmax(h_t^T theta_gate), E_t = Top-K(P_t).
// One workgroup of 4 wavefronts owns a block of tokens and all N_r <= 128 experts.  The experts are cut
// into NE tiles of 32 (NE = 1, 2 or 4); wavefront w computes expert tile w % NE for MT tiles of 32
// tokens, the 4 / NE wavefronts of one expert tile taking different tokens, so a workgroup owns
// 32 * MT * 4 / NE tokens and every token's full logit row ends in one workgroup.
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
constexpr int RT_PARTS = 8;            // shares of the reduction at most

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
            val[j] = (j == gone) ? NEG_INF : val[j];
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

// PART: workgroup (b, s) takes share s of the reduction only (`per_part` slices) and stores its products, a row of
// NE * 32 sums per token, to partial[s]; route_parts_kernel adds the shares up and ranks them.
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

    floatx16_t acc[MT];
#pragma unroll
    for (int n = 0; n < MT; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[n][r] = 0.f;

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
    for (; kt + 1 < nk; kt += 2) {
        RT_NEXT(kt, fb)
        fa.mfma(acc);
        RT_NEXT(kt + 1, fa)
        fb.mfma(acc);
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
            Ls[LL::at(row0 + n * 32 + (r >> 2) * 8 + lh * 4 + (r & 3), et * 32 + li)] = acc[n][r];
    __syncthreads();
#pragma unroll 1
    for (int g = 0; g < TOKENS; g += RT_BLOCK / RT_LANES) {
        const int tl = g + tid / RT_LANES;
        route_topk<NE>(Ls + tl * LL::STRIDE, tid % RT_LANES, t0 + tl, t0 + tl < T, N, K, renorm, out_idx, out_w, out_margin, out_probs);
    }
}

// 32 tokens per workgroup: their logits are the sums of the shares, taken in order
template <int NE>
__global__ __launch_bounds__(RT_BLOCK) void route_parts_kernel(const float *__restrict__ partial, int parts, int64_t T, int N, int K, int renorm,
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
        const floatx4_t *p = reinterpret_cast<const floatx4_t *>(partial) + t * ROW4 + c;
        floatx4_t v[RT_PARTS], sum;
#pragma unroll
        for (int s = 0; s < RT_PARTS; ++s) v[s] = p[(s < parts ? s : 0) * T * ROW4];
        sum = v[0];
#pragma unroll
        for (int s = 1; s < RT_PARTS; ++s)
            if (s < parts) sum += v[s];
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
// Shares of the reduction: with few tokens a handful of workgroups fetch the whole gate matrix, each through one
// compute unit, one slice after the other.  Given scratch memory for the shares (launch_route's `partial`), up to
// RT_PARTS workgroups take at least 8 slices each, while the blocks leave room for them on the chip (256 compute units; the
// constant, so that the size of the scratch is a function of its arguments alone).  Layer with the router as its
// largest part, caches flushed before each call, 1 / 2 / 4 / 8 shares (us): H = 2048, 128 experts, 16 tokens 75 / 67 / 62 /
// 59, 1021 tokens 114 / 107 / 102 / 100, 2048 tokens 144 / 139 / 134 / 135, 4096 tokens 187 / 182 / 183 / 188; 64 experts,
// 4096 tokens 157 / 150 / 146 / 148; H = 1024, 32 experts, 1021 tokens 52 / 48 / 45 / 44; H = 512, 128 experts, 1021
// tokens 40 / 43 / 41 / 41: below H = 1024 the second launch costs what the shares save.
constexpr int RT_PART_BLOCKS = 256;
int most_parts(int H)
{
    const int parts = H < 1024 ? 1 : H / (8 * RT_BK);
    return parts < RT_PARTS ? parts : RT_PARTS;
}
int expert_tiles(int N) { return N <= 32 ? 1 : N <= 64 ? 2 : 4; }
int block_tokens(int N) { return 32 * (4 / expert_tiles(N)); }      // of a workgroup with one token tile per wavefront

int route_parts(int64_t T, int H, int N)
{
    const int64_t room = RT_PART_BLOCKS / ceil_div(T, block_tokens(N));
    const int parts = most_parts(H);
    return parts <= room ? parts : room > 1 ? (int)room : 1;
}

template <int NE, typename XT>
remoe_status launch_tiles(const XT *x, int64_t T, int H, const float *wr, int N, int K, int renorm, int32_t *out_idx,
                          float *out_w, float *out_margin, float *out_probs, float *partial, hipStream_t stream)
{
    constexpr int UNIT = 32 * (4 / NE);    // tokens of a workgroup per token tile of a wavefront
    const dim3 block(RT_BLOCK);
#define RT_LAUNCH(MT)                                                                                              \
    hipLaunchKernelGGL((route_kernel<NE, MT, false, XT>), dim3((unsigned)ceil_div(T, UNIT * MT)), block, 0, stream, x, T, H, wr, N, K, \
                       renorm, out_idx, out_w, out_margin, out_probs, nullptr, 0)
    constexpr bool BF16 = sizeof(XT) == 2;
    constexpr int MAX_MT = NE == 1 ? (BF16 ? 2 : 1) : (BF16 ? 4 : 2);
    const int parts = partial ? route_parts(T, H, N) : 1;
    if (parts > 1) {
        const int per_part = (int)ceil_div(H / RT_BK, parts);
        hipLaunchKernelGGL((route_kernel<NE, 1, true, XT>), dim3((unsigned)ceil_div(T, UNIT), (unsigned)ceil_div(H / RT_BK, per_part)), block, 0,
                           stream, x, T, H, wr, N, K, renorm, nullptr, nullptr, nullptr, nullptr, partial, per_part);
        hipLaunchKernelGGL(route_parts_kernel<NE>, dim3((unsigned)ceil_div(T, RT_BLOCK / RT_LANES)), block, 0, stream, partial,
                           (int)ceil_div(H / RT_BK, per_part), T, N, K, renorm, out_idx, out_w, out_margin, out_probs);
        return check_hip(hipGetLastError(), "route_parts_kernel launch");
    }
    int cus = 0;
    const remoe_status st = compute_units(&cus);
    if (st != REMOE_OK) return st;
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
                          float *partial, hipStream_t stream)
{
    if (N <= 32) return launch_tiles<1, XT>(x, T, H, wr, N, K, renorm, out_idx, out_w, out_margin, out_probs, partial, stream);
    if (N <= 64) return launch_tiles<2, XT>(x, T, H, wr, N, K, renorm, out_idx, out_w, out_margin, out_probs, partial, stream);
    return launch_tiles<4, XT>(x, T, H, wr, N, K, renorm, out_idx, out_w, out_margin, out_probs, partial, stream);
}

}  // namespace

// What any batch of up to T tokens takes (so that more tokens never need less): rows of one share for at most
// RT_PART_BLOCKS blocks of tokens, 4 MB.
size_t route_scratch_bytes(int64_t T, int H, int N)
{
    const int64_t rows = most_parts(H) * T, most = (int64_t)RT_PART_BLOCKS * block_tokens(N);
    return most_parts(H) > 1 ? sizeof(float) * (size_t)(rows < most ? rows : most) * 32 * expert_tiles(N) : 0;
}

remoe_status launch_route(const void *x, int x_dtype, int64_t T, int H, const float *w_router,
                          int N, int K, int renorm, int32_t *out_idx, float *out_w,
                          float *out_margin, float *out_probs, float *partial, hipStream_t stream)
{
    if (T == 0) return REMOE_OK;
    if (x_dtype == REMOE_F32)
        return launch_typed<float>(static_cast<const float *>(x), T, H, w_router, N, K, renorm,
                                   out_idx, out_w, out_margin, out_probs, partial, stream);
    return launch_typed<bf16_t>(static_cast<const bf16_t *>(x), T, H, w_router, N, K, renorm,
                                out_idx, out_w, out_margin, out_probs, partial, stream);
}

}  // namespace remoe
