// Grouped expert GEMMs for few rows per expert (bf16, fp32 accumulate): the weights are streamed.
//
// Same contract as the 256-row kernel (gemm_bf16.hip), for batches whose experts see a few dozen rows each:
//   mode 0:  h   = silu(X_e W_gate[e]^T) * (X_e W_up[e]^T)          -> [slots, I]   bf16
//   mode 1:  out = h_e W_down[e]^T                                  -> [slots, H]   bf16
// There the time is that of reading every active expert's weights once, and a 256-row tile spends its
// matrix cores and its copies on padding.  A workgroup owns a row tile of 32 * MB slots and 128 or 256
// weight rows (mode 0: half gate rows, half the matching up rows).  Slices of 64 k-values of both operands
// move global -> LDS directly, in full 128-byte lines, into a ring of STAGES stages with one barrier per
// slice.  What bounds it is the weight bytes in flight: MB = 1 keeps 3 slices x 16 KB x 2 workgroups per
// compute unit on their way.  Measured on a Qwen3-shaped layer (128 experts, H 2048, I 768), the two
// GEMMs together, 256-row kernel before / this kernel: 16 tokens 218 / 122 us (0.77 GB of weights at
// 6.3 TB/s), 333 tokens 327 / 213 us (1.2 GB at 5.7 TB/s).  Slices of 32 k-values (64-byte rows) with twice
// the stages were 5-10 % slower throughout.
//
// The MFMAs take the weight rows as their first operand, so a lane owns one slot (row of the output) and,
// per group of four accumulators, four adjacent weight rows.  In mode 0 every 32-row group of the weights is
// 16 gate rows followed by the 16 up rows of the same columns, so g and u of one output meet in one lane.
//
// Tiles whose rows fill only NB of the MB 32-row bands copy and multiply only those.
//
// The shared expert (dense, all tokens) runs in the same launch as one more group with its own operands
// and sizes: its matrix work fills the routed experts' waits for memory, and no launch ends half empty in
// between.  Its tiles come first (in mode 1 they are the longer ones) and are dealt evenly to the XCDs.
#include "common.h"
#include "lds_copy.h"

namespace remoe {

namespace {

typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;
constexpr int ST_BK = 64;        // k-values per slice

// LDS rows of 128 bytes are 8 chunks of 16 bytes; chunk c of row r lives in row slot r ^ ((r >> 3) & 1) at
// chunk position c ^ (r & 7): 16 consecutive rows of one logical chunk cover all banks once.
__device__ __forceinline__ int st_slot(int r, int c) { return ((r ^ ((r >> 3) & 1)) << 3) + (c ^ (r & 7)); }
// row and chunk whose landing place is chunk position `u` of the tile (the inverse)
__device__ __forceinline__ void st_place(int u, int &r, int &c)
{
    const int rs = u >> 3;
    r = rs ^ ((rs >> 3) & 1);
    c = (u & 7) ^ (r & 7);
}

struct Group {
    const bf16_t *a;
    int64_t lda;
    const int32_t *gather;       // slot -> row of a, or NULL
    const bf16_t *b0, *b1;
    int k_dim, n_out;
    bf16_t *c;                   // first output row of the group
    int64_t ldc;
};

struct SArgs {
    Group routed, shared;
    const int32_t *tile_expert, *tile_row0, *tile_rows, *n_tiles;
    int shared_rows;             // tokens of the shared group (0: none)
};

__device__ __forceinline__ int st_entry(const int32_t *list, int idx)
{
    typedef const int32_t __attribute__((address_space(4))) *const_i32_ptr;
    return *(const_i32_ptr)(uintptr_t)(list + idx);
}

// WW x WA wavefronts; a wavefront multiplies TW tiles of 32 weight rows with every WA-th of the MB 32-row bands
// of A.  Every wavefront copies 32 weight rows and its share of A.
template <int WW, int WA, int TW, int MB> struct StreamTile {
    static constexpr int WAVES = WW * WA;
    static constexpr int WROWS = 32 * WW * TW;           // weight rows
    static constexpr int W_U4 = WROWS * 8;               // 16-byte units of the weight part of a stage
    static constexpr int STAGE = W_U4 + MB * 256;
    static constexpr int W_COPIES = 4;                   // copy instructions (1 KB each) per wavefront and slice
    static constexpr int TA = MB / WA;                   // bands per wavefront
    static_assert(WROWS == 32 * WAVES && MB % WA == 0, "every wavefront copies one 32-row group of the weights");
    static constexpr int a_copies(int nb) { return (nb * 4 + WAVES - 1) / WAVES; }
};

// The reduction of one tile with NB bands of 32 rows (NT: bands of this wavefront, a band past NB is not stored).
template <int MODE, int WW, int WA, int TW, int MB, int STAGES, bool DEALT, int NB>
__device__ __forceinline__ void stream_loop(u32x4_t *smem, const char *a_base, const uint32_t *a_off, const char *b_base0,
                                            const char *b_base1, const uint32_t *b_off, int nk, int wave, int li, int lh,
                                            floatx16_t (&acc)[MB / WA][TW])
{
    typedef StreamTile<WW, WA, TW, MB> ST;
    constexpr int NT = (NB + WA - 1) / WA;
    constexpr int A_COPIES = ST::a_copies(NB), A_INSTR = NB * 4;
    constexpr int COPIES = ST::W_COPIES + A_COPIES;
    // copy c of slice j -> stage st (past the end the last slice again: the count of outstanding copies never varies)
    auto copy = [&](int j, u32x4_t *st, int c) __attribute__((always_inline)) {
        const int64_t k = (int64_t)(j < nk ? j : nk - 1) * (ST_BK * 2);
        if (c < ST::W_COPIES) {
            copy16_to_lds((MODE == 0 && c >= ST::W_COPIES / 2 ? b_base1 : b_base0) + k, b_off[c], st + (wave * ST::W_COPIES + c) * 64);
        } else {
            int g = (c - ST::W_COPIES) * ST::WAVES + wave;
            if (A_INSTR % ST::WAVES != 0 && g >= A_INSTR) g -= A_INSTR;      // fewer pieces than wavefronts: fetched twice
            copy16_to_lds(a_base + k, a_off[c - ST::W_COPIES], st + ST::W_U4 + g * 64);
        }
    };
#pragma unroll
    for (int j = 0; j < STAGES - 1; ++j)
#pragma unroll
        for (int c = 0; c < COPIES; ++c) copy(j, smem + j * ST::STAGE, c);
    int cur = 0, fill = STAGES - 1;
    const int w_row = (wave / WA) * TW * 32 + li, a_row = (wave % WA) * 32 + li;
    for (int kt = 0; kt < nk; ++kt) {
        wait_vmem<(STAGES - 2) * COPIES>();
        lds_barrier();                          // slice kt is there, everyone is done with slice kt - 1
        const u32x4_t *st = smem + cur * ST::STAGE;
        u32x4_t *nst = smem + fill * ST::STAGE;
        bf16x8_t w8[2][TW], a8[2][NT];
#define ST_READ(ks)                                                                                                   \
    _Pragma("unroll") for (int t = 0; t < TW; ++t)                                                                    \
        w8[(ks) & 1][t] = *reinterpret_cast<const bf16x8_t *>(&st[st_slot(w_row + t * 32, 2 * (ks) + lh)]);           \
    _Pragma("unroll") for (int m = 0; m < NT; ++m)                                                                    \
        a8[(ks) & 1][m] = *reinterpret_cast<const bf16x8_t *>(&st[ST::W_U4 + st_slot(a_row + m * WA * 32, 2 * (ks) + lh)]);
#define ST_MFMA(ks)                                                                                                   \
    _Pragma("unroll") for (int m = 0; m < NT; ++m)                                                                    \
        _Pragma("unroll") for (int t = 0; t < TW; ++t)                                                                \
            acc[m][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w8[(ks) & 1][t], a8[(ks) & 1][m], acc[m][t], 0, 0, 0);
        if (!DEALT) {
            // memory-bound: the refill is requested before anything else happens
#pragma unroll
            for (int c = 0; c < COPIES; ++c) copy(kt + STAGES - 1, nst, c);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                ST_READ(ks)
                ST_MFMA(ks)
            }
        } else {
            // matrix-bound: fragments one k-step ahead of the MFMAs, the refill's copies dealt out over the k-steps
            ST_READ(0)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                if (ks < 3) { ST_READ(ks + 1) }
#pragma unroll
                for (int c = ks * COPIES / 4; c < (ks + 1) * COPIES / 4; ++c) copy(kt + STAGES - 1, nst, c);
                __builtin_amdgcn_sched_barrier(0);
                ST_MFMA(ks)
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#undef ST_READ
#undef ST_MFMA
        cur = cur + 1 == STAGES ? 0 : cur + 1;
        fill = fill + 1 == STAGES ? 0 : fill + 1;
    }
    wait_vmem<0>();
}

template <int MODE, int WW, int WA, int TW, int MB, int STAGES, bool DEALT>
__global__ __launch_bounds__(WW * WA * 64, 2) void stream_gemm_kernel(const SArgs p)
{
    typedef StreamTile<WW, WA, TW, MB> ST;
    constexpr int BN = MODE == 0 ? ST::WROWS / 2 : ST::WROWS;      // output columns of a tile
    constexpr int BM = 32 * MB;
    __shared__ u32x4_t smem[STAGES * ST::STAGE];

    // Workgroup b runs on XCD b % 8; every XCD takes a contiguous range of the shared tiles and then one of
    // the routed tiles (column tile fastest), so the row tiles of one expert meet in one L2.
    const int home = blockIdx.x & 7;
    int i = blockIdx.x >> 3;
    const int ntn_s = (p.shared.n_out + BN - 1) / BN, ntn_r = (p.routed.n_out + BN - 1) / BN;
    const int n_s = (p.shared_rows + BM - 1) / BM * ntn_s;
    const int chunk_s = (n_s + 7) >> 3;
    const bool shared = i < chunk_s;
    int expert = 0, row0, rows, nt;
    if (shared) {
        const int q = home * chunk_s + i;
        if (q >= n_s) return;
        const int mt = q / ntn_s;
        nt = q - mt * ntn_s;
        row0 = mt * BM;
        rows = p.shared_rows - row0;
        if (rows > BM) rows = BM;
    } else {
        i -= chunk_s;
        const int n_r = *p.n_tiles * ntn_r;
        const int chunk_r = (n_r + 7) >> 3;
        const int q = home * chunk_r + i;
        if (i >= chunk_r || q >= n_r) return;
        const int mt = q / ntn_r;
        nt = q - mt * ntn_r;
        expert = st_entry(p.tile_expert, mt);
        row0 = st_entry(p.tile_row0, mt);
        rows = st_entry(p.tile_rows, mt);
    }
    const Group &g = shared ? p.shared : p.routed;
    const int k_dim = g.k_dim, n_out = g.n_out;
    const int64_t lda = g.lda;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 31, lh = lane >> 5;
    const int nb = (rows + 31) >> 5;

    // copy i of a wavefront fills the 64 chunk positions of piece i * WAVES + wave of A (rows past the end
    // repeat the last one) and of its own 32 weight rows
    uint32_t a_off[ST::a_copies(MB)], b_off[ST::W_COPIES];
#pragma unroll
    for (int j = 0; j < ST::a_copies(MB); ++j) {
        int piece = j * ST::WAVES + wave;
        if (piece >= nb * 4) piece -= nb * 4;
        if (piece >= nb * 4) piece = 0;          // (bands that are not copied)
        int r, c;
        st_place(piece * 64 + lane, r, c);
        const int rr = r < rows ? r : rows - 1;
        const int64_t row = g.gather ? (int64_t)g.gather[row0 + rr] : (int64_t)rr;
        a_off[j] = (uint32_t)((row * lda + c * 8) * 2);
    }
    const char *a_base = reinterpret_cast<const char *>(g.gather ? g.a : g.a + (int64_t)row0 * lda);
    const int64_t estride = (int64_t)n_out * k_dim;
    const char *b_base0 = reinterpret_cast<const char *>(g.b0 + expert * estride);
    const char *b_base1 = MODE == 0 ? reinterpret_cast<const char *>(g.b1 + expert * estride) : b_base0;
#pragma unroll
    for (int j = 0; j < ST::W_COPIES; ++j) {
        int r, c;
        st_place((wave * ST::W_COPIES + j) * 64 + lane, r, c);
        int row = MODE == 0 ? nt * BN + wave * 16 + (r & 15) : nt * BN + r;
        if (row >= n_out) row = n_out - 1;       // ragged last column tile: loads stay in bounds, stores are masked
        b_off[j] = (uint32_t)(((int64_t)row * k_dim + c * 8) * 2);
    }

    floatx16_t acc[ST::TA][TW];
#pragma unroll
    for (int m = 0; m < ST::TA; ++m)
#pragma unroll
        for (int t = 0; t < TW; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[m][t][r] = 0.f;
    const int nk = k_dim / ST_BK;
#define ST_LOOP(NB) stream_loop<MODE, WW, WA, TW, MB, STAGES, DEALT, (NB) <= MB ? (NB) : MB>(smem, a_base, a_off, b_base0, b_base1, b_off, nk, wave, li, lh, acc)
    if (MB == 1 || nb == 1) ST_LOOP(1);
    else if (MB == 2 || nb == 2) ST_LOOP(2);
    else if (MB == 3 || nb == 3) ST_LOOP(3);
    else ST_LOOP(4);
#undef ST_LOOP

    // lane: slot (band) * 32 + li, weight rows 8 q + 4 lh + {0..3} of each of the wavefront's 32-row tiles
#pragma unroll
    for (int m = 0; m < ST::TA; ++m) {
        const int r = (m * WA + wave % WA) * 32 + li;
        if (r >= rows) continue;
        bf16_t *out = g.c + (int64_t)(row0 + r) * g.ldc;
#pragma unroll
        for (int t = 0; t < TW; ++t) {
            const int wt = (wave / WA) * TW + t;         // 32-row tile of the weights
            const floatx16_t &v16 = acc[m][t];
            if (MODE == 0) {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float gt = v16[4 * q + e], up = v16[4 * (q + 2) + e];
                        v[e] = gt * up * __builtin_amdgcn_rcpf(1.0f + __expf(-gt));   // the 1-ulp reciprocal is far inside bf16 rounding
                    }
                    const int col = nt * BN + wt * 16 + 8 * q + 4 * lh;
                    const u32x2_t pk = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
                    if (col < n_out) *reinterpret_cast<u32x2_t *>(out + col) = pk;
                }
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int col = nt * BN + wt * 32 + 8 * q + 4 * lh;
                    const u32x2_t pk = {pack_bf16x2(v16[4 * q], v16[4 * q + 1]), pack_bf16x2(v16[4 * q + 2], v16[4 * q + 3])};
                    if (col < n_out) *reinterpret_cast<u32x2_t *>(out + col) = pk;
                }
            }
        }
    }
}

}  // namespace

template <int WW, int WA, int TW, int MB, int STAGES, bool DEALT>
static void launch_one(int mode, const SArgs &p, int64_t max_tiles, hipStream_t stream)
{
    constexpr int WROWS = 32 * WW * TW;
    const int bn = mode == 0 ? WROWS / 2 : WROWS;
    const int64_t per_xcd = ceil_div(max_tiles * ceil_div(p.routed.n_out, bn), 8) +
                            ceil_div(ceil_div(p.shared_rows, 32 * MB) * ceil_div(p.shared.n_out, bn), 8);
    const dim3 grid((unsigned)(8 * per_xcd)), block(WW * WA * 64);
    if (mode == 0) hipLaunchKernelGGL((stream_gemm_kernel<0, WW, WA, TW, MB, STAGES, DEALT>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((stream_gemm_kernel<1, WW, WA, TW, MB, STAGES, DEALT>), grid, block, 0, stream, p);
}

remoe_status launch_stream_gemm(int mode, const GroupedGemmArgs &r, const GroupedGemmArgs *s, int tile_m, hipStream_t stream)
{
    const int64_t span = (int64_t)1 << 32;       // offsets inside one operand are 32-bit
    for (const GroupedGemmArgs *g : {&r, s}) {
        if (!g) continue;
        if (g->k_dim % ST_BK != 0 || g->n_out < 1 || g->n_out % 8 != 0)
            return fail(REMOE_E_UNSUPPORTED, "bf16 GEMM needs k %% 64 == 0 and n %% 8 == 0 (k=%d n=%d)", g->k_dim, g->n_out);
        if (g->row_gather && g->a_rows * g->lda * 2 >= span)
            return fail(REMOE_E_UNSUPPORTED, "gathered GEMM operand spans 4 GiB or more (%lld rows)", (long long)g->a_rows);
        if ((int64_t)g->n_out * g->k_dim * 2 >= span || g->lda * 2 * 128 >= span)
            return fail(REMOE_E_UNSUPPORTED, "one expert matrix or row tile spans 4 GiB or more");
    }

    SArgs p{};
    auto fill = [](Group &g, const GroupedGemmArgs &a) {
        g.a = static_cast<const bf16_t *>(a.a);
        g.lda = a.lda;
        g.gather = a.row_gather;
        g.b0 = static_cast<const bf16_t *>(a.b0);
        g.b1 = static_cast<const bf16_t *>(a.b1);
        g.k_dim = a.k_dim;
        g.n_out = a.n_out;
        g.c = static_cast<bf16_t *>(a.c) + a.c_row_offset * a.ldc;
        g.ldc = a.ldc;
    };
    fill(p.routed, r);
    p.tile_expert = r.tile_expert; p.tile_row0 = r.tile_row0; p.tile_rows = r.tile_rows; p.n_tiles = r.n_tiles;
    fill(p.shared, s ? *s : r);
    p.shared_rows = s ? (int)s->dense_rows : 0;
    if (tile_m == 32) launch_one<4, 1, 1, 1, 4, false>(mode, p, r.max_tiles, stream);
    else if (tile_m == 64) launch_one<4, 1, 1, 2, 3, false>(mode, p, r.max_tiles, stream);
    else launch_one<4, 2, 2, 4, 3, true>(mode, p, r.max_tiles, stream);
    return check_hip(hipGetLastError(), "stream_gemm launch");
}

}  // namespace remoe
