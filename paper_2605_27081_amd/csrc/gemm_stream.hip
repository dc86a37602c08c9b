// Grouped expert GEMMs for few rows per expert (bf16 with fp32 accumulation, the weights are streamed), and for fp32
// layers of any size.
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
// GEMMs together, 256-row kernel before / this kernel: 16 tokens 218 / 128 us (0.72 GB past the L2 at
// 5.6 TB/s, matrix cores busy 8 % of the time), 333 tokens 327 / 221 us (1.24 GB at 5.6 TB/s, 9 %).  With 128-row
// tiles (1021 tokens, 60 experts, shared expert) 1.35 GB pass the L2s, 1.11 GB of them weights.  Slices of 32 k-values (64-byte rows) with twice the stages
// were 5-10 % slower throughout.
//
// The MFMAs take the weight rows as their first operand, so a lane owns one slot (row of the output) and,
// per group of four accumulators, four adjacent weight rows.  In mode 0 every 32-row group of the weights is
// 16 gate rows followed by the 16 up rows of the same columns, so g and u of one output meet in one lane.
//
// fp32 layers use the same tiles and the same 128-byte rows, 32 k-values each, on v_mfma_f32_32x32x2_f32 (a
// lane's 16 bytes feed four of them).  There the matrix cores bound anything but the smallest layers: a slice is
// 2 KB of copies per 64-cycle MFMA row.  Their sizes need not be multiples of anything: the activations between the two
// GEMMs are padded with zeros to whole slices, and a weight matrix whose rows are not whole slices
// (the down projection of an I that is no multiple of 32) goes through registers, 4 bytes at a time and zero past the
// row's end.  Tiny layer (128 tokens, 16 experts, H 256, I 128), 64 x 64 FMA tiles before / this kernel: gate/up
// 47 / 11 us, down 22 / 5 us.
//
// Tiles whose rows fill only NB of the MB 32-row bands copy and multiply only those.
//
// The shared expert (dense, all tokens) runs in the same launch as one more group with its own operands
// and sizes: its matrix work fills the routed experts' waits for memory, and no launch ends half empty in
// between.  Its tiles come first (in mode 1 they are the longer ones) and are dealt evenly to the XCDs, all row tiles
// of one column tile (up to ST_GROUP, which is as good with 8 and with 32) in a row: an XCD then fetches its share of the weights once.
// With one row tile's columns in a row, every XCD fetched them all: 1021 tokens, 60 experts, shared expert of
// 5632: 1.69 against 1.35 GB past the L2s, the layer 323 against 308 us; 333 tokens 274 / 258.
#include <type_traits>

#include "common.h"
#include "lds_copy.h"

namespace remoe {

namespace {

typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;
constexpr int ST_ROW = 128;      // bytes of a row per slice: 64 bf16 or 32 fp32 k-values

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
    const void *a;
    int64_t lda;                 // elements between rows of a, a whole number of slices
    const int32_t *gather;       // slot -> row of a, or NULL
    const void *b0, *b1;
    int k_dim, n_out;            // columns of a weight row, weight rows per matrix
    void *c;                     // first output row of the group
    int64_t ldc;
    int n_store;                 // columns written; those past n_out are zeros
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

constexpr int ST_GROUP = 16;     // row tiles of the shared expert that are worked on together

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

// Offsets of the gathered rows: 32 bits for bf16 (the launcher checks), 64 for fp32, whose batches may be any size.
template <typename ET> using RowOffset = typename std::conditional<sizeof(ET) == 2, uint32_t, uint64_t>::type;

// the MFMAs that 16 bytes of a weight row and of a slot's row feed
__device__ __forceinline__ void mfma16(bf16_t, const u32x4_t &w, const u32x4_t &a, floatx16_t &acc)
{
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, w), __builtin_bit_cast(bf16x8_t, a), acc, 0, 0, 0);
}
__device__ __forceinline__ void mfma16(float, const u32x4_t &w, const u32x4_t &a, floatx16_t &acc)
{
#pragma unroll
    for (int i = 0; i < 4; ++i)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(w[i]), __uint_as_float(a[i]), acc, 0, 0, 0);
}

__device__ __forceinline__ float swiglu(bf16_t, float g, float u)
{
    return g * u * __builtin_amdgcn_rcpf(1.0f + __expf(-g));   // the 1-ulp reciprocal is far inside bf16 rounding
}
__device__ __forceinline__ float swiglu(float, float g, float u) { return g / (1.0f + expf(-g)) * u; }

// four neighbouring columns of one output row, the first `n` of which exist
__device__ __forceinline__ void store4(bf16_t *out, const float (&v)[4], int n)
{
    const u32x2_t pk = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
    if (n > 0) *reinterpret_cast<u32x2_t *>(out) = pk;           // bf16 widths are multiples of 8
}
__device__ __forceinline__ void store4(float *out, const float (&v)[4], int n)
{
    if (n >= 4) *reinterpret_cast<floatx4_t *>(out) = floatx4_t{v[0], v[1], v[2], v[3]};     // fp32 row pitches are multiples of 32
    else
        for (int e = 0; e < n; ++e) out[e] = v[e];
}

// The reduction of one tile with NB bands of 32 rows (NT: bands of this wavefront, a band past NB is not stored).
template <typename ET, int MODE, int WW, int WA, int TW, int MB, int STAGES, bool DEALT, int NB, bool RAGGED>
__device__ __forceinline__ void stream_loop(u32x4_t *smem, const char *a_base, const RowOffset<ET> *a_off, const char *b_base0,
                                            const char *b_base1, const uint32_t *b_off, int k_dim, int nk, int wave, int lane,
                                            floatx16_t (&acc)[MB / WA][TW])
{
    typedef StreamTile<WW, WA, TW, MB> ST;
    constexpr int NT = (NB + WA - 1) / WA;
    constexpr int A_COPIES = ST::a_copies(NB), A_INSTR = NB * 4;
    constexpr int W_COPIES = RAGGED ? 0 : ST::W_COPIES;
    constexpr int COPIES = W_COPIES + A_COPIES;
    const int li = lane & 31, lh = lane >> 5;
    // copy c of slice j -> stage st (past the end the last slice again: the count of outstanding copies never varies)
    auto copy = [&](int j, u32x4_t *st, int c) __attribute__((always_inline)) {
        const int64_t k = (int64_t)(j < nk ? j : nk - 1) * ST_ROW;
        if (c < W_COPIES) {
            copy16_to_lds((MODE == 0 && c >= W_COPIES / 2 ? b_base1 : b_base0) + k, b_off[c], st + (wave * W_COPIES + c) * 64);
        } else {
            int g = (c - W_COPIES) * ST::WAVES + wave;
            if (A_INSTR % ST::WAVES != 0 && g >= A_INSTR) g -= A_INSTR;      // fewer pieces than wavefronts: fetched twice
            copy16_to_lds(a_base + k, a_off[c - W_COPIES], st + ST::W_U4 + g * 64);
        }
    };
    // RAGGED (fp32): slice j of this wavefront's 32 weight rows through registers, half a wavefront per row; b_off[0] is
    // its first row, b_off[1] the last of its rows that exists
    float wv[RAGGED ? 16 : 1];
    auto w_load = [&](int j) __attribute__((always_inline)) {
        const int k = j * (ST_ROW / 4) + (lane & 31);
#pragma unroll
        for (int i = 0; i < (RAGGED ? 16 : 0); ++i) {
            const int row = 2 * i + (lane >> 5), last = (int)b_off[1];
            const float *src = reinterpret_cast<const float *>(b_base0) + (int64_t)(b_off[0] + (row < last ? row : last)) * k_dim;
            wv[i] = k < k_dim ? src[k] : 0.f;
        }
    };
    auto w_store = [&](u32x4_t *st) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < (RAGGED ? 16 : 0); ++i)
            reinterpret_cast<float *>(&st[st_slot(wave * 32 + 2 * i + (lane >> 5), (lane & 31) >> 2)])[lane & 3] = wv[i];
    };
    if (RAGGED) {
        w_load(0);
        w_store(smem);
        w_load(1);
    }
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
        if (RAGGED) {
            w_store(smem + (cur + 1 == STAGES ? 0 : cur + 1) * ST::STAGE);
            w_load(kt + 2);
        }
        u32x4_t w8[2][TW], a8[2][NT];
#define ST_READ(ks)                                                                                                   \
    _Pragma("unroll") for (int t = 0; t < TW; ++t)                                                                    \
        w8[(ks) & 1][t] = st[st_slot(w_row + t * 32, 2 * (ks) + lh)];                                                  \
    _Pragma("unroll") for (int m = 0; m < NT; ++m)                                                                    \
        a8[(ks) & 1][m] = st[ST::W_U4 + st_slot(a_row + m * WA * 32, 2 * (ks) + lh)];
#define ST_MFMA(ks)                                                                                                   \
    _Pragma("unroll") for (int m = 0; m < NT; ++m)                                                                    \
        _Pragma("unroll") for (int t = 0; t < TW; ++t)                                                                \
            mfma16(ET(), w8[(ks) & 1][t], a8[(ks) & 1][m], acc[m][t]);
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

template <typename ET, int MODE, int WW, int WA, int TW, int MB, int STAGES, bool DEALT>
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
        // groups of row tiles, row tile fastest inside one
        const int n_mt = (p.shared_rows + BM - 1) / BM, n_groups = (n_mt + ST_GROUP - 1) / ST_GROUP;
        const int per_group = (n_mt + n_groups - 1) / n_groups, grp = q / (per_group * ntn_s), left = n_mt - grp * per_group;
        const int here = left < per_group ? left : per_group, in_group = q - grp * per_group * ntn_s;
        nt = in_group / here;
        const int mt = grp * per_group + in_group - nt * here;
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
    RowOffset<ET> a_off[ST::a_copies(MB)];
    uint32_t b_off[ST::W_COPIES];
#pragma unroll
    for (int j = 0; j < ST::a_copies(MB); ++j) {
        int piece = j * ST::WAVES + wave;
        if (piece >= nb * 4) piece -= nb * 4;
        if (piece >= nb * 4) piece = 0;          // (bands that are not copied)
        int r, c;
        st_place(piece * 64 + lane, r, c);
        const int rr = r < rows ? r : rows - 1;
        const int64_t row = g.gather ? (int64_t)g.gather[row0 + rr] : (int64_t)rr;
        a_off[j] = (RowOffset<ET>)(row * lda * (int)sizeof(ET) + c * 16);
    }
    const ET *a_rows = static_cast<const ET *>(g.a);
    const char *a_base = reinterpret_cast<const char *>(g.gather ? a_rows : a_rows + (int64_t)row0 * lda);
    const int64_t first = ((int64_t)expert * n_out + nt * BN) * k_dim;      // the tile's first weight
    const char *b_base0 = reinterpret_cast<const char *>(static_cast<const ET *>(g.b0) + first);
    const char *b_base1 = MODE == 0 ? reinterpret_cast<const char *>(static_cast<const ET *>(g.b1) + first) : b_base0;
    const int last = n_out - 1 - nt * BN;        // ragged last column tile: rows past the end repeat the last, stores are masked
#pragma unroll
    for (int j = 0; j < ST::W_COPIES; ++j) {
        int r, c;
        st_place((wave * ST::W_COPIES + j) * 64 + lane, r, c);
        const int row = MODE == 0 ? wave * 16 + (r & 15) : r;
        b_off[j] = (uint32_t)(row < last ? row : last) * (uint32_t)(k_dim * (int)sizeof(ET)) + c * 16;
    }

    floatx16_t acc[ST::TA][TW];
#pragma unroll
    for (int m = 0; m < ST::TA; ++m)
#pragma unroll
        for (int t = 0; t < TW; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[m][t][r] = 0.f;
    const int nk = (k_dim * (int)sizeof(ET) + ST_ROW - 1) / ST_ROW;
#define ST_LOOP(NB, RAGGED)                                                                                                    \
    stream_loop<ET, MODE, WW, WA, TW, MB, STAGES, DEALT, (NB) <= MB ? (NB) : MB, RAGGED>(smem, a_base, a_off, b_base0, b_base1, \
                                                                                        b_off, k_dim, nk, wave, lane, acc)
    if (MODE == 1 && sizeof(ET) == 4 && k_dim % (ST_ROW / 4) != 0) {
        b_off[0] = (uint32_t)(wave * 32 < last ? wave * 32 : last);
        b_off[1] = (uint32_t)last - b_off[0];
        ST_LOOP(MB, (MODE == 1 && sizeof(ET) == 4));
    } else if (MB == 1 || nb == 1) ST_LOOP(1, false);
    else if (MB == 2 || nb == 2) ST_LOOP(2, false);
    else if (MB == 3 || nb == 3) ST_LOOP(3, false);
    else ST_LOOP(4, false);
#undef ST_LOOP

    // lane: slot (band) * 32 + li, weight rows 8 q + 4 lh + {0..3} of each of the wavefront's 32-row tiles
#pragma unroll
    for (int m = 0; m < ST::TA; ++m) {
        const int r = (m * WA + wave % WA) * 32 + li;
        if (r >= rows) continue;
        ET *out = static_cast<ET *>(g.c) + (int64_t)(row0 + r) * g.ldc;
#pragma unroll
        for (int t = 0; t < TW; ++t) {
            const int wt = (wave / WA) * TW + t;         // 32-row tile of the weights
            const floatx16_t &v16 = acc[m][t];
#pragma unroll
            for (int q = 0; q < (MODE == 0 ? 2 : 4); ++q) {
                const int col = nt * BN + (MODE == 0 ? wt * 16 : wt * 32) + 8 * q + 4 * lh;
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[e] = MODE == 0 ? swiglu(ET(), v16[4 * q + e], v16[4 * ((q + 2) & 3) + e]) : v16[4 * q + e];
                    if (sizeof(ET) == 4 && col + e >= n_out) v[e] = 0.f;
                }
                store4(out + col, v, g.n_store - col);
            }
        }
    }
}

}  // namespace

template <typename ET, int WW, int WA, int TW, int MB, int STAGES, bool DEALT>
static void launch_one(int mode, const SArgs &p, int64_t max_tiles, hipStream_t stream)
{
    constexpr int WROWS = 32 * WW * TW;
    const int bn = mode == 0 ? WROWS / 2 : WROWS;
    const int64_t per_xcd = ceil_div(max_tiles * ceil_div(p.routed.n_out, bn), 8) +
                            ceil_div(ceil_div(p.shared_rows, 32 * MB) * ceil_div(p.shared.n_out, bn), 8);
    const dim3 grid((unsigned)(8 * per_xcd)), block(WW * WA * 64);
    if (mode == 0) hipLaunchKernelGGL((stream_gemm_kernel<ET, 0, WW, WA, TW, MB, STAGES, DEALT>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((stream_gemm_kernel<ET, 1, WW, WA, TW, MB, STAGES, DEALT>), grid, block, 0, stream, p);
}

remoe_status launch_stream_gemm(int dtype, int mode, const GroupedGemmArgs &r, const GroupedGemmArgs *s, int tile_m, hipStream_t stream)
{
    const int es = dtype == REMOE_F32 ? 4 : 2;
    const int64_t span = (int64_t)1 << 32;       // offsets inside one operand are 32-bit
    for (const GroupedGemmArgs *g : {&r, s}) {
        if (!g) continue;
        const bool ragged_ok = dtype == REMOE_F32 && mode == 1;
        if (g->n_out < 1 || (g->k_dim * es % ST_ROW != 0 && !ragged_ok) || g->lda * es % 16 != 0 || (es == 2 && g->n_out % 8 != 0))
            return fail(REMOE_E_UNSUPPORTED, "GEMM with k=%d n=%d of dtype %d", g->k_dim, g->n_out, dtype);
        if (es == 2 && g->row_gather && g->a_rows * g->lda * es >= span)
            return fail(REMOE_E_UNSUPPORTED, "gathered GEMM operand spans 4 GiB or more (%lld rows)", (long long)g->a_rows);
        if ((int64_t)g->k_dim * es * 256 >= span || g->lda * es * 128 >= span)
            return fail(REMOE_E_UNSUPPORTED, "one tile of the weights or of the rows spans 4 GiB or more");
    }
    SArgs p{};
    auto fill = [&](Group &g, const GroupedGemmArgs &a) {
        g.a = a.a;
        g.lda = a.lda;
        g.gather = a.row_gather;
        g.b0 = a.b0;
        g.b1 = a.b1;
        g.k_dim = a.k_dim;
        g.n_out = a.n_out;
        g.c = static_cast<char *>(a.c) + a.c_row_offset * a.ldc * es;
        g.ldc = a.ldc;
        g.n_store = mode == 0 ? (int)a.ldc : a.n_out;
    };
    fill(p.routed, r);
    p.tile_expert = r.tile_expert; p.tile_row0 = r.tile_row0; p.tile_rows = r.tile_rows; p.n_tiles = r.n_tiles;
    fill(p.shared, s ? *s : r);
    p.shared_rows = s ? (int)s->dense_rows : 0;
    if (dtype == REMOE_F32) {
        if (tile_m == 32) launch_one<float, 4, 1, 1, 1, 4, false>(mode, p, r.max_tiles, stream);
        else launch_one<float, 4, 1, 1, 2, 3, false>(mode, p, r.max_tiles, stream);
    } else {
        if (tile_m == 32) launch_one<bf16_t, 4, 1, 1, 1, 4, false>(mode, p, r.max_tiles, stream);
        else if (tile_m == 64) launch_one<bf16_t, 4, 1, 1, 2, 3, false>(mode, p, r.max_tiles, stream);
        else launch_one<bf16_t, 4, 2, 2, 4, 3, true>(mode, p, r.max_tiles, stream);
    }
    return check_hip(hipGetLastError(), "stream_gemm launch");
}

}  // namespace remoe
