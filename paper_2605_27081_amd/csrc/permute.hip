// Token -> expert counting sort ("permute") and the tile map of the grouped GEMMs.
//
// The routed experts execute on the rows assigned to them (Sec. 4.1, step 5), so the T*K
// (token, j) pairs are sorted by expert id.  The sort is stable (tokens stay in increasing order
// inside an expert) and free of atomics on global memory, hence deterministic:
//   1. permute_count : per workgroup of 256 tokens, an LDS bit matrix [expert][token] gives each
//                      pair its rank among the workgroup's pairs of the same expert, plus the
//                      workgroup's expert histogram;
//   2. permute_scan  : one workgroup turns the histograms into per-workgroup offsets, the
//                      exclusive prefix sum over experts and the list of GEMM row tiles;
//   3. permute_place : slot = offset[expert] + block offset + rank; writes slot -> token and
//                      pair -> slot.
// For few pairs the three are one launch of one workgroup (permute_small): each step is then shorter than the launch
// and the memory round trip between it and the next, until one compute unit's scattered stores take longer.  Whole
// layer, three launches / one (us): 128 experts, top-8, 16 tokens 28.7 / 24.2, 333 tokens 34.2 / 28.7, 1000 tokens
// 38.0 / 38.4, 2048 tokens 45.7 / 55.0; 60 experts, top-4, 16 tokens 26.0 / 22.5, 1024 tokens 30.9 / 28.0, 1500
// tokens 32.5 / 30.3, 2048 tokens 34.5 / 34.1, 3000 tokens 36.3 / 39.9; hence PSM_PAIRS.
#include "common.h"

namespace remoe {

namespace {

constexpr int PM_TOKENS = 256;  // tokens per workgroup in steps 1 and 3

__global__ __launch_bounds__(PM_TOKENS) void permute_count(const int32_t *__restrict__ idx, int64_t T,
                                                           int K, int N,
                                                           int32_t *__restrict__ blk_hist,
                                                           int32_t *__restrict__ pair_rank)
{
    __shared__ uint32_t bits[128][PM_TOKENS / 32];
    const int tid = threadIdx.x;
    for (int q = tid; q < 128 * (PM_TOKENS / 32); q += PM_TOKENS) (&bits[0][0])[q] = 0u;
    __syncthreads();
    const int64_t t = (int64_t)blockIdx.x * PM_TOKENS + tid;
    const int word = tid >> 5;
    const uint32_t bit = 1u << (tid & 31);
    if (t < T)
        for (int j = 0; j < K; ++j) atomicOr(&bits[idx[t * K + j]][word], bit);
    __syncthreads();
    if (t < T)
        for (int j = 0; j < K; ++j) {
            const int e = idx[t * K + j];
            int rank = __popc(bits[e][word] & (bit - 1u));
            for (int w = 0; w < word; ++w) rank += __popc(bits[e][w]);
            pair_rank[t * K + j] = rank;
        }
    if (tid < N) {
        int c = 0;
#pragma unroll
        for (int w = 0; w < PM_TOKENS / 32; ++w) c += __popc(bits[tid][w]);
        blk_hist[(int64_t)blockIdx.x * N + tid] = c;
    }
}

// One wavefront: off and tstart (129 entries) become the exclusive prefix sums of the experts' pairs and row tiles.
// (One thread walking the 128 counts took 6 us of the launch.)
__device__ __forceinline__ void scan_experts(const int32_t *cnt, int tile_m, int max_tiles, int32_t *off, int32_t *tstart,
                                             int32_t *__restrict__ n_tiles)
{
    const int lane = threadIdx.x & 63;
    const int c0 = cnt[2 * lane], c1 = cnt[2 * lane + 1];
    const int t0 = (c0 + tile_m - 1) / tile_m, t1 = (c1 + tile_m - 1) / tile_m;
    int c = c0 + c1, t = t0 + t1;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int oc = __shfl_up(c, d, 64), ot = __shfl_up(t, d, 64);
        if (lane >= d) {
            c += oc;
            t += ot;
        }
    }
    off[2 * lane] = c - c0 - c1;
    off[2 * lane + 1] = c - c1;
    tstart[2 * lane] = t - t0 - t1;
    tstart[2 * lane + 1] = t - t1;
    if (lane == 63) {
        off[128] = c;
        tstart[128] = t;
        *n_tiles = t < max_tiles ? t : max_tiles;
    }
}

__device__ __forceinline__ void list_tiles(int e, const int32_t *cnt, const int32_t *off, const int32_t *tstart, int tile_m, int max_tiles,
                                           int32_t *__restrict__ tile_expert, int32_t *__restrict__ tile_row0,
                                           int32_t *__restrict__ tile_rows)
{
    for (int ti = tstart[e], i = 0; ti < tstart[e + 1] && ti < max_tiles; ++ti, ++i) {
        tile_expert[ti] = e;
        tile_row0[ti] = off[e] + i * tile_m;
        const int left = cnt[e] - i * tile_m;
        tile_rows[ti] = left < tile_m ? left : tile_m;
    }
}

// One workgroup of PS_SEG x 128 threads: thread (seg, e) owns expert e's counts of one segment of the
// token blocks, so the running sums over the blocks are PS_SEG times shorter chains of loads.
constexpr int PS_SEG = 8;
__global__ __launch_bounds__(PS_SEG * 128) void permute_scan(const int32_t *__restrict__ blk_hist, int n_blk,
                                                    int N, int tile_m, int max_tiles,
                                                    int32_t *__restrict__ blk_off,
                                                    int32_t *__restrict__ offsets,
                                                    int32_t *__restrict__ tile_expert,
                                                    int32_t *__restrict__ tile_row0,
                                                    int32_t *__restrict__ tile_rows,
                                                    int32_t *__restrict__ n_tiles, uint32_t *__restrict__ gemm_ctr)
{
    __shared__ int32_t cnt[128], off[129], tstart[129], seg_sum[PS_SEG][128];
    const int e = threadIdx.x & 127, seg = threadIdx.x >> 7;
    if (threadIdx.x < GEMM_CTR_SETS * 8) gemm_ctr[threadIdx.x] = 0u;   // tile counters of the GEMM launches that follow
    const int per_seg = (n_blk + PS_SEG - 1) / PS_SEG;
    const int b0 = seg * per_seg, b1 = (b0 + per_seg < n_blk) ? b0 + per_seg : n_blk;
    int sum = 0;
    if (e < N) {
#pragma unroll 8
        for (int b = b0; b < b1; ++b) sum += blk_hist[(int64_t)b * N + e];
    }
    seg_sum[seg][e] = sum;
    __syncthreads();
    int run = 0;
    for (int q = 0; q < seg; ++q) run += seg_sum[q][e];
    if (e < N) {
#pragma unroll 8
        for (int b = b0; b < b1; ++b) {
            const int c = blk_hist[(int64_t)b * N + e];
            blk_off[(int64_t)b * N + e] = run;
            run += c;
        }
    }
    if (seg == PS_SEG - 1) cnt[e] = (e < N) ? run : 0;   // the last segment ends with the expert's total
    __syncthreads();
    if (threadIdx.x < 64) scan_experts(cnt, tile_m, max_tiles, off, tstart, n_tiles);
    __syncthreads();
    if (seg == 0 && e <= N) offsets[e] = off[e];
    if (threadIdx.x == 0 && N == 128) offsets[128] = off[128];
    if (seg == 0 && e < N) list_tiles(e, cnt, off, tstart, tile_m, max_tiles, tile_expert, tile_row0, tile_rows);
}

// All three steps for up to 1024 * TPT tokens: bits[e] marks the tokens of expert e (rows padded by a word, so that the
// experts of neighbouring tokens fall into different banks), before[e] counts the marks in front of each word.
constexpr int PSM_BLOCK = 1024, PSM_PAIRS = 6144;
template <int TPT>
__global__ __launch_bounds__(PSM_BLOCK) void permute_small(const int32_t *__restrict__ idx, int T, int K, int N, int tile_m, int max_tiles,
                                                           int32_t *__restrict__ offsets, int32_t *__restrict__ tile_expert,
                                                           int32_t *__restrict__ tile_row0, int32_t *__restrict__ tile_rows,
                                                           int32_t *__restrict__ n_tiles, uint32_t *__restrict__ gemm_ctr,
                                                           int32_t *__restrict__ pair_slot, int32_t *__restrict__ slot_token)
{
    constexpr int W = PSM_BLOCK / 32 * TPT, PER = W / 8;       // words of a row; of a thread that counts them
    __shared__ uint32_t bits[128][W + 1];
    __shared__ uint16_t before[128][W + 2];
    __shared__ int32_t cnt[128], off[129], tstart[129];
    const int tid = threadIdx.x;
    if (tid < GEMM_CTR_SETS * 8) gemm_ctr[tid] = 0u;           // tile counters of the GEMM launches that follow
    for (int q = tid; q < 128 * (W + 1); q += PSM_BLOCK) (&bits[0][0])[q] = 0u;
    __syncthreads();
    int32_t e[TPT][8];
#pragma unroll
    for (int i = 0; i < TPT; ++i) {
        const int t = tid + i * PSM_BLOCK;
#pragma unroll
        for (int j = 0; j < 8; ++j) e[i][j] = t < T && j < K ? idx[t * K + j] : -1;
    }
#pragma unroll
    for (int i = 0; i < TPT; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (e[i][j] >= 0) atomicOr(&bits[e[i][j]][(tid >> 5) + i * (PSM_BLOCK / 32)], 1u << (tid & 31));
    __syncthreads();
    {
        const int row = tid >> 3, q = tid & 7;
        int sum = 0;
        int upto[PER];
#pragma unroll
        for (int w = 0; w < PER; ++w) {
            upto[w] = sum;
            sum += __popc(bits[row][q * PER + w]);
        }
        int run = sum;
#pragma unroll
        for (int d = 1; d < 8; d <<= 1) {
            const int o = __shfl_up(run, d, 8);
            if (q >= d) run += o;
        }
#pragma unroll
        for (int w = 0; w < PER; ++w) before[row][q * PER + w] = (uint16_t)(run - sum + upto[w]);
        if (q == 7) cnt[row] = run;
    }
    __syncthreads();
    if (tid < 64) scan_experts(cnt, tile_m, max_tiles, off, tstart, n_tiles);
    __syncthreads();
    if (tid <= N) offsets[tid] = off[tid];
    if (tid < N) list_tiles(tid, cnt, off, tstart, tile_m, max_tiles, tile_expert, tile_row0, tile_rows);
#pragma unroll
    for (int i = 0; i < TPT; ++i) {
        const int t = tid + i * PSM_BLOCK, word = (tid >> 5) + i * (PSM_BLOCK / 32);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int x = e[i][j];
            if (x < 0) continue;
            const int slot = off[x] + before[x][word] + __popc(bits[x][word] & ((1u << (tid & 31)) - 1u));
            pair_slot[t * K + j] = slot;
            slot_token[slot] = t;
        }
    }
}

__global__ __launch_bounds__(256) void permute_place(const int32_t *__restrict__ idx,
                                                     int64_t n_pairs,
                                                     int K, int N,
                                                     const int32_t *__restrict__ blk_off,
                                                     const int32_t *__restrict__ offsets,
                                                     int32_t *__restrict__ pair_slot,
                                                     int32_t *__restrict__ slot_token)
{
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= n_pairs) return;
    const int64_t t = p / K;
    const int e = idx[p];
    const int slot = offsets[e] + blk_off[(t / PM_TOKENS) * N + e] + pair_slot[p];
    pair_slot[p] = slot;
    slot_token[slot] = (int32_t)t;
}

}  // namespace

int permute_tokens_per_block() { return PM_TOKENS; }

remoe_status launch_permute(const int32_t *idx, int64_t T, int K, int N,
                            int tile_m, int max_tiles, const PermuteBuffers &pb, hipStream_t stream)
{
    if (T == 0) return REMOE_OK;
    if (T <= 2 * PSM_BLOCK && T * K <= PSM_PAIRS) {
        auto kernel = T <= PSM_BLOCK ? permute_small<1> : permute_small<2>;
        hipLaunchKernelGGL(kernel, dim3(1), dim3(PSM_BLOCK), 0, stream, idx, (int)T, K, N, tile_m, max_tiles, pb.offsets, pb.tile_expert,
                           pb.tile_row0, pb.tile_rows, pb.n_tiles, pb.gemm_ctr, pb.pair_slot, pb.slot_token);
        return check_hip(hipGetLastError(), "permute_small launch");
    }
    const int n_blk = (int)ceil_div(T, PM_TOKENS);
    int32_t *blk_hist = pb.blk_hist;
    int32_t *blk_off = pb.blk_hist + (int64_t)n_blk * N;
    hipLaunchKernelGGL(permute_count, dim3(n_blk), dim3(PM_TOKENS), 0, stream, idx, T, K, N, blk_hist,
                       pb.pair_slot);
    hipLaunchKernelGGL(permute_scan, dim3(1), dim3(PS_SEG * 128), 0, stream, blk_hist, n_blk, N, tile_m,
                       max_tiles, blk_off, pb.offsets, pb.tile_expert, pb.tile_row0, pb.tile_rows,
                       pb.n_tiles, pb.gemm_ctr);
    const int64_t n_pairs = T * K;
    hipLaunchKernelGGL(permute_place, dim3((unsigned)ceil_div(n_pairs, 256)), dim3(256), 0, stream, idx,
                       n_pairs, K, N, blk_off, pb.offsets, pb.pair_slot, pb.slot_token);
    return check_hip(hipGetLastError(), "permute launch");
}

}  // namespace remoe
