// sp_score / sp_score_batch: token importance from the lookahead queries'
// attention over the prompt keys (paper: Appendix A.1.1; Algorithm 1,
// "AggregateMaxMean").
//
// Three kernels, all built around the bf16 32x32x16 MFMA of gfx950:
//   stats   one workgroup per (key tile, layer, kv head): logits of the kv
//           head's whole query group against 256 keys, per-row running
//           (max, sum of exp) kept per lane, one partial per (row, tile);
//   merge   log-sum-exp combination of the partials of each row in a fixed
//           order (deterministic), giving the row's normaliser (short prompts:
//           at the start of prob, see prob_merges);
//   prob    one workgroup per (key tile, layer range), looping over its layers
//           and the kv heads:
//           logits again with the normaliser folded into the MFMA's C operand,
//           maximum over heads taken on logits (exp is monotone, so
//           max_h softmax_h = exp(max_h(logit_h - lse_h))), one exp per
//           (lookahead row, key), sum over lookahead rows and layers in
//           registers, a single store per key. Long inputs give every
//           workgroup all layers; short ones split the layers over several
//           workgroups per tile, which leave per-range results that a fourth
//           kernel (reduce) combines in a fixed order.
//
// Register/lane layout facts used throughout (v_mfma_f32_32x32x16_bf16):
//   A operand: lane i holds row i%32, eight consecutive k-values of half i/32
//   B operand: lane i holds column i%32, the same eight k-values
//   D: lane i, register r holds row 8*(r/4) + 4*(i/32) + r%4, column i%32.
// Since A and B fragments are laid out alike, one fragment of K serves as A
// (rows = keys) in the stats pass and as B (columns = keys) in the prob pass.
#include "sp_common.hpp"
#include "sp_score_dev.hpp"
#include "sp_score_fused.hpp"
#include "sp_score_plan.hpp"

#include <dlfcn.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <vector>

namespace {

using namespace sp_dev;
using namespace sp_plan;

constexpr int kThreads = 256;
constexpr int kWaves = 4;
constexpr int kMaxPrompts = 4096;
constexpr size_t kLdsBudget = 64 * 1024;
constexpr int kMaxLookRows = 224;           // padded query rows of the widest supported group

struct TileInfo {
    int64_t j0;          // first key of the tile (index into the packed token axis)
    int64_t end;         // one past the last key of the tile's prompt
    int32_t prompt;
    int32_t first_tile;  // index of the prompt's first tile
};

struct ScoreArgs {
    const uint16_t *q;        // [B][Lyr][H][n_q][d]
    int64_t k_stride_token, k_stride_head;
    const TileInfo *tiles;    // null: single prompt, tile t starts at t * tile_keys
    const int32_t *prompt_tiles;  // [B+1] first tile of each prompt (batch only)
    int64_t L;                // tokens of the call (single prompt: its length)
    float2 *part;             // [n_phases][n_tiles][rows_pad]
    float *lse_neg;           // [B][n_phases][rows_pad]  (-lse in raw-logit units, permuted); not used where the prob pass merges
    float *scores;
    uint32_t *status;         // the call's status word (cleared here: this path cannot give up)
    const int32_t *block_table;   // paged keys (single prompt): token j lives in page block_table[j / page_tokens]
    int64_t page_tokens;          // of its layer's pool, page p at element offset p * page_stride; null: contiguous
    int64_t page_stride;
    const float *look;        // [n_phases][rows_pad] lookahead-key term of each row's normaliser, or null
    const float *kscale;      // 8-bit keys: [n_phases] scale of each (layer, kv head); null: bf16 keys
    float *split_buf;         // layer-split results: MEAN [n_splits][L], MAX [n_splits][8*n_nblk][L]
    int32_t n_splits, layers_per_split;
    int32_t n_tiles, n_prompts;
    int32_t n_layers, n_q_heads, n_kv_heads, group, n_q;
    int32_t n_nblk, n_gblk, rows_pad;   // blocks of 8 lookahead rows / 4 group heads
    int32_t layer_agg;
    float c;                  // scale * log2(e)
    float inv_c;
    float out_scale;          // 1/n_q or 1/(n_q * Lyr)
};

__device__ __forceinline__ TileInfo get_tile(const ScoreArgs &a, int tile, int tile_keys)
{
    if (a.tiles) return a.tiles[tile];
    TileInfo t;
    t.j0 = (int64_t)tile * tile_keys;
    t.end = a.L;
    t.prompt = 0;
    t.first_tile = 0;
    return t;
}

// Address of key 0 of the tile's address space in (layer, kv head): the layer's buffer for contiguous
// keys; for paged keys the tile's page, moved back by the page's first token so that the absolute key
// index still applies (tiles never straddle pages: a page holds a multiple of the tile size).
__device__ __forceinline__ const uint16_t *key_base(const ScoreArgs &a, const LayerPtrs &kp, int layer, int kv,
                                                    const TileInfo &ti)
{
    const uint16_t *b = kp.p[layer] + (int64_t)kv * a.k_stride_head;
    if (a.block_table) {
        const int64_t page = ti.j0 / a.page_tokens;
        b += (int64_t)a.block_table[page] * a.page_stride - page * a.page_tokens * a.k_stride_token;
    }
    return b;
}

// Padded query-row order of one kv head's group: row = blk*32 + rho with
// blk = gblk * n_nblk + nblk, rho = 8*gl + nl  ->  group head g = 4*gblk + gl,
// lookahead row n = 8*nblk + nl. In the D layout of the prob pass this puts the
// four group heads of a block in registers r/4 of one lane.
__device__ __forceinline__ bool row_to_gn(const ScoreArgs &a, int row, int &g, int &n)
{
    const int blk = row >> 5, rho = row & 31;
    const int gblk = blk / a.n_nblk, nblk = blk - gblk * a.n_nblk;
    g = 4 * gblk + (rho >> 3);
    n = 8 * nblk + (rho & 7);
    return g < a.group && n < a.n_q;
}

// 8-bit keys (contiguous only): byte address of key 0 of (layer, kv head).
__device__ __forceinline__ const uint8_t *key_base_fp8(const ScoreArgs &a, const LayerPtrs &kp, int layer, int kv)
{
    return reinterpret_cast<const uint8_t *>(kp.p[layer]) + (int64_t)kv * a.k_stride_head;
}

template <int D>
__device__ __forceinline__ void stage_q(u32x4 *qs, const ScoreArgs &a, int prompt, int layer, int kv, int tid)
{
    constexpr int CH = D / 8;
    const uint16_t *qb = a.q + (((int64_t)prompt * a.n_layers + layer) * a.n_q_heads + (int64_t)kv * a.group) *
                                   a.n_q * D;
    for (int i = tid; i < a.rows_pad * CH; i += kThreads) {
        const int row = i / CH, ch = i - row * CH;
        int g, n;
        u32x4 v = {0u, 0u, 0u, 0u};
        if (row_to_gn(a, row, g, n))
            v = *reinterpret_cast<const u32x4 *>(qb + ((int64_t)g * a.n_q + n) * D + ch * 8);
        qs[lds_slot<D>(row, ch)] = v;
    }
}

// The same staging for 8-bit keys: kb8 addresses bytes, strides are in elements (= bytes).
template <int D, int NS>
__device__ __forceinline__ void stage_k_fp8(u32x4 *ks, const uint8_t *kb8, int64_t stride_token, int64_t j0,
                                            int64_t end, int tid)
{
    constexpr int CH = D / 8;
    constexpr int TILE = kWaves * NS * 32;
    constexpr int N = TILE * CH / kThreads;
    uint2 v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int idx = tid + i * kThreads;
        const int row = idx / CH, ch = idx % CH;
        const int64_t j = j0 + row;
        v[i] = *reinterpret_cast<const uint2 *>(kb8 + (j < end ? j : end - 1) * stride_token + ch * 8);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int idx = tid + i * kThreads;
        ks[lds_slot<D>(idx / CH, idx % CH)] = e4m3x8_to_bf16x8(v[i].x, v[i].y);
    }
}

// KERNEL: an instantiation for each kernel with loops of another shape around it. One for all of them takes its address
// arithmetic apart so that it suits neither: 24 x 4 heads of 128, 70001 tokens on the three kernels 825 us against 817,
// 16 x 8 heads of 64, 200003 tokens 1355 against 1347. (8-bit keys gain by the same: 715 us against 750.)
enum StageKernel { kStageGeneral, kStageFinish };
template <int D, int NS, StageKernel KERNEL>
__device__ __forceinline__ void stage_k(u32x4 *ks, const uint16_t *kb, int64_t stride_token, int64_t j0,
                                        int64_t end, int tid)
{
    constexpr int CH = D / 8;
    constexpr int TILE = kWaves * NS * 32;
    constexpr int N = TILE * CH / kThreads;
    u32x4 v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int idx = tid + i * kThreads;
        const int row = idx / CH, ch = idx % CH;
        const int64_t j = j0 + row;
        // rows past the end repeat the last key (every consumer masks them): unconditional loads keep
        // the register count a third of what per-load branches cost
        v[i] = *reinterpret_cast<const u32x4 *>(kb + (j < end ? j : end - 1) * stride_token + ch * 8);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int idx = tid + i * kThreads;
        ks[lds_slot<D>(idx / CH, idx % CH)] = v[i];
    }
}

// Folds one 32-key sub-tile's logits of a query row, of which `left` keys exist, into the row's running statistics.
// acc[r]: key 8*(r/4) + 4*hf + r%4 of the sub-tile.
__device__ __forceinline__ void fold_keys(const f32x16 &acc, int64_t left, int hf, float c, float &m, float &l)
{
    if (left >= 32) {
        float tm = acc[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) tm = fmaxf(tm, acc[r]);
        const float mn = fmaxf(m, tm);
        l *= fast_exp2((m - mn) * c);
        m = mn;
        const float mc = mn * c;
        float sum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) sum += fast_exp2(fmaf(acc[r], c, -mc));
        l += sum;
    } else if (left > 0) {
        float tm = neg_inf();
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int key = 8 * (r >> 2) + 4 * hf + (r & 3);
            if (key < left) tm = fmaxf(tm, acc[r]);
        }
        if (tm > neg_inf()) {
            const float mn = fmaxf(m, tm);
            l *= fast_exp2((m - mn) * c);
            m = mn;
            const float mc = mn * c;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = 8 * (r >> 2) + 4 * hf + (r & 3);
                if (key < left) l += fast_exp2(fmaf(acc[r], c, -mc));
            }
        }
    }
}

// ---------------------------------------------------------------------------
// stats: partial (max, sum exp) of every query row of one (layer, kv head)
// over one key tile.
// ---------------------------------------------------------------------------
template <int D, int NS, bool FP8>
__global__ __launch_bounds__(kThreads, 4) void sp_stats_kernel(ScoreArgs a, LayerPtrs kp)
{
    constexpr int KS = D / 16;
    constexpr int TILE = kWaves * NS * 32;
    extern __shared__ u32x4 lds[];
    u32x4 *ks = lds;                         // TILE rows
    u32x4 *qs = lds + TILE * (D / 8);        // rows_pad rows
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, hf = lane >> 5, col = lane & 31;
    const int tile = blockIdx.x, phase = blockIdx.y;
    const int layer = phase / a.n_kv_heads, kv = phase - layer * a.n_kv_heads;
    const TileInfo ti = get_tile(a, tile, TILE);
    if (tile == 0 && phase == 0 && tid == 0) *a.status = 0u;

    stage_q<D>(qs, a, ti.prompt, layer, kv, tid);
    if (FP8) stage_k_fp8<D, NS>(ks, key_base_fp8(a, kp, layer, kv), a.k_stride_token, ti.j0, ti.end, tid);
    else stage_k<D, NS, kStageGeneral>(ks, key_base(a, kp, layer, kv, ti), a.k_stride_token, ti.j0, ti.end, tid);
    __syncthreads();

    bf16x8 kf[NS][KS];
#pragma unroll
    for (int s = 0; s < NS; ++s) load_frag<D>(ks, (wave * NS + s) * 32 + col, hf, kf[s]);
    __syncthreads();                         // ks is reused for the per-wave statistics below
    float2 *wstats = reinterpret_cast<float2 *>(ks);   // [kWaves][rows_pad]

    // statistics are kept in units of the raw dot product with the stored keys; with 8-bit keys the
    // (layer, kv head)'s scale joins the logit scale
    const float c = FP8 ? a.c * a.kscale[phase] : a.c;
    const int n_blk = a.rows_pad >> 5;
    for (int blk = 0; blk < n_blk; ++blk) {
        bf16x8 qf[KS];
        load_frag<D>(qs, blk * 32 + col, hf, qf);
        float m = neg_inf(), l = 0.f;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            f32x16 acc = {0.f};
#pragma unroll
            for (int t = 0; t < KS; ++t) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s][t], qf[t], acc, 0, 0, 0);
            // acc[r]: key (wave*NS+s)*32 + 8*(r/4) + 4*hf + r%4 of the tile, query row blk*32 + col
            fold_keys(acc, ti.end - (ti.j0 + (wave * NS + s) * 32), hf, c, m, l);
        }
        const float m2 = __shfl_xor(m, 32), l2 = __shfl_xor(l, 32);
        lse_merge(m, l, m2, l2, c);
        if (hf == 0) wstats[wave * a.rows_pad + blk * 32 + col] = make_float2(m, l);
    }
    __syncthreads();
    for (int row = tid; row < a.rows_pad; row += kThreads) {
        float2 s0 = wstats[row];
        float m = s0.x, l = s0.y;
#pragma unroll
        for (int w = 1; w < kWaves; ++w) {
            const float2 sw = wstats[w * a.rows_pad + row];
            lse_merge(m, l, sw.x, sw.y, c);
        }
        a.part[((int64_t)phase * a.n_tiles + tile) * a.rows_pad + row] = make_float2(m, l);
    }
}

// ---------------------------------------------------------------------------
// merge: one workgroup per (32-row block, phase, prompt). 8 slices of the
// prompt's tiles are reduced by 32 thread groups, then combined in slice order.
// Writes -lse in raw-logit units, i.e. -(m + log2(l)/c), at the position the
// prob pass reads it from: within a block, row rho = 8*q + 4*hf + e goes to
// hf*16 + 4*q + e. Padding rows get -inf so they never win a maximum.
// ---------------------------------------------------------------------------
// -lse of a row from its statistics over all keys of its prompt.
__device__ __forceinline__ float row_normaliser(const ScoreArgs &a, int phase, int row, float m, float l, float c, float inv_c)
{
    int g, n;
    const bool valid = row_to_gn(a, row, g, n) && l > 0.f;
    float v = valid ? -(m + fast_log2(l) * inv_c) : neg_inf();
    if (valid && a.look != nullptr) {
        // the softmax also runs over the row's visible lookahead keys: log-sum-exp of both parts
        const float lp = -v, lk = a.look[(int64_t)phase * a.rows_pad + row], top = fmaxf(lp, lk);
        v = -(top + fast_log2(fast_exp2((lp - top) * a.c) + fast_exp2((lk - top) * a.c)) * a.inv_c);
    }
    return v;
}

// Where the prob pass reads row rho of a block from.
__device__ __forceinline__ int seed_pos(int rho) { return ((rho >> 2) & 1) * 16 + 4 * (rho >> 3) + (rho & 3); }

constexpr int kMergeSlices = 32;             // thread groups of 32 rows that share a prompt's tiles
constexpr int kMergeThreads = 32 * kMergeSlices;

__global__ __launch_bounds__(kMergeThreads) void sp_merge_kernel(ScoreArgs a)
{
    __shared__ float2 red[kMergeSlices][32];
    const int tid = threadIdx.x, rho = tid & 31, slice = tid >> 5;
    const int blk = blockIdx.x, phase = blockIdx.y, prompt = blockIdx.z;
    const int n_phases = a.n_layers * a.n_kv_heads;
    int t0 = 0, t1 = a.n_tiles;
    if (a.prompt_tiles) { t0 = a.prompt_tiles[prompt]; t1 = a.prompt_tiles[prompt + 1]; }
    const int row = blk * 32 + rho;
    const float c = a.kscale ? a.c * a.kscale[phase] : a.c;      // the phase's logit scale (8-bit keys carry their own)
    const float inv_c = a.kscale ? 1.0f / c : a.inv_c;
    float m = neg_inf(), l = 0.f;
    for (int t = t0 + slice; t < t1; t += kMergeSlices) {
        const float2 p = a.part[((int64_t)phase * a.n_tiles + t) * a.rows_pad + row];
        lse_merge(m, l, p.x, p.y, c);
    }
    red[slice][rho] = make_float2(m, l);
    __syncthreads();
    if (slice == 0) {
#pragma unroll
        for (int s = 1; s < kMergeSlices; ++s) lse_merge(m, l, red[s][rho].x, red[s][rho].y, c);
        const float v = row_normaliser(a, phase, row, m, l, c, inv_c);
        a.lse_neg[((int64_t)prompt * n_phases + phase) * a.rows_pad + blk * 32 + seed_pos(rho)] = v;
    }
}

// ---------------------------------------------------------------------------
// look: log-sum-exp (raw-logit units) of every query row over the lookahead
// keys it sees, one workgroup per (layer, kv head). Lookahead row n sees the
// keys of rows 0 .. n-1, and its own with look_self (a decode step attends to the
// tokens generated before it; Algorithm 1's ForwardWithAttn with lookahead = i).
// Rows that see none get -inf. k_look is dense [Lyr][Hkv][n_q][d].
// Bound by the latency of its loads (a few KB a workgroup): one thread per
// (row, key) pair, so that all of a workgroup's logits are one round of 16-byte
// loads; one thread per row walking its keys element by element took 46 us
// for 128 workgroups of 32 rows and 8 keys. Ahead of the single-launch kernel it also clears what that exchanges
// (clear_n words and the status word), one launch less (12007 tokens 79.3 -> 78.1 us).
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(kThreads) void sp_look_kernel(ScoreArgs a, const uint16_t *__restrict__ k_look,
                                                           int look_self, float *__restrict__ out, uint64_t *__restrict__ clear,
                                                           size_t clear_n, uint32_t *__restrict__ status)
{
    if (status != nullptr && blockIdx.x == 0 && threadIdx.x == 0) *status = 0u;
    for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < clear_n; i += (size_t)gridDim.x * kThreads) clear[i] = 0;
    if ((int)blockIdx.x >= a.n_layers * a.n_kv_heads) return;      // launched to clear only
    __shared__ float logit[kMaxLookRows][17];                    // [padded row][key], odd stride: no bank conflicts down a row
    const int phase = blockIdx.x;
    const int layer = phase / a.n_kv_heads, kv = phase - layer * a.n_kv_heads;
    const uint16_t *kb = k_look + ((int64_t)layer * a.n_kv_heads + kv) * a.n_q * D;
    for (int i = threadIdx.x; i < a.rows_pad * 16; i += kThreads) {
        const int row = i >> 4, j = i & 15;
        int g, n;
        if (!row_to_gn(a, row, g, n) || j >= min(n + (look_self ? 1 : 0), a.n_q)) continue;
        const u32x4 *qr = reinterpret_cast<const u32x4 *>(
            a.q + (((int64_t)layer * a.n_q_heads + (int64_t)kv * a.group + g) * a.n_q + n) * D);
        const u32x4 *kr = reinterpret_cast<const u32x4 *>(kb + j * D);
        float dot = 0.f;
#pragma unroll
        for (int c = 0; c < D / 8; ++c) {
            const u32x4 x = qr[c], y = kr[c];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                dot = fmaf(__uint_as_float(x[e] << 16), __uint_as_float(y[e] << 16), dot);
                dot = fmaf(__uint_as_float(x[e] & 0xffff0000u), __uint_as_float(y[e] & 0xffff0000u), dot);
            }
        }
        logit[row][j] = dot;
    }
    __syncthreads();
    const int row = threadIdx.x;
    if (row >= a.rows_pad) return;
    int g, n;
    float v = neg_inf();
    if (row_to_gn(a, row, g, n)) {
        const int n_vis = min(n + (look_self ? 1 : 0), a.n_q);
        float m = neg_inf(), l = 0.f;
        for (int j = 0; j < n_vis; ++j) lse_merge(m, l, logit[row][j], 1.f, a.c);
        if (l > 0.f) v = m + fast_log2(l) * a.inv_c;
    }
    out[(int64_t)phase * a.rows_pad + row] = v;
}

// ---------------------------------------------------------------------------
// prob: per key, sum over lookahead rows (and layers) of the head-maximum of
// the attention probability.
// ---------------------------------------------------------------------------
// Logits less the normalisers of one (layer, kv head)'s rows over this wave's keys, folded into the maxima over heads.
template <int D, int NS, int NB, bool FP8>
__device__ __forceinline__ void fold_heads(const u32x4 *qs, const float *ci, const bf16x8 (&kf)[NS][D / 16], int n_gblk, int col, int hf,
                                           float ksc, float (&mx)[NS][NB][4])
{
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        for (int gb = 0; gb < n_gblk; ++gb) {
            const int blk = gb * NB + nb;
            bf16x8 qf[D / 16];
            load_frag<D>(qs, blk * 32 + col, hf, qf);
            f32x16 cinit;
            const float4 *cp = reinterpret_cast<const float4 *>(ci + blk * 32 + hf * 16);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float4 x = cp[v];
                cinit[4 * v + 0] = x.x; cinit[4 * v + 1] = x.y;
                cinit[4 * v + 2] = x.z; cinit[4 * v + 3] = x.w;
            }
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                f32x16 acc = cinit;
#pragma unroll
                for (int t = 0; t < D / 16; ++t)
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[t], kf[s][t], acc, 0, 0, 0);
                // acc[r]: group head r/4, lookahead row 8*nb + 4*hf + r%4, key (wave*NS+s)*32 + col
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float v = fmaxf(fmaxf(acc[e], acc[4 + e]), fmaxf(acc[8 + e], acc[12 + e]));
                    mx[s][nb][e] = fmaxf(mx[s][nb][e], FP8 ? v * ksc : v);
                }
            }
        }
    }
}

// Sum of the probabilities of one key's row maxima, which start over.
template <int NB>
__device__ __forceinline__ float close_rows(float (&mx)[NB][4], float c)
{
    float sum = 0.f;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            sum += fast_exp2(mx[b][e] * c);
            mx[b][e] = neg_inf();
        }
    return sum;
}

// The merge of a short prompt, by every workgroup of the prob pass for the phases of its own layers: one thread per
// (phase, row) walks the prompt's tiles, eight partials in flight. `out`: [phases][rows_pad], permuted as in lse_neg.
__device__ __forceinline__ void merge_rows(const ScoreArgs &a, const TileInfo &ti, int phase0, int phases, float *out, int tid)
{
    const int t0 = a.prompt_tiles ? a.prompt_tiles[ti.prompt] : 0, t1 = a.prompt_tiles ? a.prompt_tiles[ti.prompt + 1] : a.n_tiles;
    for (int i = tid; i < phases * a.rows_pad; i += kThreads) {
        const int ph = i / a.rows_pad, row = i - ph * a.rows_pad, phase = phase0 + ph;
        const float c = a.kscale ? a.c * a.kscale[phase] : a.c;
        const float2 *src = a.part + (int64_t)phase * a.n_tiles * a.rows_pad + row;
        float m = neg_inf(), l = 0.f;
        for (int t = t0; t < t1; t += 8) {
            float2 p[8];
            float mm = m;
#pragma unroll
            for (int u = 0; u < 8; ++u) p[u] = t + u < t1 ? src[(int64_t)(t + u) * a.rows_pad] : make_float2(neg_inf(), 0.f);
#pragma unroll
            for (int u = 0; u < 8; ++u) mm = fmaxf(mm, p[u].x);
            if (mm == neg_inf()) continue;
            l *= fast_exp2((m - mm) * c);
#pragma unroll
            for (int u = 0; u < 8; ++u) l += p[u].y * fast_exp2((p[u].x - mm) * c);
            m = mm;
        }
        out[ph * a.rows_pad + (row & ~31) + seed_pos(row & 31)] = row_normaliser(a, phase, row, m, l, c, a.kscale ? 1.0f / c : a.inv_c);
    }
}

// MERGE: see prob_merges. A template argument: as a run-time branch it cost the long prompts, which never take it, 1.5 %
// (170000 paged tokens, 16 lookahead rows 1174 -> 1191 us; spilled scalar registers in the loop).
template <int D, int NS, int NB, bool FP8, bool MERGE>
__global__ __launch_bounds__(kThreads, 3) void sp_prob_kernel(ScoreArgs a, LayerPtrs kp)
{
    constexpr int KS = D / 16;
    constexpr int TILE = kWaves * NS * 32;
    extern __shared__ u32x4 lds[];
    u32x4 *ks = lds;
    u32x4 *qs = lds + TILE * (D / 8);
    float *ci0 = reinterpret_cast<float *>(qs + a.rows_pad * (D / 8));   // rows_pad floats, or as many for every phase
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, hf = lane >> 5, col = lane & 31;
    const int tile = blockIdx.x, split = blockIdx.y;
    const TileInfo ti = get_tile(a, tile, TILE);
    const int n_phases = a.n_layers * a.n_kv_heads;
    const float c = a.c;
    const int layer_lo = split * a.layers_per_split;
    const int layer_hi = min(layer_lo + a.layers_per_split, a.n_layers);
    const bool whole = a.n_splits == 1;

    float mx[NS][NB][4];
    float total[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        total[s] = 0.f;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) mx[s][b][e] = neg_inf();
    }

    if (MERGE) merge_rows(a, ti, layer_lo * a.n_kv_heads, (layer_hi - layer_lo) * a.n_kv_heads, ci0, tid);
    for (int layer = layer_lo; layer < layer_hi; ++layer) {
        for (int kv = 0; kv < a.n_kv_heads; ++kv) {
            const int phase = layer * a.n_kv_heads + kv;
            float *ci = ci0 + (MERGE ? (phase - layer_lo * a.n_kv_heads) * a.rows_pad : 0);
            __syncthreads();
            stage_q<D>(qs, a, ti.prompt, layer, kv, tid);
            if (FP8) stage_k_fp8<D, NS>(ks, key_base_fp8(a, kp, layer, kv), a.k_stride_token, ti.j0, ti.end, tid);
            else stage_k<D, NS, kStageGeneral>(ks, key_base(a, kp, layer, kv, ti), a.k_stride_token, ti.j0, ti.end, tid);
            // 8-bit keys: logit differences of this (layer, kv head) are in units of its stored keys; its scale
            // brings them to the common unit before they meet those of other heads and layers
            const float ksc = FP8 ? a.kscale[phase] : 1.0f;
            if (!MERGE)
                for (int i = tid; i < a.rows_pad; i += kThreads)
                    ci[i] = a.lse_neg[((int64_t)ti.prompt * n_phases + phase) * a.rows_pad + i];
            __syncthreads();

            bf16x8 kf[NS][KS];
#pragma unroll
            for (int s = 0; s < NS; ++s) load_frag<D>(ks, (wave * NS + s) * 32 + col, hf, kf[s]);

            fold_heads<D, NS, NB, FP8>(qs, ci, kf, a.n_gblk, col, hf, ksc, mx);
        }
        if (a.layer_agg == SP_LAYER_MEAN || (whole && layer == a.n_layers - 1)) {
#pragma unroll
            for (int s = 0; s < NS; ++s) total[s] += close_rows<NB>(mx[s], c);
        }
    }
    if (!whole && a.layer_agg == SP_LAYER_MAX) {
        // probabilities of this layer range's head-and-layer maxima, one per (lookahead row, key);
        // exp is monotone, so the maximum over ranges can be taken after it
        const int n_rows = 8 * NB;
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int n = 8 * b + 4 * hf + e;
                    const int64_t j = ti.j0 + (wave * NS + s) * 32 + col;
                    if (j < ti.end) a.split_buf[((int64_t)split * n_rows + n) * a.L + j] = fast_exp2(mx[s][b][e] * c);
                }
        return;
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const float both = total[s] + __shfl_xor(total[s], 32);
        const int local = (wave * NS + s) * 32 + col;
        const int64_t j = ti.j0 + local;
        if (hf != 0) continue;
        if (j >= ti.end) continue;
        if (!whole) a.split_buf[split * a.L + j] = both;
        else a.scores[j] = both * a.out_scale;
    }
}

// ---------------------------------------------------------------------------
// reduce: combines the layer ranges of a call, whichever kernel left them. MEAN
// adds the ranges' sums; MAX takes, per lookahead row, the largest probability
// over the ranges and adds the rows. A workgroup owns 64 keys; its four waves
// take every fourth range (MEAN) or row (MAX), so that a short prompt still has
// enough loads in flight, and their sums are added in wave order.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float reduce_ranges(const float *__restrict__ buf, int64_t total, int n_splits, int n_rows /* 0: MEAN */)
{
    __shared__ float part[4][64];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t j = (int64_t)blockIdx.x * 64 + lane;
    const float *src = buf + (j < total ? j : 0);
    float sum = 0.f;
    if (n_rows == 0) {
#pragma unroll 4
        for (int s = wave; s < n_splits; s += 4) sum += src[s * total];
    } else {
        for (int n = wave; n < n_rows; n += 4) {
            float m = 0.f;
#pragma unroll 8
            for (int s = 0; s < n_splits; ++s) m = fmaxf(m, src[((int64_t)s * n_rows + n) * total]);
            sum += m;
        }
    }
    part[wave][lane] = sum;
    __syncthreads();
    return (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
}

__global__ __launch_bounds__(256) void sp_split_reduce_kernel(const float *__restrict__ buf, int64_t total, int n_splits,
                                                              int n_rows, float out_scale,
                                                              const uint32_t *__restrict__ status,
                                                              float *__restrict__ scores)
{
    const float both = reduce_ranges(buf, total, n_splits, n_rows);
    const int64_t j = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (threadIdx.x >= 64 || j >= total) return;
    scores[j] = *status != 0u ? __uint_as_float(0x7fc00000u) : both * out_scale;     // a failed call has no scores
}

// ---------------------------------------------------------------------------
// finish: last launch of a call that took the single-launch kernel although
// sp_score_is_fused does not say so. Such a call never fails: as a rule this
// launch adds up the layer ranges (n_ranges > 1) or has nothing to do, but where
// the single-launch kernel gave up (other work held compute units its workgroups
// wait for) it computes the scores afresh, in workgroups that need none of each
// other: every one finds all rows' normalisers by itself, reading its prompt's
// keys of a (layer, kv head) once, before the probabilities of its own tile. That
// reads K once per tile instead of twice in all; with the wait before it, a call
// that comes here takes tens of milliseconds.
// ---------------------------------------------------------------------------
__device__ __forceinline__ TileInfo find_tile(const ScoreArgs &a, const int64_t *offsets, int tile, int tile_keys)
{
    TileInfo t = get_tile(a, tile, tile_keys);
    if (offsets == nullptr) return t;
    int64_t first = 0;
    for (int p = 0; p < a.n_prompts; ++p) {
        const int64_t beg = offsets[p], end = offsets[p + 1], n = (end - beg + tile_keys - 1) / tile_keys;
        if (tile < first + n) {
            t.j0 = beg + (tile - first) * tile_keys;
            t.end = end; t.prompt = p; t.first_tile = (int32_t)first;
            break;
        }
        first += n;
    }
    return t;
}

size_t finish_lds_bytes(int tile_keys, int D, int rows_pad)
{
    return (size_t)(tile_keys + rows_pad) * D * 2 + (size_t)rows_pad * (2 * kWaves * sizeof(float2) + sizeof(float));
}

template <int D, int NS, int NB, bool FP8>
__global__ __launch_bounds__(kThreads) void sp_finish_kernel(ScoreArgs a, LayerPtrs kp, const int64_t *__restrict__ offsets,
                                                             const uint32_t *__restrict__ gave_up, int n_ranges)
{
    constexpr int KS = D / 16;
    constexpr int TILE = kWaves * NS * 32;
    extern __shared__ u32x4 lds[];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, hf = lane >> 5, col = lane & 31;
    if (blockIdx.x == 0 && tid == 0) *a.status = 0u;
    float both = 0.f;
    if (n_ranges > 1) both = reduce_ranges(a.split_buf, a.L, n_ranges, a.layer_agg == SP_LAYER_MAX ? 8 * NB : 0);
    if (*gave_up == 0u) {
        const int64_t j = (int64_t)blockIdx.x * 64 + tid;
        if (n_ranges > 1 && tid < 64 && j < a.L) a.scores[j] = both * a.out_scale;
        return;
    }
    u32x4 *ks = lds;
    u32x4 *qs = lds + TILE * (D / 8);
    float2 *st = reinterpret_cast<float2 *>(qs + a.rows_pad * (D / 8));        // [wave][half of the wave][row]
    float *ci = reinterpret_cast<float *>(st + 2 * kWaves * a.rows_pad);
    for (int tile = blockIdx.x; tile < a.n_tiles; tile += gridDim.x) {
        const TileInfo mine = find_tile(a, offsets, tile, TILE);
        TileInfo ti = mine;
        auto stage = [&](int layer, int kv) {
            if (FP8) stage_k_fp8<D, NS>(ks, key_base_fp8(a, kp, layer, kv), a.k_stride_token, ti.j0, ti.end, tid);
            else stage_k<D, NS, kStageFinish>(ks, key_base(a, kp, layer, kv, ti), a.k_stride_token, ti.j0, ti.end, tid);
        };
        bf16x8 kf[NS][KS];
        float mx[NS][NB][4], total[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            total[s] = 0.f;
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e) mx[s][b][e] = neg_inf();
        }
        for (int layer = 0; layer < a.n_layers; ++layer) {
            for (int kv = 0; kv < a.n_kv_heads; ++kv) {
                const int phase = layer * a.n_kv_heads + kv;
                const float ksc = FP8 ? a.kscale[phase] : 1.0f, c = a.c * ksc;
                __syncthreads();
                stage_q<D>(qs, a, mine.prompt, layer, kv, tid);
                for (int i = tid; i < 2 * kWaves * a.rows_pad; i += kThreads) st[i] = make_float2(neg_inf(), 0.f);
                for (ti.j0 = mine.j0 - (int64_t)(tile - mine.first_tile) * TILE; ti.j0 < mine.end; ti.j0 += TILE) {
                    __syncthreads();
                    stage(layer, kv);
                    __syncthreads();
#pragma unroll
                    for (int s = 0; s < NS; ++s) load_frag<D>(ks, (wave * NS + s) * 32 + col, hf, kf[s]);
                    for (int blk = 0; blk < a.rows_pad >> 5; ++blk) {
                        bf16x8 qf[KS];
                        load_frag<D>(qs, blk * 32 + col, hf, qf);
                        float2 &slot = st[(wave * 2 + hf) * a.rows_pad + blk * 32 + col];
                        float m = slot.x, l = slot.y;
#pragma unroll
                        for (int s = 0; s < NS; ++s) {
                            f32x16 acc = {0.f};
#pragma unroll
                            for (int t = 0; t < KS; ++t) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s][t], qf[t], acc, 0, 0, 0);
                            fold_keys(acc, ti.end - (ti.j0 + (wave * NS + s) * 32), hf, c, m, l);
                        }
                        slot = make_float2(m, l);
                    }
                }
                ti.j0 = mine.j0;
                __syncthreads();
                stage(layer, kv);
                for (int row = tid; row < a.rows_pad; row += kThreads) {
                    float m = neg_inf(), l = 0.f;
                    for (int i = 0; i < 2 * kWaves; ++i) lse_merge(m, l, st[i * a.rows_pad + row].x, st[i * a.rows_pad + row].y, c);
                    ci[(row & ~31) + seed_pos(row & 31)] = row_normaliser(a, phase, row, m, l, c, FP8 ? 1.0f / c : a.inv_c);
                }
                __syncthreads();
#pragma unroll
                for (int s = 0; s < NS; ++s) load_frag<D>(ks, (wave * NS + s) * 32 + col, hf, kf[s]);
                fold_heads<D, NS, NB, FP8>(qs, ci, kf, a.n_gblk, col, hf, ksc, mx);
            }
            if (a.layer_agg == SP_LAYER_MEAN || layer == a.n_layers - 1) {
#pragma unroll
                for (int s = 0; s < NS; ++s) total[s] += close_rows<NB>(mx[s], a.c);
            }
        }
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const float sum = total[s] + __shfl_xor(total[s], 32);
            const int64_t j = mine.j0 + (wave * NS + s) * 32 + col;
            if (hf == 0 && j < mine.end) a.scores[j] = sum * a.out_scale;
        }
    }
}

// Last launch of a batch of several prompts: a call fails as a whole, and a prompt whose waits gave up may follow one that
// has left valid scores, in an earlier launch or in the same one (a prompt whose duties all sit in workgroups that
// are there does not wait for the others' at its end).
__global__ __launch_bounds__(256) void sp_fail_all_kernel(const uint32_t *__restrict__ status, int64_t total, float *__restrict__ scores)
{
    if (*status == 0u) return;
    for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < total; j += (int64_t)gridDim.x * 256) scores[j] = __uint_as_float(0x7fc00000u);
}

// Tile table of a ragged batch: tiles never straddle prompts.
__global__ void sp_tiles_kernel(const int64_t *offsets, int n_prompts, int tile_keys, TileInfo *tiles,
                                int32_t *prompt_tiles, int n_tiles_cap)
{
    for (int b = threadIdx.x; b <= n_prompts; b += blockDim.x) {
        int64_t first = 0;
        for (int p = 0; p < b; ++p) first += (offsets[p + 1] - offsets[p] + tile_keys - 1) / tile_keys;
        prompt_tiles[b] = (int32_t)first;
        if (b == n_prompts) continue;
        const int64_t beg = offsets[b], end = offsets[b + 1];
        int64_t t = first;
        for (int64_t j = beg; j < end && t < n_tiles_cap; j += tile_keys, ++t) {
            TileInfo ti;
            ti.j0 = j; ti.end = end; ti.prompt = b; ti.first_tile = (int32_t)first;
            tiles[t] = ti;
        }
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
int prob_splits(const Plan &p, int64_t n_tiles)
{
    const int lps = prob_layers_per_split(p, n_tiles);
    return (p.n_layers + lps - 1) / lps;
}

// Floats of the layer-split buffer, bounded over every tile count up to n_tiles (the workspace query
// rounds the tile count up): splits * tiles never exceeds either term of the minimum.
size_t split_buf_floats(const Plan &p, int64_t n_tiles)
{
    int64_t blocks = (int64_t)p.n_layers * n_tiles;
    if (blocks > kProbTargetWgs + n_tiles) blocks = kProbTargetWgs + n_tiles;
    const int per_key = (p.layer_agg == SP_LAYER_MAX) ? 8 * p.NB : 1;
    return (size_t)blocks * p.tile_keys * per_key;
}

sp_status make_plan(const sp_score_desc *d, Plan &p)
{
    if (!d) return sp::fail(SP_ERR_INVALID_ARG, "desc is null");
    if (d->n_layers < 1 || d->n_q_heads < 1 || d->n_kv_heads < 1 || d->n_q < 1 || d->head_dim < 1)
        return sp::fail(SP_ERR_INVALID_ARG, "desc: sizes must be positive");
    if (d->n_q_heads % d->n_kv_heads != 0)
        return sp::fail(SP_ERR_INVALID_ARG, "desc: n_q_heads (%d) is not a multiple of n_kv_heads (%d)",
                        d->n_q_heads, d->n_kv_heads);
    if (!(d->scale > 0.f) || !std::isfinite(d->scale))
        return sp::fail(SP_ERR_INVALID_ARG, "desc: scale must be finite and > 0");
    if (d->layer_agg != SP_LAYER_MEAN && d->layer_agg != SP_LAYER_MAX)
        return sp::fail(SP_ERR_INVALID_ARG, "desc: layer_agg must be SP_LAYER_MEAN or SP_LAYER_MAX");
    if (d->head_dim != 64 && d->head_dim != 128)
        return sp::fail(SP_ERR_UNSUPPORTED, "desc: head_dim %d (supported: 64, 128)", d->head_dim);
    if (d->n_q > 16) return sp::fail(SP_ERR_UNSUPPORTED, "desc: n_q %d (supported: 1..16)", d->n_q);
    if (d->n_layers > kMaxLayers)
        return sp::fail(SP_ERR_UNSUPPORTED, "desc: n_layers %d (supported: <= %d)", d->n_layers, kMaxLayers);
    const int G = d->n_q_heads / d->n_kv_heads;
    if (G > 16) return sp::fail(SP_ERR_UNSUPPORTED, "desc: %d query heads per kv head (supported: <= 16)", G);
    if (d->k_stride_token < d->head_dim || d->k_stride_head < 0 || d->k_stride_token % 8 != 0 ||
        d->k_stride_head % 8 != 0)
        return sp::fail(SP_ERR_INVALID_ARG, "desc: K strides must be multiples of 8 elements, token stride >= head_dim");
    p.D = d->head_dim;
    p.NS = (p.D == 64) ? 2 : 1;
    p.NB = (d->n_q + 7) / 8;
    p.n_gblk = (G + 3) / 4;
    p.rows_pad = p.NB * p.n_gblk * 32;
    p.tile_keys = kWaves * p.NS * 32;
    p.n_phases = d->n_layers * d->n_kv_heads;
    if (p.n_phases > 65535)
        return sp::fail(SP_ERR_UNSUPPORTED, "desc: %d (layer, kv head) pairs (supported: <= 65535)", p.n_phases);
    p.n_layers = d->n_layers;
    p.layer_agg = d->layer_agg;
    p.lds_bytes = (size_t)p.tile_keys * p.D * 2 + (size_t)p.rows_pad * p.D * 2 + (size_t)p.rows_pad * 4;
    if (p.lds_bytes > kLdsBudget)
        return sp::fail(SP_ERR_UNSUPPORTED, "desc: query group of %d heads x %d rows at head_dim %d exceeds on-chip staging",
                        G, d->n_q, p.D);
    return SP_OK;
}

struct WsLayout {
    size_t status, part, lse, tiles, prompt_tiles, split, look, fused, total;
};

// Shapes the fused single-launch kernel can hold on chip (any L; the length test is separate).
bool fused_shape_ok(const Plan &p)
{
    return p.D == 64 ? p.rows_pad <= sp_fused::kMaxRows : p.rows_pad <= sp_fused::kMaxRowsWide || fused_big(p);
}

// The shapes sp_score_is_fused speaks of and the workspace reserves an exchange area for.
bool fused_base_shape(const Plan &p) { return fused_shape_ok(p) && !fused_big(p); }

// The fewest workgroups the fused kernel is used with, all layers in one range.
int fused_min_workgroups(const Plan &p) { return p.D == 64 ? sp_fused::kMinWorkgroups : sp_fused::kMinWorkgroupsWide; }

int fused_workgroups(const Plan &p, int64_t L)
{
    const int64_t n = sp::ceil_div(L, fused_tile(p));
    return n > 0x7fffffff ? 0x7fffffff : (int)n;
}

// Compute units of the current device (0 if it cannot be queried); the fused kernel needs one per workgroup.
int device_compute_units()
{
    static thread_local int cached_dev = -1, cached_cus = 0;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (dev != cached_dev) {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 0;
        if (cus > 0 && !sp_fused::fits_one_per_cu()) cus = 0;
        cached_dev = dev;
        cached_cus = cus;
    }
    return cached_cus;
}

// The fused kernel runs one workgroup of 512 keys per compute unit: long single prompts only.
bool fused_applies(const Plan &p, int64_t L, int64_t k_stride_token)
{
    if (!fused_base_shape(p)) return false;
    if (k_stride_token > (int64_t(1) << 20)) return false;       // lane offsets within a tile are 32-bit
    const int n_wg = fused_workgroups(p, L);
    return n_wg >= fused_min_workgroups(p) && n_wg <= 256 && n_wg <= device_compute_units();
}

// Prompts that need more than one tile per compute unit, and no more than two: K is still read once (16 layers
// x 8 kv heads, head_dim 64: 256K tokens 781 us against 1514 on the three-kernel path, one token beyond 128K 523 against
// 756; 64 rows, 140000 744 against 940). 8-bit keys at head_dim 64 leave the three kernels half the bytes; their line lies
// an eighth later, where the kernels crossed when it was drawn (140000 tokens 621 / 676, 200000 651 / 935; 64 rows
// 140000 802 / 850: the present kernel is ahead from the first token beyond a tile a unit on). With 64 padded rows (whole passes, three
// kernels / this one): 16 lookahead rows 131600 901 / 758, 200000 1368 / 853, 262144 1800 / 1033, paged 200000 1515 / 1001, 8-bit keys
// 150000 878 / 805, 262144 1591 / 884; 24 x 4 heads of 128, eight query heads each, 66000 812 / 600, 131072 1587 / 905.
bool pair_applies(const Plan &p, bool fp8, int64_t L, int64_t k_stride_token)
{
    if (!fused_shape_ok(p) || k_stride_token > (int64_t(1) << 20)) return false;
    const int cus = std::min(256, device_compute_units());
    const int64_t tiles = sp::ceil_div(L, fused_tile(p));
    return cus >= 128 && tiles > (fp8 && p.D == 64 ? cus + cus / 8 : cus) && tiles <= 2 * (int64_t)cus;
}

// 8-bit keys: the single-launch kernel's variants for them fetch the codes in 16-byte pieces (strides in
// multiples of 16 elements).
bool fp8_strides_ok(const sp_score_desc *desc) { return desc->k_stride_token % 16 == 0 && desc->k_stride_head % 16 == 0; }

bool fused_applies_fp8(const Plan &p, const sp_score_desc *desc, int64_t L)
{
    return fp8_strides_ok(desc) && fused_applies(p, L, desc->k_stride_token);
}

bool duties_shared(const Plan &p, const BatchGroups &bg, size_t g)
{
    return !bg.short_prompt && bg.groups[g].n * (p.rows_pad / sp_fused::kDutyRows) <= bg.wgs[g];
}

// How many layer ranges a launch over all of `n_prompts` prompts is cut into: as many as its `tiles`
// workgroups fit the device, so that the ranges run side by side. `room`: bytes for their exchange area.
// A step of the kernel takes 1.8 us on 64 workgroups and 2.9 us on 256 (head_dim 64, 32 rows), so every
// range more is time saved (16 layers, 8 kv heads, head_dim 64: 32K tokens 245 -> 101 us with four
// ranges, 64K tokens 267 -> 188 us with two; 28 layers, head_dim 128: 32K tokens 445 -> 305 us, 16K tokens 398 -> 165
// with four).
int fused_ranges(const Plan &p, int tiles, int n_prompts, size_t room)
{
    int n = std::min({std::min(256, device_compute_units()) / tiles, p.n_layers, sp_fused::kMaxGroup / n_prompts});
    while (n > 1 && sp_fused::workspace_bytes(p.rows_pad, tiles * n, n_prompts * n) > room) --n;
    if (n < 2) return 1;
    return (int)sp::ceil_div(p.n_layers, sp::ceil_div(p.n_layers, n));       // no empty range
}

// A single prompt on the single-launch kernel: a table of one entry.
bool plan_fused_prompt(const Plan &p, int64_t L, int64_t k_stride_token, BatchGroups &out)
{
    if (!fused_shape_ok(p) || k_stride_token > (int64_t(1) << 20) || L < fused_tile(p)) return false;
    const int n_wg = fused_workgroups(p, L);
    if (n_wg > std::min(256, device_compute_units())) return false;
    sp_fused::GroupTable t;
    std::memset(&t, 0, sizeof t);
    t.n = 1;
    t.w0[1] = n_wg;
    t.layers[0] = p.n_layers;
    t.len[0] = (int32_t)L;
    out.groups.assign(1, t);
    out.wgs.assign(1, t.w0[1]);
    return true;
}

WsLayout ws_layout(const Plan &p, int64_t n_tiles, int n_prompts)
{
    WsLayout w;
    size_t off = 0;
    w.status = off; off += 256;           // the call's status word leads the workspace (see sp.h)
    w.part = off;  off = sp::align_up(off + sizeof(float2) * (size_t)p.n_phases * (size_t)n_tiles * p.rows_pad, 256);
    w.lse = off;   off = sp::align_up(off + sizeof(float) * (size_t)n_prompts * p.n_phases * p.rows_pad, 256);
    w.tiles = off; off = sp::align_up(off + sizeof(TileInfo) * (size_t)n_tiles, 256);
    w.prompt_tiles = off; off = sp::align_up(off + sizeof(int32_t) * (size_t)(n_prompts + 1), 256);
    w.split = off; off = sp::align_up(off + sizeof(float) * split_buf_floats(p, n_tiles), 256);
    w.look = off; off = sp::align_up(off + sizeof(float) * (size_t)p.n_phases * p.rows_pad, 256);
    w.fused = off;
    if (fused_base_shape(p)) {
        int64_t n_wg = n_tiles * p.tile_keys / fused_tile(p) + n_prompts;
        if (n_wg > 1024) n_wg = 1024;
        off += sp_fused::workspace_bytes(p.rows_pad, (int)n_wg, std::min(n_prompts, kMaxGroupPrompts));
    }
    w.total = off;
    return w;
}

// A ragged batch on the single-launch kernel. `w`: the call's workspace, which has to hold what a launch exchanges
// and the ranges' results.
bool plan_fused_batch(const Plan &p, const int64_t *offsets, int B, int64_t keys, int64_t k_stride_token, const WsLayout &w, Launches may,
                      BatchGroups &out)
{
    if (!fused_shape_ok(p) || k_stride_token > (int64_t(1) << 20)) return false;
    const Limits lim{std::min(kMaxUnits, device_compute_units()), kMaxGroupPrompts, sp_fused::kMaxGroup, w.split - w.part, w.look - w.split};
    return plan_batch(p, offsets, B, keys, lim, may, out);
}

sp_status launch_reduce(const ScoreArgs &a, int n_splits, hipStream_t st)
{
    hipLaunchKernelGGL(sp_split_reduce_kernel, dim3((unsigned)sp::ceil_div(a.L, 64)), dim3(256), 0, st, (const float *)a.split_buf,
                       a.L, n_splits, a.layer_agg == SP_LAYER_MAX ? 8 * a.n_nblk : 0, a.out_scale, (const uint32_t *)a.status, a.scores);
    SP_HIP_CHECK(hipGetLastError());
    return SP_OK;
}

template <int D, int NS, bool FP8>
sp_status launch_finish_as(const Plan &p, const ScoreArgs &a, const LayerPtrs &kp, const int64_t *offsets, const uint32_t *gave_up,
                           int n_ranges, hipStream_t st)
{
    const int64_t grid = n_ranges > 1 ? sp::ceil_div(a.L, 64) : std::min(a.n_tiles, 512);
    const auto kernel = p.NB == 1 ? sp_finish_kernel<D, NS, 1, FP8> : sp_finish_kernel<D, NS, 2, FP8>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(kThreads), finish_lds_bytes(p.tile_keys, p.D, p.rows_pad), st, a, kp, offsets,
                       gave_up, n_ranges);
    SP_HIP_CHECK(hipGetLastError());
    return SP_OK;
}

sp_status launch_finish(const Plan &p, const ScoreArgs &a, const LayerPtrs &kp, const int64_t *offsets, const uint32_t *gave_up,
                        int n_ranges, hipStream_t st)
{
    if (a.kscale) return p.D == 64 ? launch_finish_as<64, 2, true>(p, a, kp, offsets, gave_up, n_ranges, st)
                                   : launch_finish_as<128, 1, true>(p, a, kp, offsets, gave_up, n_ranges, st);
    return p.D == 64 ? launch_finish_as<64, 2, false>(p, a, kp, offsets, gave_up, n_ranges, st)
                     : launch_finish_as<128, 1, false>(p, a, kp, offsets, gave_up, n_ranges, st);
}

// Whether the prob pass merges the tiles' statistics itself (`longest`: tokens of the longest prompt): a launch less
// (3.5 us in a chain of launches, 2.5 us of the host) for up to 20 partials a thread of a workgroup on average, and up to 48
// tiles, which one thread walks for its row. Whole passes with the merge kernel and without, 16 layers x 8 kv heads, 32
// rows: 1000 tokens 40.9 / 37.3 us, 3000 48.5 / 46.3, 4500 (18 partials) 53.7 / 51.9, 8-bit keys 6000 (24) 52.9 / 53.8; 64
// rows: 2000 (16) 51.6 / 49.0, 4500 (36) 62.7 / 63.3; 2 layers x 2 kv heads, 1024 tokens 30.3 / 26.7. Score calls of few
// phases (fewer rows than threads): 2 x 2, 48 tiles 17.7 / 16.7, 80 19.7 / 19.9; 1 x 1, 64 rows, 48 15.2 / 14.5, 56 14.7 /
// 15.0, 80 15.4 / 16.3; 2 x 1, head_dim 128, 48 18.8 / 17.2, 80 18.9 / 19.4.
bool prob_merges(const Plan &p, const ScoreArgs &a, int64_t longest)
{
    const int64_t rows = (int64_t)a.layers_per_split * a.n_kv_heads * p.rows_pad;        // of a workgroup, over all its phases
    const int64_t tiles = sp::ceil_div(longest, p.tile_keys);
    return p.lds_bytes + sizeof(float) * (size_t)(rows - p.rows_pad) <= kLdsBudget && tiles <= 48 && rows * tiles <= 20 * kThreads;
}

template <int D, int NS, bool FP8 = false>
sp_status launch_all(const Plan &p, const ScoreArgs &a, const LayerPtrs &kp, int64_t longest, hipStream_t st)
{
    const dim3 block(kThreads);
    hipLaunchKernelGGL((sp_stats_kernel<D, NS, FP8>), dim3(a.n_tiles, p.n_phases), block, p.lds_bytes, st, a, kp);
    SP_HIP_CHECK(hipGetLastError());
    const dim3 grid(a.n_tiles, a.n_splits);
    if (prob_merges(p, a, longest)) {
        const size_t lds = p.lds_bytes + sizeof(float) * (size_t)p.rows_pad * (a.layers_per_split * a.n_kv_heads - 1);
        hipLaunchKernelGGL(p.NB == 1 ? (sp_prob_kernel<D, NS, 1, FP8, true>) : (sp_prob_kernel<D, NS, 2, FP8, true>), grid, block, lds, st, a, kp);
    } else {
        hipLaunchKernelGGL(sp_merge_kernel, dim3(p.rows_pad / 32, p.n_phases, a.n_prompts), dim3(kMergeThreads), 0, st, a);
        SP_HIP_CHECK(hipGetLastError());
        hipLaunchKernelGGL(p.NB == 1 ? (sp_prob_kernel<D, NS, 1, FP8, false>) : (sp_prob_kernel<D, NS, 2, FP8, false>), grid, block, p.lds_bytes, st, a, kp);
    }
    SP_HIP_CHECK(hipGetLastError());
    if (a.n_splits > 1) return launch_reduce(a, a.n_splits, st);
    return SP_OK;
}

// The workgroups of a single-launch kernel wait for each other. Two such kernels on different streams can each hold
// compute units that the other one needs (every XCD dispatches its share of a grid on its own, so one may start with
// the first kernel and another with the second), and both would wait until they give up. The launches of a process
// on one device therefore take turns: a call on another stream than the last one's waits, on the device, for that
// call's kernel. The event for it costs every call 3.6 us (4 layers, 33000 tokens: 26.3 -> 29.9 us; 28.8 as the stop
// event of the launch itself), so none is recorded while all calls come from one stream. The first call from another
// stream can then not wait for what the old one still has in its queue; until that stream's next call, calls from
// others are `unordered`: they give up early and have a stand-in, so that neither side fails.
// Not in a captured graph, which knows nothing of its replays' neighbours: see capturing.

// A stream's identity: handles are reused after hipStreamDestroy, ids are not; the per-thread stream has one handle
// for all threads.
struct StreamKey {
    hipStream_t handle;
    unsigned long long id;
    bool operator==(const StreamKey &o) const { return handle == o.handle && id == o.id; }
};

bool special_stream(hipStream_t st) { return st == nullptr || st == hipStreamLegacy || st == hipStreamPerThread; }

StreamKey key_of(hipStream_t st)
{
    // looked up at run time: not in every runtime of this major version
    using GetId = hipError_t (*)(hipStream_t, unsigned long long *);
    static const GetId get_id = reinterpret_cast<GetId>(dlsym(RTLD_DEFAULT, "hipStreamGetId"));
    static thread_local char tag;
    StreamKey k{st, 0};
    if (st == hipStreamPerThread) k.id = (unsigned long long)(uintptr_t)&tag;
    else if (!special_stream(st) && get_id && get_id(st, &k.id) != hipSuccess) (void)hipGetLastError();
    return k;
}

class Turn {
public:
    explicit Turn(hipStream_t st, bool take = true) : st_(st), key_(key_of(st))
    {
        if (!take) return;
        static Slot slots[64];
        int dev = 0;
        unordered_ = true;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) { (void)hipGetLastError(); return; }
        slot_ = &slots[dev];
        lock_ = std::unique_lock<std::mutex>(slot_->m);
        Slot &s = *slot_;
        const bool same = s.used && s.last == key_;
        if (!s.used || (same && !s.several)) { unordered_ = false; return; }
        if (!s.several) {
            s.several = true;
            s.n_loose = 1;
            s.loose = s.last;
        }
        s.run = same ? s.run + 1 : 0;
        // what this stream left without an event runs before this call anyway
        if (s.n_loose == 1 && s.loose == key_) s.n_loose = 0;
        const bool waits = same || s.done == nullptr || hipStreamWaitEvent(st, s.done, 0) == hipSuccess;
        if (!waits) (void)hipGetLastError();
        unordered_ = !waits || s.n_loose != 0;
    }
    ~Turn()
    {
        if (!slot_) return;
        Slot &s = *slot_;
        s.used = true;
        s.last = key_;
        if (!s.several) return;
        if (s.run >= kSettled && s.n_loose == 0) { s.several = false; return; }
        if (!s.done && hipEventCreateWithFlags(&s.done, hipEventDisableTiming | hipEventDisableSystemFence) != hipSuccess) s.done = nullptr;
        if (s.done && hipEventRecord(s.done, st_) == hipSuccess) return;
        (void)hipGetLastError();
        if (s.n_loose == 0 || !(s.loose == key_)) ++s.n_loose;      // two streams without an event: calls stay unordered
        s.loose = key_;
    }
    Turn(const Turn &) = delete;
    Turn &operator=(const Turn &) = delete;

    // No wait for some call of this process that may still be running: the launch has to make way for it.
    bool unordered() const { return unordered_; }

private:
    static constexpr int kSettled = 256;      // calls in a row from one stream after which it counts as the only one again
    struct Slot {
        std::mutex m;
        hipEvent_t done = nullptr;        // behind the last call's kernel, while there are several streams
        StreamKey last{}, loose{};        // loose: the stream whose latest calls have no event behind them
        int n_loose = 0, run = 0;
        bool used = false, several = false;
    };
    hipStream_t st_;
    StreamKey key_;
    Slot *slot_ = nullptr;
    bool unordered_ = false;
    std::unique_lock<std::mutex> lock_;
};

// A captured call takes the single-launch kernel only where sp_score_is_fused says so, since it takes no turns.
bool capturing(hipStream_t st)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &status) != hipSuccess) { (void)hipGetLastError(); return true; }
    return status != hipStreamCaptureStatusNone;
}

// Compute units that work on this stream may use: fewer than the device has where the stream was made with a mask.
// 0.2 us for a stream of the program's own.
int stream_compute_units(hipStream_t st)
{
    const int cus = device_compute_units();
    if (special_stream(st) || cus < 1) return cus;
    uint32_t mask[32] = {};
    const int words = std::min(32, (cus + 31) / 32);
    if (hipExtStreamGetCUMask(st, (uint32_t)words, mask) != hipSuccess) { (void)hipGetLastError(); return cus; }
    int n = 0;
    for (int i = 0; i < words; ++i) n += __builtin_popcount(mask[i]);
    return n < 1 ? cus : std::min(n, cus);
}

// What the variants of sp_score add to the plain call.
struct ScoreOptions {
    const void *k_look = nullptr;            // lookahead keys in the normaliser
    int32_t look_self = 0;
    const int32_t *block_table = nullptr;    // paged keys
    int64_t page_tokens = 0, page_stride = 0;
    const float *kscale = nullptr;           // 8-bit keys with these scales
};

thread_local int32_t t_path = 0;         // see sp_debug_score_path

sp_status score_impl(const sp_score_desc *desc, const void *q_dev, const void *const *k_layers_host,
                     const int64_t *offsets_host, const int64_t *offsets_dev, int32_t B, int64_t L_single,
                     const ScoreOptions &opt, float *scores_dev, void *ws_dev, size_t ws_bytes, void *hip_stream)
{
    Plan p;
    sp_status rc = make_plan(desc, p);
    if (rc != SP_OK) return rc;
    if (!q_dev || !k_layers_host || !scores_dev)
        return sp::fail(SP_ERR_INVALID_ARG, "q_dev, k_layers_host and scores_dev must not be null");
    LayerPtrs kp;
    std::memset(&kp, 0, sizeof kp);
    for (int l = 0; l < desc->n_layers; ++l) {
        if (!k_layers_host[l]) return sp::fail(SP_ERR_INVALID_ARG, "k_layers_host[%d] is null", l);
        if ((uintptr_t)k_layers_host[l] % 16 != 0)
            return sp::fail(SP_ERR_INVALID_ARG, "k_layers_host[%d] is not 16-byte aligned", l);
        kp.p[l] = static_cast<const uint16_t *>(k_layers_host[l]);
    }
    if ((uintptr_t)q_dev % 16 != 0) return sp::fail(SP_ERR_INVALID_ARG, "q_dev is not 16-byte aligned");
    if (opt.look_self != 0 && opt.look_self != 1)
        return sp::fail(SP_ERR_INVALID_ARG, "look_self = %d must be 0 or 1", opt.look_self);
    if (opt.block_table) {
        // a page holds whole tiles of either score path, and its rows are addressed with the desc's strides
        if (opt.page_tokens < sp_fused::kTileKeys || opt.page_tokens % sp_fused::kTileKeys != 0)
            return sp::fail(SP_ERR_INVALID_ARG, "page_tokens = %lld must be a positive multiple of %d",
                            (long long)opt.page_tokens, sp_fused::kTileKeys);
        if (opt.page_stride < 0 || opt.page_stride % 8 != 0)
            return sp::fail(SP_ERR_INVALID_ARG, "page_stride = %lld must be a non-negative multiple of 8 elements",
                            (long long)opt.page_stride);
    }

    int64_t total = 0, n_tiles = 0, longest = 0;
    const bool batch = offsets_host != nullptr;
    if (batch) {
        if (!offsets_dev) return sp::fail(SP_ERR_INVALID_ARG, "offsets_dev is null");
        if (B < 1 || B > kMaxPrompts) return sp::fail(SP_ERR_INVALID_ARG, "B = %d (supported: 1..%d)", B, kMaxPrompts);
        if (offsets_host[0] != 0) return sp::fail(SP_ERR_INVALID_ARG, "offsets_host[0] must be 0");
        for (int b = 0; b < B; ++b) {
            const int64_t len = offsets_host[b + 1] - offsets_host[b];
            if (len < 0) return sp::fail(SP_ERR_INVALID_ARG, "offsets_host decreases at prompt %d", b);
            n_tiles += sp::ceil_div(len, p.tile_keys);
            longest = std::max(longest, len);
        }
        total = offsets_host[B];
    } else {
        if (L_single < 0) return sp::fail(SP_ERR_INVALID_ARG, "L = %lld is negative", (long long)L_single);
        total = L_single;
        n_tiles = sp::ceil_div(total, p.tile_keys);
        longest = total;
        B = 1;
    }
    if (total == 0) return SP_OK;
    if (n_tiles > 0x7fffffff / 2) return sp::fail(SP_ERR_UNSUPPORTED, "too many key tiles (%lld)", (long long)n_tiles);

    const WsLayout w = ws_layout(p, n_tiles, B);
    if (!ws_dev) return sp::fail(SP_ERR_WORKSPACE, "ws_dev is null (%zu bytes needed)", w.total);
    if ((uintptr_t)ws_dev % 256 != 0) return sp::fail(SP_ERR_WORKSPACE, "ws_dev is not 256-byte aligned");
    if (ws_bytes < w.total) return sp::fail(SP_ERR_WORKSPACE, "workspace too small: %zu < %zu", ws_bytes, w.total);

    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    char *ws = static_cast<char *>(ws_dev);
    ScoreArgs a;
    std::memset(&a, 0, sizeof a);
    a.q = static_cast<const uint16_t *>(q_dev);
    a.k_stride_token = desc->k_stride_token;
    a.k_stride_head = desc->k_stride_head;
    a.L = total;
    a.part = reinterpret_cast<float2 *>(ws + w.part);
    a.lse_neg = reinterpret_cast<float *>(ws + w.lse);
    a.scores = scores_dev;
    a.status = reinterpret_cast<uint32_t *>(ws + w.status);
    a.split_buf = reinterpret_cast<float *>(ws + w.split);
    a.layers_per_split = prob_layers_per_split(p, n_tiles);
    a.n_splits = prob_splits(p, n_tiles);
    a.n_tiles = (int32_t)n_tiles;
    a.n_prompts = B;
    a.n_layers = desc->n_layers;
    a.n_q_heads = desc->n_q_heads;
    a.n_kv_heads = desc->n_kv_heads;
    a.group = desc->n_q_heads / desc->n_kv_heads;
    a.n_q = desc->n_q;
    a.n_nblk = p.NB;
    a.n_gblk = p.n_gblk;
    a.rows_pad = p.rows_pad;
    a.layer_agg = desc->layer_agg;
    a.c = desc->scale * 1.44269504088896340736f;
    a.inv_c = 1.0f / a.c;
    a.out_scale = (desc->layer_agg == SP_LAYER_MAX) ? 1.0f / (float)desc->n_q
                                                   : 1.0f / ((float)desc->n_q * (float)desc->n_layers);
    a.block_table = opt.block_table;
    a.page_tokens = opt.page_tokens;
    a.page_stride = opt.page_stride;
    a.kscale = opt.kscale;
    float *const look = opt.k_look ? reinterpret_cast<float *>(ws + w.look) : nullptr;
    a.look = look;
    auto launch_look = [&](void *clear, size_t clear_n, uint32_t *status) -> sp_status {
        const auto kernel = p.D == 64 ? sp_look_kernel<64> : sp_look_kernel<128>;
        // Workgroups beyond the phases clear only: with few phases the area, up to 1 MB, would be left to as few workgroups
        // (one phase, 131072 tokens, 16 lookahead rows: 38.1 us a call against 23.9; 26.4 with a clear launch).
        const int groups = std::max(p.n_phases, (int)std::min<size_t>(sp::ceil_div(clear_n, (size_t)kThreads), 256));
        hipLaunchKernelGGL(kernel, dim3(groups), dim3(kThreads), 0, st, a, static_cast<const uint16_t *>(opt.k_look),
                           (int)opt.look_self, look, static_cast<uint64_t *>(clear), clear_n, status);
        SP_HIP_CHECK(hipGetLastError());
        return SP_OK;
    };
    // the single-launch kernel fetches 8-bit keys in 16-byte pieces
    const bool may_fuse = !opt.kscale || (fp8_strides_ok(desc) && !fused_big(p));
    sp_fused::FusedArgs f;
    std::memset(&f, 0, sizeof f);
    f.q = a.q;
    f.head_dim = p.D;
    f.tile_keys = fused_tile(p);
    f.k_stride_token = a.k_stride_token;
    f.k_stride_head = a.k_stride_head;
    f.kscale = opt.kscale;
    f.look = a.look;
    f.block_table = a.block_table;
    f.page_tokens = a.page_tokens;
    f.page_stride = a.page_stride;
    f.scores = scores_dev;
    f.n_layers = a.n_layers; f.n_q_heads = a.n_q_heads; f.n_kv_heads = a.n_kv_heads;
    f.group = a.group; f.n_q = a.n_q;
    f.n_nblk = a.n_nblk; f.n_gblk = a.n_gblk; f.rows_pad = a.rows_pad;
    f.layer_agg = a.layer_agg;
    f.c = a.c; f.inv_c = a.inv_c; f.out_scale = a.out_scale;
    BatchGroups bg;
    const bool captured = may_fuse && capturing(st);
    // On part of the device the ranges that would fill it only wait for each other. What is announced keeps its kernel
    // where that has a compute unit for every workgroup of first fit, but they are spread over the XCDs without regard to the mask.
    const int cus = captured || !may_fuse ? device_compute_units() : stream_compute_units(st);
    const bool masked = cus < device_compute_units();
    // What sp_score_is_fused and sp_score_batch_is_fused announce may fail. Every other call on the single-launch kernel,
    // and one that could not be ordered behind its neighbours, gives up early (see kYieldSpins) and is finished by a
    // launch that can do without that kernel.
    bool pair = may_fuse && !captured && !batch && pair_applies(p, opt.kscale != nullptr, total, desc->k_stride_token);
    bool fused = may_fuse && !pair && (batch ? plan_fused_batch(p, offsets_host, B, n_tiles * p.tile_keys, desc->k_stride_token, w,
                                                              masked ? Launches::kFirstFit : Launches::kRanges, bg)
                                             : plan_fused_prompt(p, total, desc->k_stride_token, bg));
    const bool big = fused_big(p);
    if (pair && big)            // no exchange area of their own: see fused_big
        pair = sp_fused::workspace_bytes(p.rows_pad, (int)sp::ceil_div(total, 2 * fused_tile(p)), 1) <= w.split - w.part;
    int ranges = bg.ranges;
    if (fused && !captured && bg.groups.size() == 1) {
        // the exchange area of a launch in layer ranges takes the place of the general path's buffers
        ranges = fused_ranges(p, bg.wgs[0], bg.groups[0].n, w.split - w.part);
    }
    const bool announced = fused && !big && (batch ? bg.announced : bg.wgs[0] >= fused_min_workgroups(p));
    if (fused && !announced)
        fused = !captured && (batch || ranges > 1 || bg.wgs[0] >= fused_min_workgroups(p)) && steps_pay(p, opt.kscale != nullptr, bg.prompts, n_tiles * p.tile_keys, ranges, (int)bg.groups.size());
    if (fused && big)           // no exchange area of their own: see fused_big
        for (size_t g = 0; g < bg.groups.size(); ++g)
            fused = fused && sp_fused::workspace_bytes(p.rows_pad, bg.wgs[g], bg.groups[g].n) <= w.split - w.part;
    if (masked) {
        pair = false;
        ranges = 1;
        fused = fused && announced && *std::max_element(bg.wgs.begin(), bg.wgs.end()) <= cus;
    }
    if (fused || pair) {
        bool stand_in = !announced || masked;
        {
            const Turn turn(st, !captured);
            stand_in = stand_in || turn.unordered();
            uint32_t *const err = stand_in ? a.status + 1 : a.status;
            f.L = total;
            f.spin_max = stand_in ? sp_fused::kYieldSpins : UINT32_MAX;
            sp_status rs = SP_OK;
            // with lookahead keys (of one prompt: one launch) their kernel clears
            using sp_fused::Clear;
            const Clear clear = look ? Clear::kDone : Clear::kAll;
            auto clear_and_look = [&](int n_entries, void *area) {
                return look ? launch_look(area, sp_fused::exchange_words(p.rows_pad, f.n_wg, n_entries), err) : SP_OK;
            };
            if (pair) {
                f.tile_keys = 2 * fused_tile(p);
                f.n_wg = (int)sp::ceil_div(total, f.tile_keys);
                char *const area = ws + (big ? w.part : w.fused);
                rs = clear_and_look(1, area);
                if (rs == SP_OK) rs = sp_fused::launch(f, kp, nullptr, true, clear, area, err, st);
            } else if (ranges > 1) {
                f.split_out = a.split_buf;
                f.split_stride = total;
                for (size_t g = 0; g < bg.groups.size() && rs == SP_OK; ++g) {
                    const sp_fused::GroupTable t = split_layers(bg.groups[g], p.n_layers, ranges);
                    f.n_wg = bg.wgs[g] * ranges;
                    rs = clear_and_look(t.n, ws + w.part);
                    if (rs == SP_OK) rs = sp_fused::launch(f, kp, &t, false, g > 0 ? Clear::kExchange : clear, ws + w.part, err, st);
                }
            } else {
                for (size_t g = 0; g < bg.groups.size() && rs == SP_OK; ++g) {
                    f.n_wg = bg.wgs[g];
                    // duties rotate over all prompts of a launch where they can: within a prompt of a dozen workgroups
                    // each would have one every other phase (8 prompts of 2K .. 32K tokens: 342 against 394 us)
                    char *const area = ws + (big ? w.part : w.fused);
                    rs = clear_and_look(1, area);
                    if (rs == SP_OK)
                        rs = sp_fused::launch(f, kp, batch ? &bg.groups[g] : nullptr, duties_shared(p, bg, g), g > 0 ? Clear::kExchange : clear, area, err, st);
                }
            }
            if (rs != SP_OK) return rs;
        }
        t_path = (pair ? 2 : 1) | ranges << 8 | (pair ? 1 : (int32_t)std::min<size_t>(bg.groups.size(), 255)) << 16 | (int32_t)stand_in << 24;
        if (stand_in) return launch_finish(p, a, kp, batch ? offsets_dev : nullptr, a.status + 1, ranges, st);
        if (ranges > 1) return launch_reduce(a, ranges, st);
        if (bg.groups.size() > 1 || bg.groups[0].n > 1) {
            hipLaunchKernelGGL(sp_fail_all_kernel, dim3((unsigned)std::min<int64_t>(sp::ceil_div(total, 1024), 64)), dim3(256), 0, st,
                               (const uint32_t *)a.status, total, scores_dev);
            SP_HIP_CHECK(hipGetLastError());
        }
        return SP_OK;
    }
    t_path = 0;
    if (look) {
        const sp_status rs = launch_look(nullptr, 0, nullptr);
        if (rs != SP_OK) return rs;
    }
    if (batch) {
        TileInfo *tiles = reinterpret_cast<TileInfo *>(ws + w.tiles);
        int32_t *pt = reinterpret_cast<int32_t *>(ws + w.prompt_tiles);
        hipLaunchKernelGGL(sp_tiles_kernel, dim3(1), dim3(256), 0, st, offsets_dev, B, p.tile_keys, tiles, pt,
                           (int)n_tiles);
        SP_HIP_CHECK(hipGetLastError());
        a.tiles = tiles;
        a.prompt_tiles = pt;
    }
    if (opt.kscale) return p.D == 64 ? launch_all<64, 2, true>(p, a, kp, longest, st) : launch_all<128, 1, true>(p, a, kp, longest, st);
    if (p.D == 64) return launch_all<64, 2>(p, a, kp, longest, st);
    return launch_all<128, 1>(p, a, kp, longest, st);
}

}  // namespace

extern "C" sp_status sp_score_workspace(const sp_score_desc *desc, int64_t total_tokens, int32_t n_prompts,
                                        size_t *bytes)
{
    Plan p;
    sp_status rc = make_plan(desc, p);
    if (rc != SP_OK) return rc;
    if (!bytes) return sp::fail(SP_ERR_INVALID_ARG, "bytes is null");
    if (total_tokens < 0 || n_prompts < 1 || n_prompts > kMaxPrompts)
        return sp::fail(SP_ERR_INVALID_ARG, "total_tokens must be >= 0 and n_prompts in 1..%d", kMaxPrompts);
    const int64_t n_tiles = sp::ceil_div(total_tokens, p.tile_keys) + n_prompts;
    *bytes = ws_layout(p, n_tiles, n_prompts).total;
    return SP_OK;
}

extern "C" void sp_debug_fused_giveup(uint32_t spin_limit, int32_t force_miss)
{
    sp_fused::set_giveup(spin_limit, force_miss);
}

extern "C" int32_t sp_debug_score_path(void) { return t_path; }

extern "C" int32_t sp_score_is_fused(const sp_score_desc *desc, int64_t L)
{
    Plan p;
    if (make_plan(desc, p) != SP_OK) return -1;
    return fused_applies(p, L, desc->k_stride_token) ? 1 : 0;
}

extern "C" int32_t sp_score_fp8_is_fused(const sp_score_desc *desc, int64_t L)
{
    Plan p;
    if (make_plan(desc, p) != SP_OK) return -1;
    return fused_applies_fp8(p, desc, L) ? 1 : 0;
}

extern "C" int32_t sp_score_batch_is_fused(const sp_score_desc *desc, const int64_t *offsets_host, int32_t B)
{
    Plan p;
    if (make_plan(desc, p) != SP_OK || !offsets_host || B < 1 || B > kMaxPrompts) return -1;
    for (int b = 0; b < B; ++b)
        if (offsets_host[b + 1] < offsets_host[b]) return -1;
    if (!fused_base_shape(p)) return 0;
    int64_t n_tiles = 0;
    for (int b = 0; b < B; ++b) n_tiles += sp::ceil_div(offsets_host[b + 1] - offsets_host[b], p.tile_keys);
    if (n_tiles > 0x7fffffff / 2) return 0;
    BatchGroups bg;
    if (!plan_fused_batch(p, offsets_host, B, n_tiles * p.tile_keys, desc->k_stride_token, ws_layout(p, n_tiles, B), Launches::kRanges, bg) || !bg.announced) return 0;
    return (int32_t)bg.groups.size();
}

extern "C" sp_status sp_score(const sp_score_desc *desc, const void *q_dev, const void *const *k_layers_host,
                              int64_t L, float *scores_dev, void *ws_dev, size_t ws_bytes, void *hip_stream)
{
    return score_impl(desc, q_dev, k_layers_host, nullptr, nullptr, 1, L, ScoreOptions(), scores_dev, ws_dev, ws_bytes,
                      hip_stream);
}

extern "C" sp_status sp_score_look(const sp_score_desc *desc, const void *q_dev, const void *const *k_layers_host,
                                   int64_t L, const void *k_look_dev, int32_t look_self, float *scores_dev,
                                   void *ws_dev, size_t ws_bytes, void *hip_stream)
{
    if (!k_look_dev) return sp::fail(SP_ERR_INVALID_ARG, "k_look_dev is null");
    if ((uintptr_t)k_look_dev % 16 != 0) return sp::fail(SP_ERR_INVALID_ARG, "k_look_dev is not 16-byte aligned");
    ScoreOptions opt;
    opt.k_look = k_look_dev;
    opt.look_self = look_self;
    return score_impl(desc, q_dev, k_layers_host, nullptr, nullptr, 1, L, opt, scores_dev, ws_dev, ws_bytes, hip_stream);
}

extern "C" sp_status sp_score_paged(const sp_score_desc *desc, const void *q_dev, const void *const *k_pools_host,
                                    const int32_t *block_table_dev, int64_t page_tokens, int64_t page_stride, int64_t L,
                                    float *scores_dev, void *ws_dev, size_t ws_bytes, void *hip_stream)
{
    if (!block_table_dev) return sp::fail(SP_ERR_INVALID_ARG, "block_table_dev is null");
    ScoreOptions opt;
    opt.block_table = block_table_dev;
    opt.page_tokens = page_tokens;
    opt.page_stride = page_stride;
    return score_impl(desc, q_dev, k_pools_host, nullptr, nullptr, 1, L, opt, scores_dev, ws_dev, ws_bytes, hip_stream);
}

extern "C" sp_status sp_score_fp8(const sp_score_desc *desc, const void *q_dev, const void *const *k8_layers_host,
                                  const float *kscale_dev, int64_t L, float *scores_dev, void *ws_dev, size_t ws_bytes,
                                  void *hip_stream)
{
    if (!kscale_dev) return sp::fail(SP_ERR_INVALID_ARG, "kscale_dev is null");
    ScoreOptions opt;
    opt.kscale = kscale_dev;
    return score_impl(desc, q_dev, k8_layers_host, nullptr, nullptr, 1, L, opt, scores_dev, ws_dev, ws_bytes, hip_stream);
}

extern "C" sp_status sp_score_batch(const sp_score_desc *desc, const void *q_dev, const void *const *k_layers_host,
                                    const int64_t *offsets_host, const int64_t *offsets_dev, int32_t B,
                                    float *scores_dev, void *ws_dev, size_t ws_bytes, void *hip_stream)
{
    if (!offsets_host) return sp::fail(SP_ERR_INVALID_ARG, "offsets_host is null");
    return score_impl(desc, q_dev, k_layers_host, offsets_host, offsets_dev, B, 0, ScoreOptions(), scores_dev, ws_dev,
                      ws_bytes, hip_stream);
}
