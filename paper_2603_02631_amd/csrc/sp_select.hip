// sp_select: average pooling, chunk means, top-k chunks, merged spans
// (paper: Algorithm 1 "AvgPool1D", "PartitionIntoChunks", "TopKChunks",
// "MergeAdjacentChunks"; Appendix A.1.2; Appendix A.3).
//
// Two kernels (prompts of a few chunks take both in one launch, sp_select_one_kernel):
//   sp_chunk_kernel  one wavefront per chunk: the mean of the chunk's window
//                    sums as one weighted sum, reduced by a fixed-order shuffle
//                    tree. The pooled vector is never written out.
//   sp_topk_kernel   one workgroup. MSB-first radix select (up to 4 passes of 8
//                    bits) on order-preserving integer images of the fp32 chunk
//                    scores finds the k-th largest score exactly; chunks above
//                    it are kept, chunks equal to it are kept in index order
//                    until k is reached (lower index wins a tie); the kept
//                    set as a bit string gives the indices in ascending order
//                    and the merged spans.
// Everything is integer or fixed-order fp32 work, so results are deterministic.
//
// sp_select_budget (Section 3.1: a fixed target-side length of the compressed
// prompt) finds k on the device instead of taking it from the host. With
// rank[j] = position of chunk j in the order (score descending, index
// ascending), the top-k chunks are those of rank < k, and whether target token t
// is kept by the top-k chunks depends on k only through one number r(t): a token
// with at least one character is kept iff some chunk whose character interval it
// overlaps is selected, r(t) = the smallest rank among those chunks; a token
// without characters is kept iff it lies strictly inside a merged span, i.e.
// inside one chunk or on a boundary whose chunks on both sides are all selected,
// r(t) = the largest rank among them. Kept tokens at k = #{t : r(t) < k}: a
// histogram of r and a prefix sum give the count for every k at once.
// Up to 8192 chunks the tokens need not wait for the ranks: whether a token's number is the smallest or the largest
// rank among some chunks, it is the rank of one of them, which their scores tell as well.
//   sp_chunk_kernel       also leaves the chunk boundaries' character offsets in a
//                         compact array and clears the counters of the next one;
//   sp_rank_tokens_kernel  some workgroups: rank of every chunk by counting, tiles of 1024
//                         chunks against tiles of 64; the others: one thread per target token,
//                         binary search of the compact boundary array, the chunk whose rank is
//                         r(t), histogram by chunk;
//   sp_budget_select_kernel  one workgroup: histogram by rank, prefix sum, largest k within
//                         the budget, and the chunks of rank < k with their spans.
// Beyond 8192 chunks ranks (sp_rank_kernel) and tokens (sp_token_rank_kernel, histogram by
// rank) are two launches, and so is the last one: sp_budget_kernel for k, and
// sp_topk_kernel as above, reading k from device memory.
#include "sp_common.hpp"

#include <algorithm>
#include <atomic>

namespace {

constexpr int kChunkThreads = 256;           // 4 waves, one chunk each
constexpr int kMaxPool = 129;
constexpr int kTopkThreads = 1024;

// Sum over the wave, the same in all lanes: four butterfly steps of data-parallel-primitive moves within the rows of
// 16, then the four rows' sums (no trip through LDS as shuffles make).
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v)
{
    return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float wave_sum(float v)
{
    v = dpp_add<0xB1>(v);           // quad_perm [1,0,3,2]
    v = dpp_add<0x4E>(v);           // quad_perm [2,3,0,1]
    v = dpp_add<0x141>(v);          // mirror within 8 lanes
    v = dpp_add<0x140>(v);          // mirror within 16 lanes
    auto row = [&](int lane) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane)); };
    return (row(0) + row(16)) + (row(32) + row(48));
}

// Chunk scores of chunks ci, ci + stride, .. (N of them, those past the last excepted) by one wave, the same in all
// lanes. The mean of the chunk's window sums is a weighted sum of its tokens and the (w - 1) / 2 on either side, a
// token's weight being the number of the chunk's windows that contain it: one load and one fma per token instead
// of pool_w additions, nothing staged.
template <int N>
__device__ __forceinline__ void chunk_means(const float *__restrict__ scores, int64_t L, int pool_w, int chunk, int64_t n_chunks,
                                            int64_t ci, int stride, float (&mean)[N])
{
    const int lane = threadIdx.x & 63, half = (pool_w - 1) / 2;
    const float *src[N];            // the first token's score; positions below count from half tokens before it
    uint32_t size[N], lo[N], hi[N];         // a chunk and its neighbours may pass 2^31 tokens
    uint32_t n_tok = 0;
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const int64_t begin = (ci + u * stride) * chunk;
        const bool live = ci + u * stride < n_chunks;
        size[u] = live ? (uint32_t)(begin + chunk < L ? chunk : L - begin) : 1;
        src[u] = scores + (live ? begin : 0);
        lo[u] = begin < half ? (uint32_t)(half - begin) : 0;                       // tokens before the prompt are zeros,
        hi[u] = live ? size[u] + half + (uint32_t)(L - begin - size[u] < half ? L - begin - size[u] : half) : 0;     // and those behind it
        n_tok = hi[u] > n_tok ? hi[u] : n_tok;
        mean[u] = 0.f;
    }
    for (uint32_t t = lane; t < n_tok; t += 64) {
        float v[N];
#pragma unroll
        for (int u = 0; u < N; ++u) v[u] = t >= lo[u] && t < hi[u] ? src[u][(int64_t)t - half] : 0.f;
#pragma unroll
        for (int u = 0; u < N; ++u) {
            // windows centred on this chunk's tokens t - 2 half .. t contain the token
            const uint32_t first = t > 2u * half ? t - 2u * half : 0u, last = t < size[u] - 1 ? t : size[u] - 1;
            mean[u] = fmaf((float)(last - first + 1), v[u], mean[u]);
        }
    }
#pragma unroll
    for (int u = 0; u < N; ++u) mean[u] = wave_sum(mean[u]) / ((float)pool_w * (float)size[u]) + 0.0f;
}

__device__ __forceinline__ void chunk_body(const float *__restrict__ scores, int64_t L, int pool_w, int chunk,
                                           int64_t n_chunks, float *__restrict__ cs_ws, float *__restrict__ cs_out,
                                           const int64_t *__restrict__ draft_off, int64_t *__restrict__ bnd,
                                           int32_t *__restrict__ rank, int32_t *__restrict__ hist)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t ci = (int64_t)blockIdx.x * (kChunkThreads / 64) + wave;
    if (ci >= n_chunks) return;              // whole wave leaves together; no block barrier is used
    float v[1];
    chunk_means<1>(scores, L, pool_w, chunk, n_chunks, ci, 0, v);
    if (lane == 0) {
        cs_ws[ci] = v[0];
        if (cs_out) cs_out[ci] = v[0];
        if (bnd) {
            // set-up for the budget search: character offset of the chunk's first token (one more entry:
            // the end of the text), cleared rank counters and histogram bins (one more: "never kept")
            bnd[ci] = draft_off[ci * chunk];
            rank[ci] = 0;
            hist[ci] = 0;
            if (ci == n_chunks - 1) {
                bnd[n_chunks] = draft_off[L];
                hist[n_chunks] = 0;
            }
        }
    }
}

__global__ __launch_bounds__(kChunkThreads) void sp_chunk_kernel(const float *__restrict__ scores, int64_t L,
                                                                 int pool_w, int chunk, int64_t n_chunks,
                                                                 float *__restrict__ cs_ws,
                                                                 float *__restrict__ cs_out,
                                                                 const int64_t *__restrict__ draft_off,
                                                                 int64_t *__restrict__ bnd,
                                                                 int32_t *__restrict__ rank,
                                                                 int32_t *__restrict__ hist)
{
    chunk_body(scores, L, pool_w, chunk, n_chunks, cs_ws, cs_out, draft_off, bnd, rank, hist);
}

// Ragged batch: prompt b = blockIdx.y owns scores [off[b], off[b+1]) and the chunk-score slots from
// off[b] / chunk + b on (distinct prompts' slots cannot overlap: a prompt has at most
// off[b+1] / chunk - off[b] / chunk + 1 chunks).
__device__ __forceinline__ int64_t batch_chunk_slot(int64_t off_b, int b, int chunk) { return off_b / chunk + b; }

__global__ __launch_bounds__(kChunkThreads) void sp_chunk_batch_kernel(const float *__restrict__ scores,
                                                                       const int64_t *__restrict__ off, int pool_w,
                                                                       int chunk, float *__restrict__ cs_ws,
                                                                       float *__restrict__ cs_out)
{
    const int b = blockIdx.y;
    const int64_t o = off[b], L = off[b + 1] - o;
    const int64_t n_chunks = (L + chunk - 1) / chunk;
    if ((int64_t)blockIdx.x * (kChunkThreads / 64) >= n_chunks) return;        // also: empty prompt
    const int64_t slot = batch_chunk_slot(o, b, chunk);
    chunk_body(scores + o, L, pool_w, chunk, n_chunks, cs_ws + slot, cs_out ? cs_out + slot : nullptr, nullptr, nullptr,
               nullptr, nullptr);
}

// fp32 -> uint32 whose unsigned order is the float order (-0 mapped onto +0 first).
__device__ __forceinline__ uint32_t order_key(float v)
{
    const uint32_t u = __float_as_uint(v + 0.0f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Inclusive block scan of one int per thread (1024 threads = 16 waves).
__device__ __forceinline__ int block_scan_incl(int v, int *wave_tot /*[16]*/, int &block_total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    __syncthreads();                         // protects wave_tot from the previous use
    if (lane == 63) wave_tot[wave] = x;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kTopkThreads / 64; ++w) {
        const int t = wave_tot[w];
        if (w < wave) base += t;
        tot += t;
    }
    block_total = tot;
    return x + base;
}

// The k-th largest key's bucket: keys whose bits under `mask` equal `prefix`, of which the first `need` in index
// order are kept (all of them if the search could stop before the last bit), besides every larger one.
struct Threshold {
    uint32_t prefix, mask;
    int64_t need;
};

// Radix select by one workgroup, most significant byte first. Per pass all threads count their candidates into
// a 256-bin histogram; wave 0 alone scans the bins from the top (four per lane, one shuffle scan), picks the bin
// that holds the k-th, and clears the histogram for the next pass: two barriers per pass. The search ends as
// soon as the bin holds exactly the keys still needed (one of distinct scores: three passes, seldom four).
// Scores share a handful of exponents, so in the first pass a wave adds up its keys of one bin before it
// touches the counter: one by one, 64 keys of a bin take 64 turns at it. Two bins so; what is left is spread, and goes
// one by one (8000 lognormal chunk scores: 15.9 us, with three turns 18.8, with as many as there are bins 19.1; spread
// over 200 powers of two 14.8, 17.9 and 69.0).
// count(f) calls f(key, live) for each of this thread's keys, the same number of times in every thread of a wave.
template <class Count>
__device__ __forceinline__ Threshold radix_select(int64_t k, const Count &count)
{
    __shared__ int hist[256];
    __shared__ uint32_t s_prefix;
    __shared__ int64_t s_need;
    __shared__ int s_found;
    const int tid = threadIdx.x;
    Threshold t{0u, 0u, k};
    if (tid < 256) hist[tid] = 0;
    __syncthreads();
    for (int shift = 24; shift >= 0; shift -= 8) {
        if (shift == 24) {
            count([&](uint32_t key, bool live) {
                const uint32_t bin = key >> 24;
                uint64_t left = __ballot(live);
#pragma unroll
                for (int turn = 0; turn < 2; ++turn) {
                    if (left == 0) return;             // uniform
                    const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)bin, __ffsll((unsigned long long)left) - 1);
                    const uint64_t same = __ballot(live && bin == b) & left;
                    if ((tid & 63) == 0) atomicAdd(&hist[b], __popcll(same));
                    left &= ~same;
                }
                if ((left >> (tid & 63)) & 1) atomicAdd(&hist[bin], 1);
            });
        } else {
            count([&](uint32_t key, bool live) {
                if (live && (key & t.mask) == t.prefix) atomicAdd(&hist[(key >> shift) & 255u], 1);
            });
        }
        __syncthreads();
        if (tid < 64) {
            // lane l owns bins 255-4l .. 252-4l, in that (descending) order
            int h[4], lane_sum = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                h[j] = hist[255 - 4 * tid - j];
                hist[255 - 4 * tid - j] = 0;
                lane_sum += h[j];
            }
            int incl = lane_sum;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int y = __shfl_up(incl, off);
                if (tid >= off) incl += y;
            }
            int64_t before = incl - lane_sum;        // candidates in the bins above this lane's
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (before < t.need && before + h[j] >= t.need) {
                    s_prefix = t.prefix | ((uint32_t)(255 - 4 * tid - j) << shift);
                    s_need = t.need - before;
                    s_found = h[j];
                }
                before += h[j];
            }
        }
        __syncthreads();
        t.prefix = s_prefix;
        t.need = s_need;
        t.mask |= 255u << shift;
        if (s_found == t.need) break;                // uniform
    }
    return t;
}

// Lowest n set bits of x.
__device__ __forceinline__ uint64_t lowest_bits(uint64_t x, int64_t n)
{
    if (n <= 0) return 0;
    for (int64_t drop = __popcll(x) - n; drop > 0; --drop) x &= ~(1ull << (63 - __clzll((long long)x)));
    return x;
}

// Kept chunks and merged spans of up to R * 1024 chunks; chunk r * 1024 + thread is kept if gt[r], or if eq[r] and
// it is among the first `need` of those in index order. The kept set is a bit string in LDS, 64 chunks a word: one
// wave decides the ties and turns the words' population counts into output positions, the starts and ends of its
// runs are the spans, and every thread writes its own chunks' entries; nothing written is read back.
template <int R>
__device__ __forceinline__ void emit_kept(const bool (&gt)[R], const bool (&eq)[R], int64_t need, int chunk, int64_t L,
                                          int32_t *__restrict__ sel, int64_t *__restrict__ spans, int32_t *__restrict__ n_spans)
{
    constexpr int kWords = R * kTopkThreads / 64;
    static_assert(kWords % 2 == 0 && kWords <= 128, "two words a lane");
    __shared__ uint64_t s_gt[kWords], s_eq[kWords], s_start[kWords], s_end[kWords];
    __shared__ int32_t s_pos[kWords], s_id[kWords];       // kept chunks and spans before the word
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint64_t g = __ballot(gt[r]), e = __ballot(eq[r]);
        if (lane == 0) { s_gt[r * (kTopkThreads / 64) + wave] = g; s_eq[r * (kTopkThreads / 64) + wave] = e; }
    }
    __syncthreads();
    if (wave == 0) {
        const bool has = 2 * lane < kWords;               // lane l: words 2l and 2l + 1
        const uint64_t q0 = has ? s_eq[2 * lane] : 0, q1 = has ? s_eq[2 * lane + 1] : 0;
        const int e0 = __popcll(q0), e = e0 + __popcll(q1);
        int ei = e;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int y = __shfl_up(ei, off);
            if (lane >= off) ei += y;
        }
        const int64_t room = need - (ei - e);           // equal keys still to keep from this lane's first word on
        const uint64_t k0 = (has ? s_gt[2 * lane] : 0) | lowest_bits(q0, room);
        const uint64_t k1 = (has ? s_gt[2 * lane + 1] : 0) | lowest_bits(q1, room - e0);
        int before = __shfl_up((int)(k1 >> 63), 1), after = __shfl_down((int)(k0 & 1), 1);
        if (lane == 0) before = 0;
        if (lane == 63) after = 0;
        const uint64_t b0 = k0 & ~((k0 << 1) | (uint64_t)before), b1 = k1 & ~((k1 << 1) | (k0 >> 63));
        const uint64_t f0 = k0 & ~((k0 >> 1) | (k1 << 63)), f1 = k1 & ~((k1 >> 1) | ((uint64_t)after << 63));
        const int p0 = __popcll(k0) | __popcll(b0) << 16, p = p0 + (__popcll(k1) | __popcll(b1) << 16);
        int pi = p;                                       // both counts fit 16 bits
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int y = __shfl_up(pi, off);
            if (lane >= off) pi += y;
        }
        const int px = pi - p, py = px + p0;
        if (has) {
            s_gt[2 * lane] = k0;      s_gt[2 * lane + 1] = k1;
            s_start[2 * lane] = b0;   s_start[2 * lane + 1] = b1;
            s_end[2 * lane] = f0;     s_end[2 * lane + 1] = f1;
            s_pos[2 * lane] = px & 0xffff; s_pos[2 * lane + 1] = py & 0xffff;
            s_id[2 * lane] = px >> 16;     s_id[2 * lane + 1] = py >> 16;
        }
        if (lane == 63) *n_spans = pi >> 16;
    }
    __syncthreads();
    const uint64_t below = (1ull << lane) - 1;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int w = r * (kTopkThreads / 64) + wave;
        const uint64_t kept = s_gt[w], start = s_start[w];
        if (((kept >> lane) & 1) == 0) continue;
        const int64_t i = (int64_t)r * kTopkThreads + tid;
        sel[s_pos[w] + __popcll(kept & below)] = (int32_t)i;
        const int64_t id = s_id[w] + __popcll(start & (below << 1 | 1)) - 1;
        if ((start >> lane) & 1) spans[2 * id] = i * chunk;
        if ((s_end[w] >> lane) & 1) spans[2 * id + 1] = (i + 1) * chunk < L ? (i + 1) * chunk : L;
    }
}

// Up to R * 1024 chunks, whose keys stay in registers.
// Bound by its chain of dependent steps: the workgroup reads 8 KB. With a block scan per 1024 chunks, the kept
// indices read back for the spans, and four passes of the radix select always, 2048 chunks took 11 us instead of 8.
template <int R, class Score>
__device__ __forceinline__ void topk_words(const Score &score, int64_t n_chunks, int64_t k, int chunk, int64_t L,
                                           int32_t *__restrict__ sel, int64_t *__restrict__ spans, int32_t *__restrict__ n_spans)
{
    const int tid = threadIdx.x;
    uint32_t key[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = (int64_t)r * kTopkThreads + tid;
        key[r] = i < n_chunks ? order_key(score(i)) : 0u;
    }
    const Threshold t = radix_select(k, [&](auto &&f) {
#pragma unroll
        for (int r = 0; r < R; ++r) f(key[r], (int64_t)r * kTopkThreads + tid < n_chunks);
    });
    bool gt[R], eq[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool live = (int64_t)r * kTopkThreads + tid < n_chunks;
        gt[r] = live && (key[r] & t.mask) > t.prefix;
        eq[r] = live && (key[r] & t.mask) == t.prefix;
    }
    emit_kept<R>(gt, eq, t.need, chunk, L, sel, spans, n_spans);
}

// Any number of chunks, their scores read again in every pass.
__device__ __forceinline__ void topk_stream(const float *__restrict__ cs, int64_t n_chunks, int64_t k, int chunk, int64_t L,
                                            int32_t *sel, int64_t *__restrict__ spans, int32_t *__restrict__ n_spans)
{
    __shared__ int wave_tot[kTopkThreads / 64];
    const int tid = threadIdx.x;
    const Threshold t = radix_select(k, [&](auto &&f) {
        for (int64_t base = 0; base < n_chunks; base += kTopkThreads) {
            const int64_t i = base + tid;
            f(i < n_chunks ? order_key(cs[i]) : 0u, i < n_chunks);
        }
    });

    // ---- emit kept chunk indices in ascending order ----
    // One scan per segment of a packed pair (above in the low half, equal in the high half) gives each chunk's
    // output position: chunks above before it plus min(equal chunks before it, need).
    int64_t eq_seen = 0, gt_seen = 0;
    for (int64_t base = 0; base < n_chunks; base += kTopkThreads) {
        const int64_t i = base + tid;
        const uint32_t key = i < n_chunks ? order_key(cs[i]) & t.mask : 0u;
        const int is_eq = (i < n_chunks && key == t.prefix) ? 1 : 0;
        const int is_gt = (i < n_chunks && key > t.prefix) ? 1 : 0;
        int total;
        const int incl = block_scan_incl(is_gt | (is_eq << 16), wave_tot, total);
        const int64_t gt_before = gt_seen + (incl & 0xffff) - is_gt;
        const int64_t eq_before = eq_seen + (incl >> 16) - is_eq;
        if (is_gt) sel[gt_before + (eq_before < t.need ? eq_before : t.need)] = (int32_t)i;
        else if (is_eq && eq_before < t.need) sel[gt_before + eq_before] = (int32_t)i;
        gt_seen += total & 0xffff;
        eq_seen += total >> 16;
    }
    __syncthreads();                         // sel[] written by this block is read below

    // ---- merge runs of adjacent kept chunks into token spans ----
    int64_t span_base = 0;
    for (int64_t base = 0; base < k; base += kTopkThreads) {
        const int64_t p = base + tid;
        int start = 0, last = 0;
        int32_t c = 0;
        if (p < k) {
            c = sel[p];
            start = (p == 0) || (sel[p - 1] != c - 1);
            last = (p == k - 1) || (sel[p + 1] != c + 1);
        }
        int tot;
        const int id = block_scan_incl(start, wave_tot, tot);            // 1-based span id of this element
        if (p < k) {
            const int64_t s = span_base + id - 1;
            if (start) spans[2 * s] = (int64_t)c * chunk;
            if (last) {
                const int64_t e = ((int64_t)c + 1) * chunk;
                spans[2 * s + 1] = e < L ? e : L;
            }
        }
        span_base += tot;
    }
    if (tid == 0) *n_spans = (int32_t)span_base;
}

// R > 0: up to R * 1024 chunks; R = 0: any number.
template <int R>
__device__ __forceinline__ void topk_body(const float *__restrict__ cs, int64_t n_chunks, int64_t k,
                                          const int64_t *__restrict__ k_dev, int chunk, int64_t L, int32_t *sel,
                                          int64_t *__restrict__ spans, int32_t *__restrict__ n_spans)
{
    if (k_dev) {                             // k chosen on the device (budget search); always within 1..n_chunks
        k = *k_dev;
        k = k < 1 ? 1 : (k > n_chunks ? n_chunks : k);
    }
    if constexpr (R > 0) topk_words<R>([&](int64_t i) { return cs[i]; }, n_chunks, k, chunk, L, sel, spans, n_spans);
    else topk_stream(cs, n_chunks, k, chunk, L, sel, spans, n_spans);
}

template <int R>
__global__ __launch_bounds__(kTopkThreads) void sp_topk_kernel(const float *__restrict__ cs, int64_t n_chunks,
                                                               int64_t k, const int64_t *__restrict__ k_dev,
                                                               int chunk, int64_t L, int32_t *sel,
                                                               int64_t *__restrict__ spans,
                                                               int32_t *__restrict__ n_spans)
{
    topk_body<R>(cs, n_chunks, k, k_dev, chunk, L, sel, spans, n_spans);
}

// Short prompts: chunk scores and selection by one workgroup, the scores through LDS. At most four chunks a wave.
constexpr int kOneLoads = 4;
constexpr int kOneChunks = kOneLoads * (kTopkThreads / 64);

__device__ __forceinline__ void select_one_body(const float *__restrict__ scores, int64_t L, int pool_w, int chunk,
                                                int64_t n_chunks, int64_t k, float *__restrict__ cs_out, int32_t *__restrict__ sel,
                                                int64_t *__restrict__ spans, int32_t *__restrict__ n_spans)
{
    constexpr int kWaves = kTopkThreads / 64;
    __shared__ float cs[kOneChunks];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    float v[kOneLoads];
    chunk_means<kOneLoads>(scores, L, pool_w, chunk, n_chunks, wave, kWaves, v);
#pragma unroll
    for (int u = 0; u < kOneLoads; ++u)
        if (lane == u && wave + u * kWaves < n_chunks) cs[wave + u * kWaves] = v[u];
    __syncthreads();
    if (cs_out && threadIdx.x < n_chunks) cs_out[threadIdx.x] = cs[threadIdx.x];
    topk_words<1>([&](int64_t i) { return cs[i]; }, n_chunks, k, chunk, L, sel, spans, n_spans);
}

__global__ __launch_bounds__(kTopkThreads) void sp_select_one_kernel(const float *__restrict__ scores, int64_t L, int pool_w,
                                                                     int chunk, int64_t n_chunks, int64_t k,
                                                                     float *__restrict__ cs_out, int32_t *__restrict__ sel,
                                                                     int64_t *__restrict__ spans, int32_t *__restrict__ n_spans)
{
    select_one_body(scores, L, pool_w, chunk, n_chunks, k, cs_out, sel, spans, n_spans);
}

__global__ __launch_bounds__(kTopkThreads) void sp_select_one_batch_kernel(const float *__restrict__ scores,
                                                                           const int64_t *__restrict__ off, int pool_w,
                                                                           const int64_t *__restrict__ kept_off, int chunk,
                                                                           float *__restrict__ cs_out, int32_t *__restrict__ sel,
                                                                           int64_t *__restrict__ spans,
                                                                           int32_t *__restrict__ n_spans)
{
    const int b = blockIdx.x;
    const int64_t o = off[b], L = off[b + 1] - o;
    const int64_t n_chunks = (L + chunk - 1) / chunk;
    const int64_t k0 = kept_off[b];
    int64_t k = kept_off[b + 1] - k0;
    if (n_chunks == 0 || k < 1) {            // uniform
        if (threadIdx.x == 0) n_spans[b] = 0;
        return;
    }
    k = k > n_chunks ? n_chunks : k;
    select_one_body(scores + o, L, pool_w, chunk, n_chunks, k, cs_out ? cs_out + batch_chunk_slot(o, b, chunk) : nullptr, sel + k0,
                    spans + 2 * k0, n_spans + b);
}

// Whether one workgroup does a prompt: a wave takes every 16th chunk, 64 tokens a load. Four loads a wave (2048
// tokens in chunks of 32) take no longer than the two launches on the device and spare the host one of them (1024
// tokens: 6.2 against 6.4 us, called back to back 9.7 against 12.2); sixteen (8192 tokens) take 12.7 against 7.3 us.
bool one_workgroup(int64_t n_chunks, int chunk, int pool_w)
{
    // a chunk is one load at least, so this many loads are kOneChunks chunks at most
    return n_chunks <= kOneChunks && sp::ceil_div(n_chunks, kTopkThreads / 64) * sp::ceil_div((int64_t)chunk + pool_w - 1, 64) <= kOneLoads;
}

// Ragged batch: one workgroup per prompt; prompt b keeps k_b = kept_off[b+1] - kept_off[b] chunks and
// writes its indices and spans from kept_off[b] on. An empty prompt keeps nothing.
template <int R>
__global__ __launch_bounds__(kTopkThreads) void sp_topk_batch_kernel(const float *__restrict__ cs,
                                                                     const int64_t *__restrict__ off,
                                                                     const int64_t *__restrict__ kept_off, int chunk,
                                                                     int32_t *sel, int64_t *__restrict__ spans,
                                                                     int32_t *__restrict__ n_spans)
{
    const int b = blockIdx.x;
    const int64_t o = off[b], L = off[b + 1] - o;
    const int64_t n_chunks = (L + chunk - 1) / chunk;
    const int64_t k0 = kept_off[b];
    int64_t k = kept_off[b + 1] - k0;
    if (n_chunks == 0 || k < 1) {            // uniform
        if (threadIdx.x == 0) n_spans[b] = 0;
        return;
    }
    k = k > n_chunks ? n_chunks : k;
    topk_body<R>(cs + batch_chunk_slot(o, b, chunk), n_chunks, k, nullptr, chunk, L, sel + k0, spans + 2 * k0, n_spans + b);
}

// ---------------------------------------------------------------------------
// budget search
// ---------------------------------------------------------------------------
constexpr int kRankThreads = 256;
constexpr int kMaxBudgetChunks = 1 << 16;

// rank[j] = number of chunks that come before chunk j in the order (score descending, index
// ascending). A workgroup counts, for the THREADS chunks of tile x, the 64 chunks of tile y that come
// before them and adds the counts to rank (cleared beforehand): C^2 comparisons over
// C^2 / (64 THREADS) workgroups (2048 chunks; with square tiles of 256 it took 8.4 us).
constexpr int kRankTile = 64;
template <int THREADS>
__device__ __forceinline__ void rank_tile(const float *__restrict__ cs, int n_chunks, int32_t *__restrict__ rank, int x, int y, uint4 *tile)
{
    const int j = x * THREADS + threadIdx.x;
    const int base = y * kRankTile;
    // entries past the last chunk get key 0, the image of no finite score: they never count
    if (threadIdx.x < kRankTile)
        reinterpret_cast<uint32_t *>(tile)[threadIdx.x] = base + (int)threadIdx.x < n_chunks ? order_key(cs[base + threadIdx.x]) : 0u;
    const uint32_t mine = j < n_chunks ? order_key(cs[j]) : 0u;
    __syncthreads();
    if (j >= n_chunks) return;
    int before = 0;
#pragma unroll
    for (int t = 0; t < kRankTile / 4; ++t) {
        const uint4 o = tile[t];
        const int i0 = base + 4 * t;
        before += (o.x > mine) || (o.x == mine && i0 < j);
        before += (o.y > mine) || (o.y == mine && i0 + 1 < j);
        before += (o.z > mine) || (o.z == mine && i0 + 2 < j);
        before += (o.w > mine) || (o.w == mine && i0 + 3 < j);
    }
    if (before) atomicAdd(&rank[j], before);
}

__global__ __launch_bounds__(kRankThreads) void sp_rank_kernel(const float *__restrict__ cs, int n_chunks,
                                                               int32_t *__restrict__ rank)
{
    __shared__ uint4 tile[kRankTile / 4];
    rank_tile<kRankThreads>(cs, n_chunks, rank, blockIdx.x, blockIdx.y, tile);
}

// First boundary index in [lo, hi] whose offset is > x (STRICT) or >= x; hi + 1 if none.
template <bool STRICT>
__device__ __forceinline__ int first_boundary(const int64_t *bnd, int lo, int hi, int64_t x)
{
    int a = lo, b = hi + 1;
    while (a < b) {
        const int mid = a + ((b - a) >> 1);
        const int64_t e = bnd[mid];
        if (STRICT ? (e > x) : (e >= x)) b = mid; else a = mid + 1;
    }
    return a;
}

// The chunks that decide about a target token of characters [a, b): any(j) is called for each of which one
// has to be selected, or all(j) for each of those that have to be selected together, or neither (kept by no selection).
template <class Any, class All>
__device__ __forceinline__ void deciding_chunks(const int64_t *bnd, int C, int64_t a, int64_t b, const Any &any, const All &all)
{
    if (b > a) {
        // chunks j with a < e[j+1] and b > e[j]: a contiguous range
        for (int j = first_boundary<true>(bnd, 1, C, a) - 1; j < C && bnd[j] < b; ++j) any(j);
        return;
    }
    const int m1 = first_boundary<false>(bnd, 0, C, a);                            // first boundary >= a
    if (m1 > C || m1 < 1) return;
    if (bnd[m1] != a) { any(m1 - 1); return; }                                      // strictly inside chunk m1 - 1
    const int m2 = first_boundary<true>(bnd, m1, C, a) - 1;                         // last boundary == a
    if (m2 < C)
        for (int j = m1 - 1; j <= m2; ++j) all(j);
}

// Neighbouring tokens mostly share their bin: the first lane of every run of equal bins within the
// wave adds the run's length (integer counts: the histogram is the same in any order). bin < 0: no token.
__device__ __forceinline__ void count_runs(int32_t *__restrict__ hist, int bin)
{
    const int lane = threadIdx.x & 63;
    const int prev = __shfl_up(bin, 1);
    const bool leader = lane == 0 || prev != bin;
    const uint64_t leaders = __ballot(leader);
    if (leader && bin >= 0) {
        const uint64_t later = lane == 63 ? 0 : leaders >> (lane + 1);
        const int run = later ? __ffsll((unsigned long long)later) : 64 - lane;
        atomicAdd(&hist[bin], run);
    }
}

constexpr int kTokenThreads = 1024;

// The same for a histogram by chunk: waves that lie within one chunk are added up over the workgroup first. Bins of
// neighbouring chunks share cache lines, so where a chunk has many tokens (12 to a draft token) all workgroups in flight
// add to the same few lines: 1572864 tokens in 1024 chunks 32.3 us a wave at a time, 21.9 this way, 149422 in 2048 13.5 / 13.6.
__device__ __forceinline__ void count_runs_together(int32_t *__restrict__ hist, int bin)
{
    __shared__ int whole[kTokenThreads / 64];
    const int lane = threadIdx.x & 63;
    const int first = __builtin_amdgcn_readfirstlane(bin);
    const bool one = __all(bin == first) && first >= 0;
    if (!one) count_runs(hist, bin);
    if (lane == 0) whole[threadIdx.x >> 6] = one ? first : -1;
    __syncthreads();
    if (threadIdx.x >= 64) return;
    bin = lane < kTokenThreads / 64 ? whole[lane] : -1;
    const int prev = __shfl_up(bin, 1);
    const bool leader = lane == 0 || prev != bin;
    const uint64_t leaders = __ballot(leader);
    if (leader && bin >= 0) atomicAdd(&hist[bin], 64 * (__ffsll((unsigned long long)(leaders >> (lane + 1)))));
}

__global__ __launch_bounds__(kTokenThreads) void sp_token_rank_kernel(const int64_t *__restrict__ bnd, int n_chunks,
                                                                      const int64_t *__restrict__ toff, int64_t M,
                                                                      const int32_t *__restrict__ rank,
                                                                      int32_t *__restrict__ hist)
{
    const int64_t t = (int64_t)blockIdx.x * kTokenThreads + threadIdx.x;
    int r = -1;
    if (t < M) {
        r = n_chunks;                            // kept by no selection
        deciding_chunks(bnd, n_chunks, toff[t], toff[t + 1], [&](int j) { r = min(r, rank[j]); },
                        [&](int j) { r = r == n_chunks ? rank[j] : max(r, rank[j]); });
    }
    count_runs(hist, r);
}

// Ranks and tokens in one launch, up to 8192 chunks: the first `rank_groups` workgroups count ranks, the others a
// histogram of the tokens by the chunk whose rank decides about them. Bound by latency: with the tokens in a launch of
// their own behind the ranks (4.2 and 4.5 us) a cut of 131072 tokens in 2048 chunks took 31.7 us with projection and
// assembly, now 29.9.
// LDS: the boundaries' offsets (up to kLdsBounds of them) are staged, so that the searches do not go to memory for
// every step (2048 chunks: a search is 11 dependent loads).
constexpr int kLdsBounds = 4097;
template <bool LDS>
__global__ __launch_bounds__(kTokenThreads) void sp_rank_tokens_kernel(const float *__restrict__ cs, const int64_t *__restrict__ g_bnd, int n_chunks,
                                                                       const int64_t *__restrict__ toff, int64_t M, int rank_groups,
                                                                       int32_t *__restrict__ rank, int32_t *__restrict__ hist)
{
    __shared__ int64_t s_bnd[LDS ? kLdsBounds : 1];
    __shared__ uint4 tile[kRankTile / 4];
    const int C = n_chunks;
    if ((int)blockIdx.x < rank_groups) {
        const int across = (C + kTokenThreads - 1) / kTokenThreads;
        rank_tile<kTokenThreads>(cs, C, rank, blockIdx.x % across, blockIdx.x / across, tile);
        return;
    }
    const int64_t t = (int64_t)(blockIdx.x - rank_groups) * kTokenThreads + threadIdx.x;
    const bool live = t < M;
    const int64_t a = live ? toff[t] : 0, b = live ? toff[t + 1] : 0;
    if (LDS) {
        for (int i = threadIdx.x; i <= C; i += kTokenThreads) s_bnd[i] = g_bnd[i];
        __syncthreads();
    }
    int bin = -1;
    if (live) {
        bin = C;
        uint32_t key = 0;
        // in ascending order of the chunks: of equal scores the first has the smallest rank and the last the largest
        deciding_chunks(LDS ? s_bnd : g_bnd, C, a, b,
                        [&](int j) { const uint32_t k = order_key(cs[j]); if (bin == C || k > key) { bin = j; key = k; } },
                        [&](int j) { const uint32_t k = order_key(cs[j]); if (bin == C || k <= key) { bin = j; key = k; } });
    }
    count_runs_together(hist, bin);
}

// kept(k) = hist[0] + .. + hist[k-1]; writes the largest k in 1..C with kept(k) <= budget (1 if none)
// and kept at that k.
__global__ __launch_bounds__(kTopkThreads) void sp_budget_kernel(const int32_t *__restrict__ hist, int n_chunks,
                                                                 int64_t budget, int64_t *__restrict__ k_out,
                                                                 int64_t *__restrict__ kept_out)
{
    __shared__ int wave_tot[kTopkThreads / 64];
    __shared__ int s_first;
    const int tid = threadIdx.x;
    int64_t carry = 0, within = 0, kept_within = 0;
    for (int base = 0; base < n_chunks; base += kTopkThreads) {
        const int i = base + tid;
        if (base == 0 && tid == 0) s_first = hist[0];
        const int h = i < n_chunks ? hist[i] : 0;
        int total;
        const int64_t incl = carry + block_scan_incl(h, wave_tot, total);   // kept(i + 1)
        const int ok = (i < n_chunks && incl <= budget) ? 1 : 0;             // a prefix of the k's: kept is monotone
        int ok_total;
        block_scan_incl(ok, wave_tot, ok_total);
        within += ok_total;
        carry += total;
        // kept at the last k within the budget: the largest incl that is <= budget
        int64_t cand = ok ? incl : 0;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const int64_t o = __shfl_xor(cand, off);
            cand = o > cand ? o : cand;
        }
        __shared__ int64_t wave_best[kTopkThreads / 64];
        __syncthreads();
        if ((tid & 63) == 0) wave_best[tid >> 6] = cand;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kTopkThreads / 64; ++w) kept_within = wave_best[w] > kept_within ? wave_best[w] : kept_within;
    }
    if (tid == 0) {
        *k_out = within >= 1 ? within : 1;
        if (kept_out) *kept_out = within >= 1 ? kept_within : (int64_t)s_first;
    }
}

// The same with the selection itself, for up to R * 1024 chunks and a histogram by chunk: chunk i is kept iff
// rank[i] < k. A thread holds the bins of R consecutive ranks, so one block scan does for all of them.
template <int R>
__global__ __launch_bounds__(kTopkThreads) void sp_budget_select_kernel(const int32_t *__restrict__ hist, const int32_t *__restrict__ rank,
                                                                        int n_chunks, int64_t budget, int chunk, int64_t L,
                                                                        int64_t *__restrict__ k_out, int64_t *__restrict__ kept_out,
                                                                        int32_t *__restrict__ sel, int64_t *__restrict__ spans,
                                                                        int32_t *__restrict__ n_spans)
{
    __shared__ int wave_tot[kTopkThreads / 64], wave_ok[kTopkThreads / 64], wave_best[kTopkThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    __shared__ int32_t by_rank[R * kTopkThreads];
    int h[R], mine[R], sum = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * kTopkThreads + tid;
        h[r] = i < n_chunks ? hist[i] : 0;
        mine[r] = i < n_chunks ? rank[i] : n_chunks;
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (mine[r] < n_chunks) by_rank[mine[r]] = h[r];                  // ranks are a permutation of 0 .. n_chunks - 1
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        h[r] = tid * R + r < n_chunks ? by_rank[tid * R + r] : 0;
        sum += h[r];
    }
    int total;
    int kept = block_scan_incl(sum, wave_tot, total) - sum;               // kept(tid * R)
    int ok = 0, best = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        kept += h[r];                                                     // kept(k) is monotone in k
        if (tid * R + r < n_chunks && kept <= budget) { ++ok; best = kept; }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        ok += __shfl_xor(ok, off);
        best = max(best, __shfl_xor(best, off));
    }
    if (lane == 0) { wave_ok[wave] = ok; wave_best[wave] = best; }
    __syncthreads();
    int within = 0, kept_within = 0;
#pragma unroll
    for (int w = 0; w < kTopkThreads / 64; ++w) {
        within += wave_ok[w];
        kept_within = max(kept_within, wave_best[w]);
    }
    const int k = within >= 1 ? within : 1;
    if (tid == 0) {
        *k_out = k;
        if (kept_out) *kept_out = within >= 1 ? kept_within : h[0];
    }
    bool gt[R], eq[R];
#pragma unroll
    for (int r = 0; r < R; ++r) { gt[r] = mine[r] < k; eq[r] = false; }
    emit_kept<R>(gt, eq, 0, chunk, L, sel, spans, n_spans);
}

void launch_topk(hipStream_t st, const float *cs, int64_t C, int64_t k, const int64_t *k_dev, int chunk, int64_t L,
                 int32_t *sel, int64_t *spans, int32_t *n_spans)
{
    const dim3 grid(1), block(kTopkThreads);
    if (C <= 2 * kTopkThreads)
        hipLaunchKernelGGL((sp_topk_kernel<2>), grid, block, 0, st, cs, C, k, k_dev, chunk, L, sel, spans, n_spans);
    else if (C <= 8 * kTopkThreads)
        hipLaunchKernelGGL((sp_topk_kernel<8>), grid, block, 0, st, cs, C, k, k_dev, chunk, L, sel, spans, n_spans);
    else
        hipLaunchKernelGGL((sp_topk_kernel<0>), grid, block, 0, st, cs, C, k, k_dev, chunk, L, sel, spans, n_spans);
}

size_t budget_ws_layout(int64_t C, size_t &off_rank, size_t &off_hist, size_t &off_bnd)
{
    size_t off = sp::align_up(sizeof(float) * (size_t)C, 256);
    off_rank = off; off = sp::align_up(off + sizeof(int32_t) * (size_t)C, 256);
    off_hist = off; off = sp::align_up(off + sizeof(int32_t) * ((size_t)C + 1), 256);
    off_bnd = off;  off = sp::align_up(off + sizeof(int64_t) * ((size_t)C + 1), 256);
    return off;
}

}  // namespace

extern "C" sp_status sp_select_workspace(int64_t L, int32_t chunk, size_t *bytes)
{
    if (!bytes) return sp::fail(SP_ERR_INVALID_ARG, "bytes is null");
    if (L < 1 || chunk < 1) return sp::fail(SP_ERR_INVALID_ARG, "L and chunk must be >= 1");
    const int64_t C = sp::ceil_div(L, chunk);
    *bytes = sp::align_up(sizeof(float) * (size_t)C, 256);
    return SP_OK;
}

namespace {

// Validation shared by the two selection entry points, then the launches; `cs` receives the chunk scores.
sp_status select_check(const float *scores_dev, int64_t L, int32_t pool_w, int32_t chunk, int64_t k,
                       const int32_t *sel_chunks_dev, const int64_t *spans_dev, const int32_t *n_spans_dev, int64_t &C)
{
    if (!scores_dev || !sel_chunks_dev || !spans_dev || !n_spans_dev)
        return sp::fail(SP_ERR_INVALID_ARG, "scores_dev, sel_chunks_dev, spans_dev and n_spans_dev must not be null");
    if (L < 1) return sp::fail(SP_ERR_INVALID_ARG, "L = %lld must be >= 1", (long long)L);
    if (chunk < 1) return sp::fail(SP_ERR_INVALID_ARG, "chunk = %d must be >= 1", chunk);
    if (pool_w < 1 || pool_w % 2 == 0) return sp::fail(SP_ERR_INVALID_ARG, "pool_w = %d must be odd and >= 1", pool_w);
    if (pool_w > kMaxPool) return sp::fail(SP_ERR_UNSUPPORTED, "pool_w = %d (supported: <= %d)", pool_w, kMaxPool);
    C = sp::ceil_div(L, chunk);
    if (C > (1 << 30)) return sp::fail(SP_ERR_UNSUPPORTED, "too many chunks (%lld)", (long long)C);
    if (k < 1 || k > C) return sp::fail(SP_ERR_INVALID_ARG, "k = %lld outside 1..%lld", (long long)k, (long long)C);
    return SP_OK;
}

sp_status select_launch(const float *scores_dev, int64_t L, int32_t pool_w, int32_t chunk, int64_t k, int64_t C,
                        int32_t *sel_chunks_dev, int64_t *spans_dev, int32_t *n_spans_dev, float *chunk_scores_dev,
                        float *cs, hipStream_t st)
{
    if (one_workgroup(C, chunk, pool_w)) {
        hipLaunchKernelGGL(sp_select_one_kernel, dim3(1), dim3(kTopkThreads), 0, st, scores_dev, L, (int)pool_w, (int)chunk, C, k,
                           chunk_scores_dev, sel_chunks_dev, spans_dev, n_spans_dev);
        SP_HIP_CHECK(hipGetLastError());
        return SP_OK;
    }
    const int waves_per_block = kChunkThreads / 64;
    const unsigned grid = (unsigned)((C + waves_per_block - 1) / waves_per_block);
    hipLaunchKernelGGL(sp_chunk_kernel, dim3(grid), dim3(kChunkThreads), 0, st, scores_dev, L, (int)pool_w,
                       (int)chunk, C, cs, chunk_scores_dev, (const int64_t *)nullptr, (int64_t *)nullptr,
                       (int32_t *)nullptr, (int32_t *)nullptr);
    SP_HIP_CHECK(hipGetLastError());
    launch_topk(st, cs, C, k, nullptr, (int)chunk, L, sel_chunks_dev, spans_dev, n_spans_dev);
    SP_HIP_CHECK(hipGetLastError());
    return SP_OK;
}

}  // namespace

extern "C" sp_status sp_select(const float *scores_dev, int64_t L, int32_t pool_w, int32_t chunk, int64_t k,
                               int32_t *sel_chunks_dev, int64_t *spans_dev, int32_t *n_spans_dev,
                               float *chunk_scores_dev, void *ws_dev, size_t ws_bytes, void *hip_stream)
{
    int64_t C = 0;
    const sp_status rc = select_check(scores_dev, L, pool_w, chunk, k, sel_chunks_dev, spans_dev, n_spans_dev, C);
    if (rc != SP_OK) return rc;
    const size_t need = sp::align_up(sizeof(float) * (size_t)C, 256);
    if (!ws_dev) return sp::fail(SP_ERR_WORKSPACE, "ws_dev is null (%zu bytes needed)", need);
    if ((uintptr_t)ws_dev % 256 != 0) return sp::fail(SP_ERR_WORKSPACE, "ws_dev is not 256-byte aligned");
    if (ws_bytes < need) return sp::fail(SP_ERR_WORKSPACE, "workspace too small: %zu < %zu", ws_bytes, need);
    return select_launch(scores_dev, L, pool_w, chunk, k, C, sel_chunks_dev, spans_dev, n_spans_dev, chunk_scores_dev,
                         static_cast<float *>(ws_dev), static_cast<hipStream_t>(hip_stream));
}

// ---------------------------------------------------------------------------
// sp_select for a ragged batch: one launch for prompts of a few chunks, two otherwise.
// ---------------------------------------------------------------------------
namespace {
constexpr int kMaxBatchPrompts = 4096;

size_t select_batch_ws(int64_t total, int32_t B, int32_t chunk)
{
    return sp::align_up(sizeof(float) * (size_t)(total / chunk + B + 1), 256);
}
}  // namespace

extern "C" sp_status sp_select_batch_workspace(int64_t total_tokens, int32_t B, int32_t chunk, size_t *bytes)
{
    if (!bytes) return sp::fail(SP_ERR_INVALID_ARG, "bytes is null");
    if (total_tokens < 0 || chunk < 1 || B < 1 || B > kMaxBatchPrompts)
        return sp::fail(SP_ERR_INVALID_ARG, "total_tokens >= 0, chunk >= 1 and B in 1..%d are required", kMaxBatchPrompts);
    if (total_tokens / chunk > (int64_t(1) << 42))       // 4096 prompts of 2^30 chunks: what sp_select_batch accepts at most
        return sp::fail(SP_ERR_UNSUPPORTED, "too many chunks (%lld)", (long long)(total_tokens / chunk));
    *bytes = select_batch_ws(total_tokens, B, chunk);
    return SP_OK;
}

extern "C" sp_status sp_select_batch(const float *scores_dev, const int64_t *offsets_host, const int64_t *offsets_dev,
                                     int32_t B, int32_t pool_w, int32_t chunk, const int64_t *kept_off_host,
                                     const int64_t *kept_off_dev, int32_t *sel_chunks_dev, int64_t *spans_dev,
                                     int32_t *n_spans_dev, float *chunk_scores_dev, void *ws_dev, size_t ws_bytes,
                                     void *hip_stream)
{
    if (!scores_dev || !offsets_host || !offsets_dev || !kept_off_host || !kept_off_dev || !sel_chunks_dev || !spans_dev ||
        !n_spans_dev)
        return sp::fail(SP_ERR_INVALID_ARG, "only chunk_scores_dev may be null");
    if (B < 1 || B > kMaxBatchPrompts) return sp::fail(SP_ERR_INVALID_ARG, "B = %d (supported: 1..%d)", B, kMaxBatchPrompts);
    if (chunk < 1) return sp::fail(SP_ERR_INVALID_ARG, "chunk = %d must be >= 1", chunk);
    if (pool_w < 1 || pool_w % 2 == 0) return sp::fail(SP_ERR_INVALID_ARG, "pool_w = %d must be odd and >= 1", pool_w);
    if (pool_w > kMaxPool) return sp::fail(SP_ERR_UNSUPPORTED, "pool_w = %d (supported: <= %d)", pool_w, kMaxPool);
    if (offsets_host[0] != 0 || kept_off_host[0] != 0)
        return sp::fail(SP_ERR_INVALID_ARG, "offsets_host[0] and kept_off_host[0] must be 0");
    int64_t max_chunks = 0;
    for (int b = 0; b < B; ++b) {
        const int64_t len = offsets_host[b + 1] - offsets_host[b], k = kept_off_host[b + 1] - kept_off_host[b];
        if (len < 0) return sp::fail(SP_ERR_INVALID_ARG, "offsets_host decreases at prompt %d", b);
        const int64_t C = sp::ceil_div(len, chunk);
        if (C > (1 << 30)) return sp::fail(SP_ERR_UNSUPPORTED, "too many chunks (%lld) in prompt %d", (long long)C, b);
        if (len == 0 ? k != 0 : (k < 1 || k > C))
            return sp::fail(SP_ERR_INVALID_ARG, "prompt %d keeps %lld chunks of %lld (1..C, or 0 of an empty prompt)", b,
                            (long long)k, (long long)C);
        max_chunks = std::max(max_chunks, C);
    }
    const size_t need = select_batch_ws(offsets_host[B], B, chunk);
    if (!ws_dev) return sp::fail(SP_ERR_WORKSPACE, "ws_dev is null (%zu bytes needed)", need);
    if ((uintptr_t)ws_dev % 256 != 0) return sp::fail(SP_ERR_WORKSPACE, "ws_dev is not 256-byte aligned");
    if (ws_bytes < need) return sp::fail(SP_ERR_WORKSPACE, "workspace too small: %zu < %zu", ws_bytes, need);
    if (max_chunks == 0) max_chunks = 1;     // all prompts empty: the top-k launch still writes n_spans = 0
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    float *cs = static_cast<float *>(ws_dev);
    if (one_workgroup(max_chunks, chunk, pool_w)) {
        hipLaunchKernelGGL(sp_select_one_batch_kernel, dim3((unsigned)B), dim3(kTopkThreads), 0, st, scores_dev, offsets_dev,
                           (int)pool_w, kept_off_dev, (int)chunk, chunk_scores_dev, sel_chunks_dev, spans_dev, n_spans_dev);
        SP_HIP_CHECK(hipGetLastError());
        return SP_OK;
    }
    const int waves_per_block = kChunkThreads / 64;
    hipLaunchKernelGGL(sp_chunk_batch_kernel, dim3((unsigned)sp::ceil_div(max_chunks, waves_per_block), (unsigned)B),
                       dim3(kChunkThreads), 0, st, scores_dev, offsets_dev, (int)pool_w, (int)chunk, cs, chunk_scores_dev);
    SP_HIP_CHECK(hipGetLastError());
    const dim3 grid((unsigned)B), block(kTopkThreads);
    if (max_chunks <= 2 * kTopkThreads)
        hipLaunchKernelGGL((sp_topk_batch_kernel<2>), grid, block, 0, st, cs, offsets_dev, kept_off_dev, (int)chunk,
                           sel_chunks_dev, spans_dev, n_spans_dev);
    else if (max_chunks <= 8 * kTopkThreads)
        hipLaunchKernelGGL((sp_topk_batch_kernel<8>), grid, block, 0, st, cs, offsets_dev, kept_off_dev, (int)chunk,
                           sel_chunks_dev, spans_dev, n_spans_dev);
    else
        hipLaunchKernelGGL((sp_topk_batch_kernel<0>), grid, block, 0, st, cs, offsets_dev, kept_off_dev, (int)chunk,
                           sel_chunks_dev, spans_dev, n_spans_dev);
    SP_HIP_CHECK(hipGetLastError());
    return SP_OK;
}

// ---------------------------------------------------------------------------
// sp_select without a workspace argument, for callers that cannot allocate: the
// chunk scores go to a device array that is part of the library's image.
// ---------------------------------------------------------------------------
constexpr int64_t kStaticChunks = SP_SELECT_STATIC_MAX_CHUNKS;
static __device__ __align__(256) float scratch[kStaticChunks];

namespace {

constexpr int kMaxDevices = 64;
// Device address of `scratch` on each device, resolved once per device with that device current.
// (In host code the array's name only stands for the symbol; it is not a device address.)
std::atomic<float *> g_scratch[kMaxDevices];

sp_status scratch_of_current_device(float *&out)
{
    int dev = -1;
    SP_HIP_CHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return sp::fail(SP_ERR_UNSUPPORTED, "device index %d (supported: < %d)", dev, kMaxDevices);
    float *p = g_scratch[dev].load(std::memory_order_acquire);
    if (!p) {
        void *sym = nullptr;
        SP_HIP_CHECK(hipGetSymbolAddress(&sym, HIP_SYMBOL(scratch)));
        if (!sym) return sp::fail(SP_ERR_DEVICE, "the library's scratch array has no address on device %d", dev);
        p = static_cast<float *>(sym);
        g_scratch[dev].store(p, std::memory_order_release);     // every thread resolves the same address
    }
    out = p;
    return SP_OK;
}

}  // namespace

extern "C" sp_status sp_select_static(const float *scores_dev, int64_t L, int32_t pool_w, int32_t chunk, int64_t k,
                                      int32_t *sel_chunks_dev, int64_t *spans_dev, int32_t *n_spans_dev,
                                      float *chunk_scores_dev, void *hip_stream)
{
    int64_t C = 0;
    const sp_status rc = select_check(scores_dev, L, pool_w, chunk, k, sel_chunks_dev, spans_dev, n_spans_dev, C);
    if (rc != SP_OK) return rc;
    if (C > kStaticChunks)
        return sp::fail(SP_ERR_UNSUPPORTED, "%lld chunks exceed the %lld the library's own scratch array holds; use sp_select",
                        (long long)C, (long long)kStaticChunks);
    float *cs = nullptr;
    const sp_status rs = scratch_of_current_device(cs);
    if (rs != SP_OK) return rs;
    // every chunk score the top-k kernel reads is written by the chunk kernel of this call: nothing to clear
    return select_launch(scores_dev, L, pool_w, chunk, k, C, sel_chunks_dev, spans_dev, n_spans_dev, chunk_scores_dev, cs,
                         static_cast<hipStream_t>(hip_stream));
}

extern "C" sp_status sp_select_budget_workspace(int64_t L, int32_t chunk, size_t *bytes)
{
    if (!bytes) return sp::fail(SP_ERR_INVALID_ARG, "bytes is null");
    if (L < 1 || chunk < 1) return sp::fail(SP_ERR_INVALID_ARG, "L and chunk must be >= 1");
    const int64_t C = sp::ceil_div(L, chunk);
    if (C > kMaxBudgetChunks)
        return sp::fail(SP_ERR_UNSUPPORTED, "%lld chunks (the budget search supports <= %d)", (long long)C, kMaxBudgetChunks);
    size_t a, b, c;
    *bytes = budget_ws_layout(C, a, b, c);
    return SP_OK;
}

extern "C" sp_status sp_select_budget(const float *scores_dev, int64_t L, int32_t pool_w, int32_t chunk,
                                      const int64_t *draft_off_dev, const int64_t *target_off_dev, int64_t M,
                                      int64_t budget, int32_t *sel_chunks_dev, int64_t *spans_dev,
                                      int32_t *n_spans_dev, int64_t *k_dev, int64_t *n_kept_dev,
                                      float *chunk_scores_dev, void *ws_dev, size_t ws_bytes, void *hip_stream)
{
    if (!scores_dev || !draft_off_dev || !target_off_dev || !sel_chunks_dev || !spans_dev || !n_spans_dev || !k_dev)
        return sp::fail(SP_ERR_INVALID_ARG, "only n_kept_dev and chunk_scores_dev may be null");
    if (L < 1 || M < 1) return sp::fail(SP_ERR_INVALID_ARG, "L = %lld and M = %lld must be >= 1", (long long)L, (long long)M);
    if (chunk < 1) return sp::fail(SP_ERR_INVALID_ARG, "chunk = %d must be >= 1", chunk);
    if (pool_w < 1 || pool_w % 2 == 0) return sp::fail(SP_ERR_INVALID_ARG, "pool_w = %d must be odd and >= 1", pool_w);
    if (pool_w > kMaxPool) return sp::fail(SP_ERR_UNSUPPORTED, "pool_w = %d (supported: <= %d)", pool_w, kMaxPool);
    if (budget < 0) return sp::fail(SP_ERR_INVALID_ARG, "budget = %lld is negative", (long long)budget);
    if (M >= (int64_t(1) << 31)) return sp::fail(SP_ERR_UNSUPPORTED, "M = %lld (supported: < 2^31)", (long long)M);
    const int64_t C = sp::ceil_div(L, chunk);
    if (C > kMaxBudgetChunks)
        return sp::fail(SP_ERR_UNSUPPORTED, "%lld chunks (the budget search supports <= %d)", (long long)C, kMaxBudgetChunks);
    size_t off_rank, off_hist, off_bnd;
    const size_t need = budget_ws_layout(C, off_rank, off_hist, off_bnd);
    if (!ws_dev) return sp::fail(SP_ERR_WORKSPACE, "ws_dev is null (%zu bytes needed)", need);
    if ((uintptr_t)ws_dev % 256 != 0) return sp::fail(SP_ERR_WORKSPACE, "ws_dev is not 256-byte aligned");
    if (ws_bytes < need) return sp::fail(SP_ERR_WORKSPACE, "workspace too small: %zu < %zu", ws_bytes, need);

    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    char *ws = static_cast<char *>(ws_dev);
    float *cs = reinterpret_cast<float *>(ws);
    int32_t *rank = reinterpret_cast<int32_t *>(ws + off_rank);
    int32_t *hist = reinterpret_cast<int32_t *>(ws + off_hist);
    int64_t *bnd = reinterpret_cast<int64_t *>(ws + off_bnd);
    const int waves_per_block = kChunkThreads / 64;
    hipLaunchKernelGGL(sp_chunk_kernel, dim3((unsigned)((C + waves_per_block - 1) / waves_per_block)),
                       dim3(kChunkThreads), 0, st, scores_dev, L, (int)pool_w, (int)chunk, C, cs, chunk_scores_dev,
                       draft_off_dev, bnd, rank, hist);
    SP_HIP_CHECK(hipGetLastError());
    if (C <= 8 * kTopkThreads) {
        const int64_t rank_groups = sp::ceil_div(C, kTokenThreads) * sp::ceil_div(C, kRankTile), token_groups = sp::ceil_div(M, kTokenThreads);
        const auto rank_tokens = C < kLdsBounds ? sp_rank_tokens_kernel<true> : sp_rank_tokens_kernel<false>;
        hipLaunchKernelGGL(rank_tokens, dim3((unsigned)(rank_groups + token_groups)), dim3(kTokenThreads), 0, st, (const float *)cs,
                           (const int64_t *)bnd, (int)C, target_off_dev, M, (int)rank_groups, rank, hist);
        SP_HIP_CHECK(hipGetLastError());
        const auto budget_select = C <= 2 * kTopkThreads ? sp_budget_select_kernel<2> : sp_budget_select_kernel<8>;
        hipLaunchKernelGGL(budget_select, dim3(1), dim3(kTopkThreads), 0, st, (const int32_t *)hist, (const int32_t *)rank, (int)C,
                           budget, (int)chunk, L, k_dev, n_kept_dev, sel_chunks_dev, spans_dev, n_spans_dev);
        SP_HIP_CHECK(hipGetLastError());
        return SP_OK;
    }
    hipLaunchKernelGGL(sp_rank_kernel, dim3((unsigned)sp::ceil_div(C, kRankThreads), (unsigned)sp::ceil_div(C, kRankTile)),
                       dim3(kRankThreads), 0, st, (const float *)cs, (int)C, rank);
    SP_HIP_CHECK(hipGetLastError());
    hipLaunchKernelGGL(sp_token_rank_kernel, dim3((unsigned)sp::ceil_div(M, kTokenThreads)), dim3(kTokenThreads), 0, st,
                       (const int64_t *)bnd, (int)C, target_off_dev, M, (const int32_t *)rank, hist);
    SP_HIP_CHECK(hipGetLastError());
    hipLaunchKernelGGL(sp_budget_kernel, dim3(1), dim3(kTopkThreads), 0, st, (const int32_t *)hist, (int)C, budget, k_dev,
                       n_kept_dev);
    SP_HIP_CHECK(hipGetLastError());
    launch_topk(st, cs, C, 1, k_dev, (int)chunk, L, sel_chunks_dev, spans_dev, n_spans_dev);
    SP_HIP_CHECK(hipGetLastError());
    return SP_OK;
}
