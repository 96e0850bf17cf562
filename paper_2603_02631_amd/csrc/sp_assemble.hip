// sp_assemble: token ids and position ids of the compressed target prompt
// (paper: Algorithm 1 "ConcatWithDelim", the target tokenisation of the
// compressed text and the new contiguous position ids; Section 3.2).
//
// The kept target ranges are copied in order with the delimiter's ids between
// consecutive ranges. Range r occupies one block of the output: its delimiter
// (for r > 0) followed by its tokens.
//
// Buffers of up to 2048 ranges and 2^19 output entries take one launch, sp_assemble_one_kernel: every
// workgroup prefix-sums the block lengths for itself (a few KB out of the caches)
// into LDS, then one thread per output entry binary-searches the block starts
// there and copies a delimiter id or a token id. More take two launches:
//   sp_assemble_offsets_kernel  one workgroup: exclusive prefix sum of the block
//                               lengths -> block starts (workspace), total length.
//   sp_assemble_gather_kernel   one thread per output entry, as above on the
//                               starts in the workspace.
#include "sp_common.hpp"

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

__device__ __forceinline__ int64_t clamp64(int64_t v, int64_t lo, int64_t hi) { return v < lo ? lo : (v > hi ? hi : v); }

// Block starts of n ranges by one workgroup of THREADS: block_start[0 .. n], the last one the total length.
template <int THREADS>
__device__ __forceinline__ int64_t block_starts(const int64_t *__restrict__ tspans, int n, int64_t M, int n_delim,
                                                int64_t *block_start, int64_t (&wave_tot)[THREADS / 64])
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int64_t carry = 0;
    for (int base = 0; base < n; base += THREADS) {
        const int r = base + tid;
        int64_t len = 0;
        if (r < n) {
            const int64_t b = clamp64(tspans[2 * r], 0, M), e = clamp64(tspans[2 * r + 1], b, M);
            len = (e - b) + (r > 0 ? n_delim : 0);
        }
        int64_t x = len;                    // inclusive scan within the wave
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int64_t y = __shfl_up(x, off);
            if (lane >= off) x += y;
        }
        __syncthreads();                    // wave_tot of the previous segment has been read
        if (lane == 63) wave_tot[wave] = x;
        __syncthreads();
        int64_t before = 0, total = 0;
#pragma unroll
        for (int w = 0; w < THREADS / 64; ++w) {
            if (w < wave) before += wave_tot[w];
            total += wave_tot[w];
        }
        if (r < n) block_start[r] = carry + before + x - len;
        carry += total;
    }
    if (tid == 0) block_start[n] = carry;   // sentinel: one past the last block
    return carry;
}

// Output entry i of the n blocks that start at block_start.
__device__ __forceinline__ void gather_entry(int64_t i, const int64_t *block_start, int n, const int32_t *__restrict__ target_ids,
                                             int64_t M, const int64_t *__restrict__ tspans, const int32_t *__restrict__ delim,
                                             int n_delim, int32_t *__restrict__ out_ids, int32_t *__restrict__ out_pos,
                                             int64_t *__restrict__ out_src)
{
    // last block whose start is <= i
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = lo + ((hi - lo) >> 1);
        if (block_start[mid] <= i) lo = mid + 1; else hi = mid;
    }
    const int r = lo - 1;
    int64_t j = i - block_start[r];
    int32_t id;
    int64_t src;
    if (r > 0 && j < n_delim) {
        id = delim[j];
        src = -1;
    } else {
        if (r > 0) j -= n_delim;
        src = clamp64(tspans[2 * r], 0, M) + j;
        id = target_ids[src];
    }
    out_ids[i] = id;
    out_pos[i] = (int32_t)i;
    if (out_src) out_src[i] = src;
}

__global__ __launch_bounds__(kThreads) void sp_assemble_offsets_kernel(const int64_t *__restrict__ tspans,
                                                                       const int32_t *__restrict__ n_tspans_p,
                                                                       int max_spans, int64_t M, int n_delim,
                                                                       int64_t *__restrict__ block_start,
                                                                       int64_t *__restrict__ out_len)
{
    __shared__ int64_t wave_tot[kWaves];
    int n = *n_tspans_p;
    n = n < 0 ? 0 : (n > max_spans ? max_spans : n);
    const int64_t total = block_starts<kThreads>(tspans, n, M, n_delim, block_start, wave_tot);
    if (threadIdx.x == 0) *out_len = total;
}

__global__ __launch_bounds__(kThreads) void sp_assemble_gather_kernel(const int32_t *__restrict__ target_ids, int64_t M,
                                                                      const int64_t *__restrict__ tspans,
                                                                      const int32_t *__restrict__ n_tspans_p,
                                                                      int max_spans,
                                                                      const int32_t *__restrict__ delim, int n_delim,
                                                                      const int64_t *__restrict__ block_start,
                                                                      int64_t out_capacity, int32_t *__restrict__ out_ids,
                                                                      int32_t *__restrict__ out_pos,
                                                                      int64_t *__restrict__ out_src)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    int n = *n_tspans_p;
    n = n < 0 ? 0 : (n > max_spans ? max_spans : n);
    if (i >= block_start[n] || i >= out_capacity) return;
    gather_entry(i, block_start, n, target_ids, M, tspans, delim, n_delim, out_ids, out_pos, out_src);
}

// One launch: bound by its chain of round trips (count, ranges, scan, search, id), five instead of eight and a
// launch: 5.9 us for the two on 163 ranges and 16384 tokens.
constexpr int kOneThreads = 1024;
constexpr int kOneSpans = 2048;
constexpr int64_t kOneEntries = 1 << 19;        // as many workgroups as are resident at once, each with a scan of its own first
__global__ __launch_bounds__(kOneThreads) void sp_assemble_one_kernel(const int32_t *__restrict__ target_ids, int64_t M,
                                                                      const int64_t *__restrict__ tspans,
                                                                      const int32_t *__restrict__ n_tspans_p,
                                                                      int max_spans,
                                                                      const int32_t *__restrict__ delim, int n_delim,
                                                                      int64_t out_capacity, int32_t *__restrict__ out_ids,
                                                                      int32_t *__restrict__ out_pos,
                                                                      int64_t *__restrict__ out_src,
                                                                      int64_t *__restrict__ out_len)
{
    __shared__ int64_t wave_tot[kOneThreads / 64];
    __shared__ int64_t block_start[kOneSpans + 1];
    int n = *n_tspans_p;
    n = n < 0 ? 0 : (n > max_spans ? max_spans : n);
    const int64_t total = block_starts<kOneThreads>(tspans, n, M, n_delim, block_start, wave_tot);
    if (blockIdx.x == 0 && threadIdx.x == 0) *out_len = total;
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * kOneThreads + threadIdx.x;
    if (i >= total || i >= out_capacity) return;
    gather_entry(i, block_start, n, target_ids, M, tspans, delim, n_delim, out_ids, out_pos, out_src);
}

size_t workspace_need(int32_t max_spans) { return sp::align_up(sizeof(int64_t) * ((size_t)max_spans + 1), 256); }

}  // namespace

extern "C" sp_status sp_assemble_workspace(int32_t max_spans, size_t *bytes)
{
    if (!bytes) return sp::fail(SP_ERR_INVALID_ARG, "bytes is null");
    if (max_spans < 1 || max_spans > (1 << 24))
        return sp::fail(SP_ERR_INVALID_ARG, "max_spans = %d outside 1..2^24", max_spans);
    *bytes = workspace_need(max_spans);
    return SP_OK;
}

extern "C" sp_status sp_assemble(const int32_t *target_ids_dev, int64_t M, const int64_t *tspans_dev,
                                 const int32_t *n_tspans_dev, int32_t max_spans, const int32_t *delim_ids_dev,
                                 int32_t n_delim, int64_t out_capacity, int32_t *out_ids_dev, int32_t *out_pos_dev,
                                 int64_t *out_src_dev, int64_t *out_len_dev, void *ws_dev, size_t ws_bytes,
                                 void *hip_stream)
{
    if (!target_ids_dev || !tspans_dev || !n_tspans_dev || !out_ids_dev || !out_pos_dev || !out_len_dev)
        return sp::fail(SP_ERR_INVALID_ARG, "only delim_ids_dev (with n_delim = 0) and out_src_dev may be null");
    if (M < 1) return sp::fail(SP_ERR_INVALID_ARG, "M = %lld must be >= 1", (long long)M);
    if (max_spans < 1 || max_spans > (1 << 24))
        return sp::fail(SP_ERR_INVALID_ARG, "max_spans = %d outside 1..2^24", max_spans);
    if (n_delim < 0 || n_delim > 1024) return sp::fail(SP_ERR_INVALID_ARG, "n_delim = %d outside 0..1024", n_delim);
    if (n_delim > 0 && !delim_ids_dev) return sp::fail(SP_ERR_INVALID_ARG, "delim_ids_dev is null with n_delim = %d", n_delim);
    if (out_capacity < 1 || out_capacity >= (int64_t(1) << 31))
        return sp::fail(SP_ERR_INVALID_ARG, "out_capacity = %lld outside 1..2^31-1", (long long)out_capacity);
    const size_t need = workspace_need(max_spans);
    if (!ws_dev) return sp::fail(SP_ERR_WORKSPACE, "ws_dev is null (%zu bytes needed)", need);
    if ((uintptr_t)ws_dev % 256 != 0) return sp::fail(SP_ERR_WORKSPACE, "ws_dev is not 256-byte aligned");
    if (ws_bytes < need) return sp::fail(SP_ERR_WORKSPACE, "workspace too small: %zu < %zu", ws_bytes, need);

    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    int64_t *block_start = static_cast<int64_t *>(ws_dev);
    // the output cannot be longer than every target token plus a delimiter per range
    int64_t bound = M + (int64_t)(max_spans - 1) * n_delim;
    if (bound > out_capacity) bound = out_capacity;
    if (max_spans <= kOneSpans && bound <= kOneEntries) {
        hipLaunchKernelGGL(sp_assemble_one_kernel, dim3((unsigned)sp::ceil_div(bound, kOneThreads)), dim3(kOneThreads), 0, st,
                           target_ids_dev, M, tspans_dev, n_tspans_dev, (int)max_spans, delim_ids_dev, (int)n_delim,
                           out_capacity, out_ids_dev, out_pos_dev, out_src_dev, out_len_dev);
        SP_HIP_CHECK(hipGetLastError());
        return SP_OK;
    }
    hipLaunchKernelGGL(sp_assemble_offsets_kernel, dim3(1), dim3(kThreads), 0, st, tspans_dev, n_tspans_dev,
                       (int)max_spans, M, (int)n_delim, block_start, out_len_dev);
    SP_HIP_CHECK(hipGetLastError());
    const unsigned grid = (unsigned)((bound + kThreads - 1) / kThreads);
    hipLaunchKernelGGL(sp_assemble_gather_kernel, dim3(grid), dim3(kThreads), 0, st, target_ids_dev, M, tspans_dev,
                       n_tspans_dev, (int)max_spans, delim_ids_dev, (int)n_delim, (const int64_t *)block_start,
                       out_capacity, out_ids_dev, out_pos_dev, out_src_dev);
    SP_HIP_CHECK(hipGetLastError());
    return SP_OK;
}
