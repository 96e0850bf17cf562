// Host interface of the fused single-launch score kernel (see sp_score_fused.hip).
#pragma once

#include "sp_common.hpp"
#include "sp_score_dev.hpp"

namespace sp_fused {

constexpr int kTileKeys = 512;   // keys owned by one workgroup at head_dim 64; 256 at head_dim 128
constexpr int kMaxRowsWide = 32; // head_dim 128, one block of query rows (bf16 keys take two as well: fused_big)
constexpr int kMaxRows = 64;     // padded query rows per kv head the kernel holds on chip
constexpr int kSlots = 8;        // depth of the exchange ring
constexpr int kDutyRows = 4;     // consecutive query rows one workgroup's duty covers
// Fewest workgroups with all layers in one range; shorter prompts (of captured calls, for instance) take the three kernels.
// Three kernels / single launch, us: 16 x 8 heads of 64, 16384 tokens 100 / 243, 28672 184 / 241, 32768 (64 workgroups) 202 /
// 239; 28 x 8 heads of 128, 12288 tokens 296 / 386, 16384 387 / 385, 24576 (96 workgroups) 537 / 400.
constexpr int kMinWorkgroups = 64;       // head_dim 64
constexpr int kMinWorkgroupsWide = 96;   // head_dim 128
constexpr int kMaxGroup = 64;          // entries of a launch's table

// The (prompt, layer range) pairs that share a launch. Entry i scores layers layer0[i] .. layer0[i] +
// layers[i] - 1 of prompt `prompt[i]` of the batch (its queries), whose keys are [start[i], start[i] +
// len[i]) of the packed key arrays (shorter than a tile only where duties are not shared), on workgroups
// w0[i] .. w0[i+1]-1. An entry is on its own in everything: its partials are combined among its workgroups and it has its own row of
// normalisers. n == 0: all layers of a single prompt described by FusedArgs::L.
// An entry has at least as many workgroups as duty blocks (rows_pad / kDutyRows) or few enough for
// every one to combine all partials by itself (direct_max), so any number does.
// 32-bit fields only: a smaller one would be read with a vector load, which the kernel's exact
// counting of vector-memory operations does not know about.
struct GroupTable {
    int32_t n;
    int32_t w0[kMaxGroup + 1];
    int32_t prompt[kMaxGroup];
    int32_t layer0[kMaxGroup];
    int32_t layers[kMaxGroup];
    int32_t slice[kMaxGroup];       // which row (MEAN) or rows (MAX) of split_out the entry fills
    int32_t len[kMaxGroup];
    int64_t start[kMaxGroup];
};

struct FusedArgs {
    const uint16_t *q;           // [Lyr][H][n_q][head_dim]
    int32_t head_dim;            // 64 or 128
    int32_t tile_keys;           // keys per workgroup: 512 at head_dim 64, 256 at head_dim 128, or two such tiles
    int64_t k_stride_token, k_stride_head;
    int64_t L;
    uint64_t *part;              // [kSlots][n_wg][rows_pad]  (max, sum exp) partials, parity in bit 63
    uint64_t *lse;               // [kSlots][rows_pad]        (-lse, phase + 1)
    uint32_t *err;               // the call's status word: raised by any workgroup whose bounded wait gave up
    uint32_t spin_max;           // polls before a wait gives up
    int32_t force_miss;          // test hook: duty waves treat partials as never arriving
    const float *kscale;         // 8-bit keys (E4M3 codes): [n_phases] scale of each (layer, kv head); null: bf16 keys
    const float *look;           // [n_phases][rows_pad] log-sum-exp of each row over its visible lookahead keys
                                 // (raw-logit units, -inf for none), or null: prompt keys only
    const int32_t *block_table;  // paged keys: token j of a layer sits in page block_table[j / page_tokens] of that
    int64_t page_tokens;         // layer's pool, page p at element offset p * page_stride; null: contiguous keys
    int64_t page_stride;
    float *scores;
    float *split_out;            // layers in ranges: results per range instead of scores (see sp_split_reduce_kernel), or null
    int64_t split_stride;        // tokens of the whole call: one row of split_out
    int32_t n_wg;
    int32_t n_gp, p_idx;         // set in the kernel: entries of the launch, this workgroup's entry among them,
    int32_t ent_w0, ent_n;       // its first workgroup and number of workgroups,
    int32_t phase0, last_layer;  // first phase, layer after which an open maximum is closed
    int32_t n_layers, n_q_heads, n_kv_heads, group, n_q;
    int32_t n_nblk, n_gblk, rows_pad;
    int32_t layer_agg;
    float c, inv_c, out_scale;
};

// 8-byte words of the exchange area of a launch of n_wg workgroups and n_entries entries (one prompt: 1).
inline size_t exchange_words(int rows_pad, int n_wg, int n_entries) { return (size_t)kSlots * rows_pad * (n_wg + n_entries); }
inline size_t workspace_bytes(int rows_pad, int n_wg, int n_entries)
{
    return sp::align_up(sizeof(uint64_t) * exchange_words(rows_pad, n_wg, n_entries), 256);
}

// What the launch has to clear first: the exchange area and the status word (the first launch of a call), the area
// only, or nothing, when an earlier launch on the stream has cleared both.
enum class Clear { kAll, kExchange, kDone };

// Entries of fewer workgroups than duty blocks exchange directly: every workgroup combines all partials of
// its entry by itself. Only those: at 16 or 32 workgroups an entry the extra loads (8 KB a workgroup and phase
// past the caches) cost more than the saved round trip (8192 tokens, 16 layers x 8 kv heads, head_dim 64:
// 47 us against 43; 28 x 8, head_dim 128: 130 us against 102).
constexpr int direct_max(int rows_pad) { return rows_pad / kDutyRows - 1; }

// True when the device can hold one workgroup of the fused kernel per compute unit.
bool fits_one_per_cu();

// Enqueues the clear kernel, as far as `clear` asks for it, and the fused kernel. `ws` must hold workspace_bytes();
// `status_word` (device) is raised if the call gives up, after at most `a.spin_max` polls in a wait.
// `group` (or null for one prompt) describes the entries of the launch.
// `shared`: the duties rotate over all workgroups of the launch (whole prompts of at least a tile only, at
// least as many workgroups as duty blocks); otherwise every entry keeps to itself.
sp_status launch(FusedArgs a, const sp_dev::LayerPtrs &kp, const GroupTable *group, bool shared, Clear clear, void *ws,
                 uint32_t *status_word, hipStream_t st);

// Polls (about 30 ms) after which a launch gives up that a later launch can stand in for: early, so that it frees its
// compute units for a launch that nothing stands in for, and late enough for the workgroups of ordinary kernels to leave.
constexpr uint32_t kYieldSpins = 1u << 15;

// Test hook: polls before a bounded wait gives up (default 2^20) and whether duty waves treat their
// partials as never arriving or launches lack a workgroup; applies to launches that follow.
void set_giveup(uint32_t spin_max, int32_t force_miss);

}  // namespace sp_fused
