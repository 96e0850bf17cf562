// Host-side choices of the score calls: layer ranges, how a ragged batch is packed into launches of the single-launch
// kernel, and where the three-kernel path is left for it. Arithmetic only: what the device and the workspace have room
// for comes in as numbers.
#pragma once

#include "sp_score_fused.hpp"

#include <algorithm>
#include <cstring>
#include <functional>
#include <queue>
#include <utility>
#include <vector>

namespace sp_plan {

constexpr int kMaxUnits = 256;             // workgroups of a launch, whatever the device has
constexpr int kMaxGroupPrompts = 32;       // prompts one launch of the fused kernel serves

struct Plan {
    int D, NS, NB, n_gblk, rows_pad, tile_keys, n_phases, n_layers, layer_agg;
    size_t lds_bytes;
};

// Two blocks of query rows at head_dim 128 (bf16 keys, one tile a workgroup or two): their exchange area always takes the
// place of the general path's buffers, so the workspace is as large as without them.
inline bool fused_big(const Plan &p) { return p.D == 128 && p.NB == 1 && p.n_gblk == 2; }

// Keys a workgroup of the fused kernel owns: 512 at head_dim 64, 256 at head_dim 128 (twice the tile of
// the two-pass path).
inline int fused_tile(const Plan &p) { return p.D == 64 ? sp_fused::kTileKeys : sp_fused::kTileKeys / 2; }

constexpr int kProbTargetWgs = 1024;       // the prob pass splits layers until it has about this many workgroups

// Layers per workgroup of the prob pass: all of them once the tiles alone fill the device, and where a workgroup gets through
// all phases of a short prompt in less time than the launch that adds up the ranges takes. A phase costs it as much for
// every block of 32 padded query rows; the launch costs more with the maximum over layers, since it adds up 8 or 16 rows of maxima.
// Score calls with ranges and without, us: 32 rows, four phases of head_dim 64, 1 tile 14.6 / 12.0, 12 14.9 / 13.6, 24 15.0 / 13.9,
// of 128, 1 14.4 / 13.5, 20 15.0 / 15.2; 64 rows, two phases 1 tile 14.3 / 12.5, 24 14.9 / 14.7, three 13.0 / 13.5 (8 tiles), four
// 14.8 / 15.5 (of head_dim 128 15.0 / 17.8); maximum over layers, four phases of 64 rows and 16 lookahead rows 16.9 / 15.2, of head_dim
// 128 18.1 / 17.4 and with 8 lookahead rows 16.8 / 17.8; 128 rows, two phases 17.4 / 15.2, mean 14.7 / 15.3.
inline int prob_layers_per_split(const Plan &p, int64_t n_tiles)
{
    const int work = p.n_phases * (p.rows_pad / 32);
    const bool max_rows = p.layer_agg == SP_LAYER_MAX && (p.NB == 2 || p.D == 64);
    if ((work <= 4 && n_tiles <= (p.D == 64 ? 24 : 20)) || (max_rows && work <= 8 && n_tiles <= 20)) return p.n_layers;
    int64_t want = (kProbTargetWgs + n_tiles - 1) / n_tiles;
    if (want < 1) want = 1;
    if (want > p.n_layers) want = p.n_layers;
    return (int)((p.n_layers + want - 1) / want);
}

// What the device and the call's workspace leave room for.
struct Limits {
    int units;                             // workgroups of a launch
    int prompts;                           // of a launch
    int entries;                           // of a launch's table
    size_t exchange, results;              // bytes of a launch's exchange area in layer ranges, and of the ranges' results
};

// A ragged batch on the single-launch kernel: the prompts are packed into launches of at most one
// workgroup per compute unit, each prompt with all its 512-key tiles in one launch. Possible when every prompt fits a
// launch and the batch holds at least one tile of keys.
struct BatchGroups {
    std::vector<sp_fused::GroupTable> groups;
    std::vector<int> wgs;
    int ranges = 1;                 // layer ranges side by side in each of several launches
    int prompts = 1;                // that are not empty
    bool short_prompt = false;      // a prompt is shorter than a tile
    bool announced = false;         // see announces
};

// The prompts that are not empty, longest first, in the order in which they are packed.
struct Batch {
    std::vector<int> prompt, tiles;
    int64_t total = 0;              // tiles of all
    int count = 0, longest = 0;
    bool short_prompt = false;
};

// How they are packed: which launch the i-th one is in, and each launch's workgroups and prompts.
struct Packing {
    std::vector<int> launch, wgs, prompts;
    int most() const { return *std::max_element(wgs.begin(), wgs.end()); }
};

inline void survey(const Plan &p, const int64_t *offsets, int B, Batch &b)
{
    for (int i = 0; i < B; ++i) {
        const int64_t len = offsets[i + 1] - offsets[i];
        if (len == 0) continue;
        const int64_t tiles = sp::ceil_div(len, fused_tile(p));
        b.short_prompt |= len < fused_tile(p);
        b.longest = (int)std::max<int64_t>(b.longest, std::min<int64_t>(tiles, kMaxUnits + 1));
        b.total += tiles;
        ++b.count;
    }
}

// Longest first, in the order of the batch among equals; every prompt has at most kMaxUnits tiles.
inline void sort_prompts(const Plan &p, const int64_t *offsets, int B, Batch &b)
{
    int at[kMaxUnits + 2] = {};
    auto tiles_of = [&](int i) { return (int)sp::ceil_div(offsets[i + 1] - offsets[i], fused_tile(p)); };
    for (int i = 0; i < B; ++i) ++at[kMaxUnits - tiles_of(i) + 1];
    for (int t = 1; t <= kMaxUnits; ++t) at[t] += at[t - 1];
    b.prompt.resize(b.count);
    b.tiles.resize(b.count);
    for (int i = 0; i < B; ++i) {
        const int tiles = tiles_of(i);
        if (tiles == 0) continue;
        const int to = at[kMaxUnits - tiles]++;
        b.prompt[to] = i;
        b.tiles[to] = tiles;
    }
}

// First fit, longest first. Launches only fill up: one that has had no room for a prompt has none for the next of the
// same length.
inline Packing first_fit(const Batch &b, int cap, int max_prompts)
{
    Packing k;
    k.launch.resize(b.tiles.size());
    size_t g = 0;
    for (size_t i = 0; i < b.tiles.size(); ++i) {
        if (i > 0 && b.tiles[i] != b.tiles[i - 1]) g = 0;
        while (g < k.wgs.size() && (k.wgs[g] + b.tiles[i] > cap || k.prompts[g] >= max_prompts)) ++g;
        if (g == k.wgs.size()) {
            k.wgs.push_back(0);
            k.prompts.push_back(0);
        }
        k.wgs[g] += b.tiles[i];
        ++k.prompts[g];
        k.launch[i] = (int)g;
    }
    return k;
}

// The same number of launches with the workgroups shared out evenly: every prompt to the launch that has the fewest,
// longest first. False where that leaves no room for one of them.
inline bool share_out(const Batch &b, size_t launches, int cap, int max_prompts, Packing &k)
{
    k.launch.resize(b.tiles.size());
    k.wgs.assign(launches, 0);
    k.prompts.assign(launches, 0);
    using Item = std::pair<int, int>;              // workgroups, launch
    std::vector<Item> all(launches);
    for (size_t g = 0; g < launches; ++g) all[g].second = (int)g;
    std::priority_queue<Item, std::vector<Item>, std::greater<Item>> open(std::greater<Item>(), std::move(all));
    for (size_t i = 0; i < b.tiles.size(); ++i) {
        if (open.empty() || open.top().first + b.tiles[i] > cap) return false;
        const int g = open.top().second;
        open.pop();
        k.wgs[g] += b.tiles[i];
        k.launch[i] = g;
        if (++k.prompts[g] < max_prompts) open.push({k.wgs[g], g});
    }
    return true;
}

// In every launch the duties can rotate over all prompts (see score_impl).
inline bool duties_shared(const Plan &p, const Batch &b, const Packing &k)
{
    bool shared = !b.short_prompt;
    for (size_t g = 0; g < k.wgs.size(); ++g) shared &= k.prompts[g] * (p.rows_pad / sp_fused::kDutyRows) <= k.wgs[g];
    return shared;
}

// The same number of launches as first fit, shared out evenly where that is possible.
inline Packing pack(const Plan &p, const Batch &b, int cap, int max_prompts, const Packing &first)
{
    if (first.wgs.size() < 2) return first;
    Packing even;
    if (!share_out(b, first.wgs.size(), cap, max_prompts, even)) return first;
    return duties_shared(p, b, first) && !duties_shared(p, b, even) ? first : even;       // what is announced stays so
}

// First fit tells how many launches there are, and fills all but the last, unless it is the number of prompts that ends them.
inline bool fills_launches(const Packing &first, int cap) { return 4 * first.most() >= 3 * cap; }

// Whether launches of all layers take less time evenly filled. Steps do not get shorter in proportion to a launch's
// workgroups (head_dim 64: 2.05 us on 144, 2.6 on 255, where HBM bounds them). Whole passes of 656 workgroups in three launches
// 995 -> 956 us, 279 in two 641 -> 606, 287 670 / 670; head_dim 128, 295 in two 1079 -> 1023, 260 1078 -> 1028. Not where the number
// of prompts ends the launches (33 prompts, 63 workgroups in the fullest, 628 -> 701; 3 phases of head_dim 128, 37 prompts 28
// -> 51), nor with two blocks of query rows where many prompts exchange directly (see sp_fused::direct_max): first fit
// leaves those to its last launches, an even share has them lengthen the steps of all (12 x 12 phases, 16 lookahead rows,
// 24 prompts of 308 workgroups 1025 -> 1155, 36 of 409 1070 -> 1178; up to three a launch 0.82 .. 0.98 of the time).
inline bool even_pays(const Plan &p, const Batch &b, int cap, const Packing &first)
{
    if (!fills_launches(first, cap)) return false;
    if (p.rows_pad <= 32 || duties_shared(p, b, first)) return true;
    const auto direct = std::count_if(b.tiles.begin(), b.tiles.end(), [&](int t) { return t <= sp_fused::direct_max(p.rows_pad); });
    return direct <= 3 * (int64_t)first.wgs.size();
}

// Batches the single-launch kernel takes whatever their size: every prompt fills a tile, no launch of first fit has more
// duty blocks than workgroups, and one range of layers fills enough of the device.
inline bool announces(const Plan &p, const Batch &b, const Packing &first)
{
    return !fused_big(p) && duties_shared(p, b, first) && b.total >= sp_fused::kMinWorkgroups;
}

// Otherwise (few workgroups, or tiles that short prompts leave half empty): whether the single-launch kernel beats the
// three-kernel path. A launch costs its steps (a range's phases and five more to fill and drain the pipeline); the three
// kernels take the longer the more keys their tiles hold, `keys` with the empty places. Each variant has its line,
// in MB of bf16 keys: `per_step` for each step, or `steep` for each step less `base` where the fixed cost of the three
// launches counts. Steps of several prompts in layer ranges take the longer the more of them there are, since what exchanges
// directly (see sp_fused::direct_max) and last tiles that are partly empty are then a larger part of a launch: with 32 rows such
// batches have lines of their own, at head_dim 64 from 18 steps on. The lines of 32 rows lie where the present kernels cross (8-bit keys of head_dim 64 apart); the others
// where they crossed before the single launch's steps became 5 to 25 % shorter and short prompts lost their merge launch;
// the present kernels cross at or a little before them. Measured on these (tokens: three kernels / single launch, us; * =
// the line still takes the slower one; 16 layers x 8 kv heads unless noted):
//   32 rows                      3000 32 / 34, 3600 36 / 36, 4600 41 / 36, 6000 48 / 37, 9000 63 / 53, 12000 75 / 54; 28 layers,
//                                head_dim 128: 700 33 / 34, 1000* 38 / 36, 1500 46 / 37; 4 x 4 heads, head_dim 128: 9000 29 / 29,
//                                12000 32 / 31; 30 prompts of 1100 .. 1500 271 / 175, 24 of 60 .. 4000 364 / 189. Whole passes:
//                                3900 51.1 / 51.4, 4200 54.0 / 50.3, 4850 56.5 / 50.6; 28 layers, 2800 57.2 / 52.2; 28 layers, head_dim
//                                128: 1030 51.8 / 48.0, 1400 57.6 / 49.6; 16 layers, 2200 59.9 / 52.5; 16 x 16 phases, 3500 55 / 47
//   32 rows, batches in ranges   9 prompts of 316 .. 2681 (8744 in all) 59 / 70, 22 of 317 .. 2800 134 / 168, 39 of 73 .. 3477 in two launches
//                                of three ranges 237 / 280, 6 (16 tiles) 51 / 51; 13 steps: 4 x 4 phases, 30 (75 tiles) 39 / 35; 28 layers,
//                                head_dim 128: 5 (2373 in all) 59 / 69, 8 (2832) 68 / 85, 3 (10 tiles) 51 / 48
//   64 rows, 9+ lookahead rows   3600 47 / 47, 4500* 51 / 48, 5000 53 / 49, 6200 58 / 51, 9000 75 / 79, 10100* 79 / 73, 12000 88 / 73,
//                                16384 121 / 76; 24 prompts of 60 .. 4000 460 / 293, 30 of 1100 .. 1500 359 / 291
//   64 rows, 5+ heads a kv head  4600 51 / 51, 6200 58 / 52, 9000 73 / 80, 12000* 86 / 74, 16384 117 / 78
//   64 rows, head_dim 128        24 x 4 heads: 3000 50 / 52, 3600* 54 / 50, 4500 70 / 50; 24 prompts of 60 .. 4000 671 / 429
//   8-bit keys, 32 rows          4500 35 / 38, 6000 43 / 38, 8192 49 / 38, 10000 56 / 56, 12000 62 / 55, 16400 86 / 73, 18000 95 / 74,
//                                22000 105 / 94; 28 layers, head_dim 128 (32 rows): 1000 34 / 35, 1500 40 / 36, as with bf16 keys
//   8-bit keys, 64 rows          6200 56 / 53, 9000 69 / 86, 12100 80 / 85, 13000 97 / 84, 16384 108 / 86, 18000* 122 / 113, 19000 124 / 113,
//                                22000 137 / 142, 24500* 145 / 147, 30000 189 / 141 (no line has the crossing at 17600 as well)
inline bool steps_pay(const Plan &p, bool fp8, int prompts, int64_t keys, int ranges, int launches)
{
    struct Line { double per_step, steep, base; };
    const bool wide = p.rows_pad > 32;
    const Line line = p.D == 128 ? (wide ? Line{8.0, 8.0, 0} : fp8 ? Line{5.2, 5.2, 0} : Line{4.7, 4.7, 0})
                    : fp8        ? (wide ? Line{11.0, 12.4, 59} : Line{9.35, 13.2, 77})
                    : !wide      ? Line{5.2, 5.2, 0}
                    : p.NB == 2  ? Line{8.0, 11.25, 68}
                                 : Line{9.4, 14.0, 91};
    const double a_launch = (double)(sp::ceil_div(p.n_layers, ranges) * (p.n_phases / p.n_layers) + 5), steps = launches * a_launch;
    double least = std::min(line.per_step * steps, line.steep * steps - line.base * launches);
    if (prompts > 1 && ranges > 1 && !wide)
        least = p.D == 128 ? std::max(least, launches * (7.2 * a_launch - 48.5)) : steps > 17 ? 6.3 * steps : least;
    return (double)keys * p.n_phases * p.D * 2e-6 >= least;
}

// Layer ranges tried for a batch of several launches.
constexpr int kMaxSpread = 4;

inline int max_prompts(const Limits &lim, int ranges) { return std::min(lim.prompts, lim.entries / ranges); }

inline int64_t fewest_launches(const Batch &b, const Limits &lim, int ranges)
{
    return std::max(sp::ceil_div(b.total, lim.units / ranges), sp::ceil_div(b.count, max_prompts(lim, ranges)));
}

// Whether no packing into several launches, with whatever ranges, can be worth it for a batch of `keys` keys: steps_pay with
// the fewest launches that workgroups and prompts allow. Asked before anything is sorted and packed: 4096 prompts of 60 to 90
// tokens cost the host 5.0 ms before the three kernels took them, now 0.01 (64: 7.1 -> 0.2 us).
inline bool never_pays(const Plan &p, const Batch &b, int64_t keys, const Limits &lim)
{
    for (int ranges = 1; ranges <= std::min(kMaxSpread, p.n_layers); ++ranges) {
        if (b.longest > lim.units / ranges) break;
        const int64_t launches = fewest_launches(b, lim, ranges);
        if (launches < 2 || steps_pay(p, false, b.count, keys, ranges, (int)launches)) return false;
    }
    return true;
}

// A batch of several launches may do with fewer steps on more of them: launches of at most half the workgroups run their
// layers as two ranges side by side, in half the steps. A launch costs the steps of a range and some nine more to
// be launched, to fill and to drain; a step takes 2.05 us on up to 200 workgroups and 2.6 on 256, where HBM bounds it. Whole
// passes, 16 x 8 phases of head_dim 64: 279 workgroups in nine prompts 606 -> 516 us, token-major 343 in fifteen 721 -> 585; 28 x 8 of head_dim
// 128: 260 1028 -> 840, 298 in nine 1019 -> 790, in twelve 1073 -> 839.
// Replaces `best`, the launches of all layers evenly filled, and tells the number of ranges.
inline int spread_batch(const Plan &p, const Batch &b, int64_t tokens, const Limits &lim, Packing &best)
{
    const size_t result = sizeof(float) * (size_t)tokens * (p.layer_agg == SP_LAYER_MAX ? 8 * p.NB : 1);      // of a range
    auto model = [&](double launches, int ranges, int most) {
        return launches * (sp::ceil_div(p.n_layers, ranges) * (p.n_phases / p.n_layers) + 9) * std::max(0.8, ranges * most / 256.0);
    };
    int n = 1;
    double least = 0.92 * model((double)best.wgs.size(), 1, best.most());         // not for less than the model is worth
    for (int ranges = 2; ranges <= std::min(kMaxSpread, p.n_layers) && ranges * result <= lim.results; ++ranges) {
        if (b.longest > lim.units / ranges) break;
        if (sp::ceil_div(p.n_layers, sp::ceil_div(p.n_layers, ranges)) != ranges) continue;      // a range would be empty
        if (model((double)fewest_launches(b, lim, ranges), ranges, 0) >= least) continue;
        const int cap = lim.units / ranges, prompts = max_prompts(lim, ranges);
        const Packing k = pack(p, b, cap, prompts, first_fit(b, cap, prompts));
        const double time = model((double)k.wgs.size(), ranges, k.most());
        if (k.wgs.size() < 2 || time >= least) continue;
        bool room = true;
        for (size_t g = 0; g < k.wgs.size(); ++g)
            room &= sp_fused::workspace_bytes(p.rows_pad, k.wgs[g] * ranges, k.prompts[g] * ranges) <= lim.exchange;
        if (!room) continue;
        least = time;
        n = ranges;
        best = k;
    }
    return n;
}

inline void fill_tables(const Plan &p, const int64_t *offsets, const Batch &b, const Packing &k, BatchGroups &out)
{
    sp_fused::GroupTable empty;
    std::memset(&empty, 0, sizeof empty);
    out.groups.assign(k.wgs.size(), empty);
    out.wgs = k.wgs;
    for (size_t i = 0; i < b.prompt.size(); ++i) {
        sp_fused::GroupTable &t = out.groups[k.launch[i]];
        const int64_t start = offsets[b.prompt[i]];
        t.prompt[t.n] = b.prompt[i];
        t.start[t.n] = start;
        t.len[t.n] = (int32_t)(offsets[b.prompt[i] + 1] - start);
        t.layers[t.n] = p.n_layers;
        t.w0[t.n + 1] = t.w0[t.n] + b.tiles[i];
        ++t.n;
    }
}

// What a batch of several launches may do: first fit only, or even launches and layer ranges. Both announce the same batches.
enum class Launches { kFirstFit, kRanges };

// The launches of a ragged batch of a shape that the kernel holds; false where it has none or the three kernels are
// certain to be faster. `keys`: of the three-kernel path's tiles.
inline bool plan_batch(const Plan &p, const int64_t *offsets, int B, int64_t keys, const Limits &lim, Launches may, BatchGroups &out)
{
    if (lim.units < sp_fused::kMinWorkgroups || offsets[B] < fused_tile(p)) return false;
    Batch b;
    survey(p, offsets, B, b);
    if (b.longest > lim.units || (b.short_prompt && never_pays(p, b, keys, lim))) return false;
    sort_prompts(p, offsets, B, b);
    const Packing first = first_fit(b, lim.units, lim.prompts);
    out.announced = announces(p, b, first);
    Packing k = first;
    if (may == Launches::kRanges && first.wgs.size() > 1) {
        k = pack(p, b, lim.units, lim.prompts, first);
        // two blocks of query rows at head_dim 64: 59 prompts of 147 workgroups 575 us on the three kernels, 610 in ranges
        if (p.D == 128 || p.rows_pad <= 32 || fills_launches(first, lim.units)) out.ranges = spread_batch(p, b, offsets[B], lim, k);
        if (out.ranges == 1 && !even_pays(p, b, lim.units, first)) k = first;
    }
    out.short_prompt = b.short_prompt;
    out.prompts = b.count;
    fill_tables(p, offsets, b, k, out);
    return true;
}

// The table of a launch with every entry of `t` once per layer range.
inline sp_fused::GroupTable split_layers(const sp_fused::GroupTable &t, int n_layers, int ranges)
{
    sp_fused::GroupTable r;
    std::memset(&r, 0, sizeof r);
    const int per_range = (int)sp::ceil_div(n_layers, ranges);
    for (int s = 0; s < ranges; ++s)
        for (int i = 0; i < t.n; ++i) {
            r.prompt[r.n] = t.prompt[i];
            r.start[r.n] = t.start[i];
            r.len[r.n] = t.len[i];
            r.layer0[r.n] = s * per_range;
            r.layers[r.n] = std::min(per_range, n_layers - s * per_range);
            r.slice[r.n] = s;
            r.w0[r.n + 1] = r.w0[r.n] + t.w0[i + 1] - t.w0[i];
            ++r.n;
        }
    return r;
}

}  // namespace sp_plan
