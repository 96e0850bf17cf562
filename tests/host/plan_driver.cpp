// Host-side driver for the choices of the score calls (sp_score_plan.hpp; needs no GPU): random batches against the
// definitions of first fit and of an even share written out plainly, what holds for every plan, and the cost of planning.
#include "sp_score_plan.hpp"

#include <chrono>
#include <cstdio>
#include <cstring>
#include <random>
#include <string>

using namespace sp_plan;

static int g_fail = 0;
#define EXPECT(cond)                                                                                   \
    do {                                                                                               \
        if (!(cond)) { std::printf("FAILED %s:%d: %s\n", __FILE__, __LINE__, #cond); ++g_fail; }       \
    } while (0)

static Plan shape(int layers, int kv, int G, int D, int n_q, int agg = 0)
{
    Plan p;
    std::memset(&p, 0, sizeof p);
    p.D = D;
    p.NB = (n_q + 7) / 8;
    p.n_gblk = (G + 3) / 4;
    p.rows_pad = 32 * p.NB * p.n_gblk;
    p.tile_keys = D == 64 ? 256 : 128;
    p.n_layers = layers;
    p.n_phases = layers * kv;
    p.layer_agg = agg;
    return p;
}

static const Plan kShapes[] = {shape(16, 8, 4, 64, 8),  shape(16, 8, 4, 64, 16), shape(16, 4, 8, 64, 8), shape(28, 8, 2, 128, 8),
                               shape(24, 4, 8, 128, 8), shape(12, 12, 1, 64, 8), shape(2, 2, 2, 64, 16), shape(5, 3, 1, 64, 8, 1)};

static Limits device(int units = 256) { return Limits{units, kMaxGroupPrompts, sp_fused::kMaxGroup, SIZE_MAX, SIZE_MAX}; }

static std::vector<int64_t> batch(std::mt19937 &rng, int B, double lo, double hi)
{
    std::vector<int64_t> off{0};
    std::uniform_real_distribution<double> u(std::log(lo), std::log(hi));
    for (int b = 0; b < B; ++b) off.push_back(off.back() + (rng() % 8 == 0 ? 0 : (int64_t)std::exp(u(rng))));
    return off;
}

static int64_t keys_of(const Plan &p, const std::vector<int64_t> &off)
{
    int64_t n = 0;
    for (size_t b = 0; b + 1 < off.size(); ++b) n += sp::ceil_div(off[b + 1] - off[b], p.tile_keys);
    return n * p.tile_keys;
}

// Every prompt that is not empty is in exactly one launch, whole, and no launch is over its limits.
static void check_plan(const Plan &p, const std::vector<int64_t> &off, const Limits &lim, const BatchGroups &bg)
{
    std::vector<int> seen(off.size() - 1, 0);
    for (size_t g = 0; g < bg.groups.size(); ++g) {
        const sp_fused::GroupTable &t = bg.groups[g];
        EXPECT(t.n >= 1 && t.n <= lim.prompts && t.w0[0] == 0 && t.w0[t.n] == bg.wgs[g] && bg.wgs[g] * bg.ranges <= lim.units);
        for (int i = 0; i < t.n; ++i) {
            ++seen[t.prompt[i]];
            EXPECT(t.start[i] == off[t.prompt[i]] && t.len[i] == off[t.prompt[i] + 1] - off[t.prompt[i]]);
            EXPECT(t.w0[i + 1] - t.w0[i] == sp::ceil_div(t.len[i], fused_tile(p)));
            EXPECT(t.layer0[i] == 0 && t.layers[i] == p.n_layers && t.slice[i] == 0);
        }
        if (bg.ranges == 1) continue;
        EXPECT(t.n * bg.ranges <= lim.entries);
        const sp_fused::GroupTable r = split_layers(t, p.n_layers, bg.ranges);
        EXPECT(r.n == t.n * bg.ranges && r.w0[r.n] == bg.wgs[g] * bg.ranges);
        for (int i = 0; i < r.n; ++i) EXPECT(r.layers[i] >= 1 && r.layer0[i] >= 0 && r.layer0[i] + r.layers[i] <= p.n_layers);
    }
    for (size_t b = 0; b < seen.size(); ++b) EXPECT(seen[b] == (off[b + 1] > off[b]));
}

static void test_packing()
{
    std::mt19937 rng(5);
    for (int n = 0; n < 4000; ++n) {
        const Plan &p = kShapes[rng() % 8];
        const int cap = 40 + (int)(rng() % 217), most = 1 + (int)(rng() % 32);
        const auto off = batch(rng, 1 + (int)(rng() % 200), 20, fused_tile(p) * (1 + rng() % (cap - 1)));
        Batch b;
        survey(p, off.data(), (int)off.size() - 1, b);
        if (b.count == 0) continue;
        sort_prompts(p, off.data(), (int)off.size() - 1, b);
        EXPECT((int)b.prompt.size() == b.count && b.tiles[0] == b.longest);
        for (int i = 0; i + 1 < b.count; ++i) EXPECT(b.tiles[i] > b.tiles[i + 1] || (b.tiles[i] == b.tiles[i + 1] && b.prompt[i] < b.prompt[i + 1]));
        std::vector<int> wgs, prompts, launch;
        for (int t : b.tiles) {                                    // first fit
            size_t g = 0;
            while (g < wgs.size() && (wgs[g] + t > cap || prompts[g] == most)) ++g;
            if (g == wgs.size()) { wgs.push_back(0); prompts.push_back(0); }
            wgs[g] += t;
            ++prompts[g];
            launch.push_back((int)g);
        }
        const Packing first = first_fit(b, cap, most);
        EXPECT(first.wgs == wgs && first.prompts == prompts && first.launch == launch);
        std::fill(wgs.begin(), wgs.end(), 0);                      // an even share: the emptiest launch with room
        std::fill(prompts.begin(), prompts.end(), 0);
        bool room = true;
        for (size_t i = 0; i < b.tiles.size() && room; ++i) {
            size_t to = wgs.size();
            for (size_t g = 0; g < wgs.size(); ++g)
                if (wgs[g] + b.tiles[i] <= cap && prompts[g] < most && (to == wgs.size() || wgs[g] < wgs[to])) to = g;
            room = to < wgs.size();
            if (!room) break;
            wgs[to] += b.tiles[i];
            ++prompts[to];
            launch[i] = (int)to;
        }
        Packing even;
        EXPECT(share_out(b, wgs.size(), cap, most, even) == room);
        if (room) EXPECT(even.wgs == wgs && even.prompts == prompts && even.launch == launch);
    }
}

static void test_plans()
{
    std::mt19937 rng(7);
    int launches = 0, spread = 0, announced = 0, refused = 0;
    for (int n = 0; n < 20000; ++n) {
        const Plan &p = kShapes[rng() % 8];
        const double lo[] = {60, 60, 500, 2000, 1000}, hi[] = {90, 4000, 20000, 66000, 1500};
        const int kind = (int)(rng() % 5);
        const auto off = batch(rng, 1 + (int)(rng() % (kind == 0 ? 500 : 60)), lo[kind], hi[kind]);
        const int B = (int)off.size() - 1;
        const int64_t keys = keys_of(p, off);
        const Limits lim = device();
        BatchGroups bg, plain;
        if (!plan_batch(p, off.data(), B, keys, lim, Launches::kRanges, bg)) {
            // refused before packing: then no number of launches and ranges is worth it
            Batch b;
            survey(p, off.data(), B, b);
            if (b.longest > lim.units || off[B] < fused_tile(p)) continue;
            ++refused;
            sort_prompts(p, off.data(), B, b);
            Packing k = pack(p, b, lim.units, lim.prompts, first_fit(b, lim.units, lim.prompts));
            EXPECT(k.wgs.size() > 1 && !announces(p, b, first_fit(b, lim.units, lim.prompts)));
            const int ranges = spread_batch(p, b, off[B], lim, k);
            EXPECT(!steps_pay(p, false, b.count, keys, ranges, (int)k.wgs.size()));
            continue;
        }
        check_plan(p, off, lim, bg);
        launches += bg.groups.size() > 1;
        spread += bg.ranges > 1;
        announced += bg.announced;
        EXPECT(plan_batch(p, off.data(), B, keys, lim, Launches::kFirstFit, plain) && plain.ranges == 1 && plain.announced == bg.announced);
        check_plan(p, off, lim, plain);
        Batch b;
        survey(p, off.data(), B, b);
        sort_prompts(p, off.data(), B, b);
        EXPECT(plain.wgs == first_fit(b, lim.units, lim.prompts).wgs);
    }
    EXPECT(launches > 1000 && spread > 300 && announced > 1000 && refused > 300);
}

// Small layer counts, of which some ranges would be empty (4 layers in three, 5, 6 or 9 in four), and launches of few prompts,
// which several ranges suit better than with the device's own limits.
static void test_ranges()
{
    std::mt19937 rng(13);
    int spread = 0;
    for (int n = 0; n < 40000; ++n) {
        const int D = rng() % 2 ? 64 : 128;
        const Plan p = shape(1 + (int)(rng() % 12), 1 + (int)(rng() % 8), 1 + (int)(rng() % 4), D, 8, (int)(rng() % 2));
        Limits lim = device(64 + (int)(rng() % 193));
        lim.prompts = 2 << rng() % 5;
        lim.entries = 16 << rng() % 3;
        const auto off = batch(rng, 1 + (int)(rng() % 60), 100, 100 * (1 + rng() % 300));
        BatchGroups bg;
        if (!plan_batch(p, off.data(), (int)off.size() - 1, keys_of(p, off), lim, Launches::kRanges, bg)) continue;
        check_plan(p, off, lim, bg);
        spread += bg.ranges > 1;
    }
    EXPECT(spread > 1000);
}

// The last prompt is shorter than a tile.
static std::vector<int> launches_of(const Plan &p, const std::vector<int> &tiles)
{
    std::vector<int64_t> off{0};
    for (int t : tiles) off.push_back(off.back() + (int64_t)t * fused_tile(p));
    off.back() -= 7;
    BatchGroups bg;
    EXPECT(plan_batch(p, off.data(), (int)tiles.size(), int64_t(1) << 40, device(), Launches::kRanges, bg) && bg.ranges == 1);
    return bg.wgs;
}

// Which launches of all layers are filled evenly: where first fit fills the first ones, and with two blocks of query rows
// where few prompts exchange directly (one layer: no ranges).
static void test_even()
{
    using V = std::vector<int>;
    const Plan narrow = shape(1, 8, 4, 64, 8), wide = shape(1, 8, 4, 64, 16), big = shape(1, 4, 8, 128, 8);
    const V direct6 = {200, 190, 10, 9, 8, 7, 6, 1}, direct7 = {200, 190, 10, 9, 8, 7, 6, 5, 1};
    EXPECT((launches_of(narrow, direct6) == V{216, 215}));
    EXPECT((launches_of(narrow, direct7) == V{220, 216}));
    EXPECT((launches_of(narrow, V(33, 1)) == V{32, 1}));               // the number of prompts ends a launch
    for (const Plan &p : {wide, big}) {
        EXPECT((launches_of(p, direct6) == V{216, 215}));              // three a launch
        EXPECT((launches_of(p, direct7) == V{246, 190}));              // one more
        EXPECT((launches_of(p, {200, 190, 20, 18, 1}) == V{218, 211}));
    }
}

// Few phases: all layers of the prob pass in one workgroup, or a range of one layer each.
static void test_whole()
{
    auto whole = [](const Plan &p, int tiles) { return prob_layers_per_split(p, tiles) == p.n_layers; };
    const Plan narrow = shape(2, 2, 2, 64, 8), narrow128 = shape(2, 2, 2, 128, 8), rows64 = shape(2, 2, 2, 64, 16), three = shape(3, 1, 8, 128, 8);
    EXPECT(whole(narrow, 1) && whole(narrow, 24) && !whole(narrow, 25));
    EXPECT(whole(narrow128, 20) && !whole(narrow128, 21));
    EXPECT(!whole(shape(5, 1, 4, 64, 8), 1));
    EXPECT(!whole(rows64, 1) && !whole(three, 1) && !whole(shape(2, 1, 8, 64, 16), 1));       // two and four blocks of rows
    EXPECT(whole(shape(2, 1, 4, 64, 16), 24) && whole(shape(2, 1, 8, 128, 8), 20));
    EXPECT(whole(shape(2, 2, 2, 64, 16, SP_LAYER_MAX), 20) && !whole(shape(2, 2, 2, 64, 16, SP_LAYER_MAX), 21));
    EXPECT(whole(shape(2, 2, 2, 128, 16, SP_LAYER_MAX), 1) && !whole(shape(2, 2, 8, 128, 8, SP_LAYER_MAX), 1));
    EXPECT(!whole(shape(5, 1, 4, 64, 16, SP_LAYER_MAX), 1));
    EXPECT(whole(shape(1, 64, 8, 64, 16), 1000) && whole(shape(16, 8, 4, 64, 8), 1024));          // nothing to split, or enough tiles
}

static void test_cost()
{
    // the documented maximum, of prompts that the three kernels take; best of some runs
    std::mt19937 rng(11);
    const Plan &p = kShapes[0];
    for (int B : {512, 4096}) {
        const auto off = batch(rng, B, 60, 90);
        double best = 1e9;
        for (int i = 0; i < 20; ++i) {
            BatchGroups bg;
            const auto t0 = std::chrono::steady_clock::now();
            EXPECT(!plan_batch(p, off.data(), B, keys_of(p, off), device(), Launches::kRanges, bg));
            best = std::min(best, std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count());
        }
        std::printf("planning %d prompts of 60 to 90 tokens: %.1f us\n", B, best * 1e6);
        EXPECT(best < B * 0.1e-6);
    }
    // and of prompts that it packs: 4096 of 600 to 3000 tokens
    const auto off = batch(rng, 4096, 600, 3000);
    double best = 1e9;
    for (int i = 0; i < 20; ++i) {
        BatchGroups bg;
        const auto t0 = std::chrono::steady_clock::now();
        EXPECT(plan_batch(p, off.data(), 4096, keys_of(p, off), device(), Launches::kRanges, bg));
        best = std::min(best, std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count());
    }
    std::printf("planning 4096 prompts of 600 to 3000 tokens: %.1f us\n", best * 1e6);
    EXPECT(best < 4096 * 0.8e-6);
}

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "packing") test_packing();
    else if (what == "plans") test_plans();
    else if (what == "ranges") test_ranges();
    else if (what == "even") test_even();
    else if (what == "whole") test_whole();
    else if (what == "cost") test_cost();
    else { std::printf("unknown test %s\n", what.c_str()); return 2; }
    std::printf(g_fail ? "plan driver: %d check(s) failed\n" : "plan driver: all checks passed\n", g_fail);
    return g_fail ? 1 : 0;
}
