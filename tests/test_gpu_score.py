"""GPU parity of sp_score / sp_score_batch against the CPU float64 oracle,
element by element on the same seeded inputs. Tolerance (stated target of the
build): |gpu - oracle| <= 1e-3 * |oracle| for every token, both aggregation
modes. All calls go through the C ABI."""
from __future__ import annotations

import dataclasses
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def small_workload(name, Lyr, H, Hkv, d, n_q, L, cfg_id=100, hh=(1, 100)):
    return synth.Workload(name, cfg_id, Lyr, H, Hkv, d, n_q, L, hh_frac_num=hh[0], hh_frac_den=hh[1])


SHAPES = [
    # name, Lyr, H, Hkv, d, n_q, L   (several key tiles and a ragged tail unless noted)
    ("g4_nq16_d64", 3, 8, 2, 64, 16, 1500),
    ("g4_nq8_d64", 2, 8, 2, 64, 8, 777),
    ("g2_nq8_d128", 3, 4, 2, 128, 8, 777),
    ("g1_nq3_d64", 2, 3, 3, 64, 3, 333),
    ("g8_nq5_d128", 2, 8, 1, 128, 5, 300),
    ("g16_nq8_d64", 1, 16, 1, 64, 8, 260),
    ("g8_nq16_d64", 1, 16, 2, 64, 16, 260),
    ("g3_nq9_d64", 2, 6, 2, 64, 9, 515),
    ("one_key", 2, 4, 2, 64, 8, 1),
    ("exact_tile", 2, 4, 2, 64, 8, 256),
    ("tile_plus_one", 2, 4, 2, 64, 8, 257),
    ("sub_tile_d128", 2, 4, 2, 128, 8, 31),
    # general path with the layers of the prob pass in ranges of 2 + 1, and with enough tiles for no split
    ("uneven_split_d128", 3, 2, 1, 128, 4, 70001),
    ("unsplit_d128", 2, 2, 1, 128, 4, 131072 + 77),
]


@pytest.mark.parametrize("shape", SHAPES, ids=[s[0] for s in SHAPES])
@pytest.mark.parametrize("mode", [oracle.LAYER_MEAN, oracle.LAYER_MAX], ids=["mean", "max"])
def test_score_matches_oracle(shape, mode):
    from gpu_util import assert_scores_close, gpu_score
    name, Lyr, H, Hkv, d, n_q, L = shape
    say(f"[score] {name} mode={mode} Lyr={Lyr} H={H} Hkv={Hkv} d={d} n_q={n_q} L={L}")
    w = small_workload(name, Lyr, H, Hkv, d, n_q, L, cfg_id=100 + SHAPES.index(shape))
    inp = synth.make_score_inputs(w)
    want = oracle.score(inp["q"][0], inp["k"], w.scale, mode)
    got = gpu_score(inp["q"][0], inp["k"], w.scale, mode)
    assert_scores_close(got, want)


@pytest.mark.parametrize("tokens", [8 * 256, 8 * 256 + 1, 48 * 256, 48 * 256 + 1])
@pytest.mark.parametrize("n_q", [8, 16])
def test_score_around_the_merge_in_the_prob_pass(tokens, n_q):
    """Three-kernel path: eight partials a turn of the merge loop, and the last length the prob pass merges itself
    (two phases of 32 rows a workgroup: 48 tiles; of 64 rows: 40) against the first that takes the merge kernel."""
    from gpu_util import assert_scores_close, gpu_score, score_path
    if n_q == 16 and tokens > 40 * 256:
        tokens -= 8 * 256
    say(f"[score] merge n_q={n_q} L={tokens}")
    w = small_workload("merge", 2, 8, 2, 64, n_q, tokens, cfg_id=180, hh=(1, 200))
    inp = synth.make_score_inputs(w)
    for mode in (0, 1):
        got = gpu_score(inp["q"][0], inp["k"], w.scale, mode)
        assert score_path() == "general"
        assert_scores_close(got, oracle.score(inp["q"][0], inp["k"], w.scale, mode))


@pytest.mark.parametrize("cfg", ["tiny"])
@pytest.mark.parametrize("layout", ["HND", "NHD"])
@pytest.mark.parametrize("mode", [0, 1], ids=["mean", "max"])
def test_score_tiny_config_both_layouts(cfg, layout, mode):
    from gpu_util import assert_scores_close, gpu_score
    say(f"[score] cfg={cfg} layout={layout} mode={mode}")
    w = synth.get_config(cfg)
    inp = synth.make_score_inputs(w, layout=layout)
    want = oracle.score(inp["q"][0], inp["k"], w.scale, mode, layout=layout)
    got = gpu_score(inp["q"][0], inp["k"], w.scale, mode, layout=layout)
    assert_scores_close(got, want)


def test_score_closed_forms_on_gpu():
    """Uniform keys give 1/L; a single dominant key captures the score; a huge
    common shift of all keys does not change the result (max-subtraction)."""
    from gpu_util import gpu_score
    say("[score] closed forms")
    rng = np.random.default_rng(5)
    Lyr, H, Hkv, n_q, d, L = 2, 8, 2, 8, 64, 700
    q = synth.f32_to_bf16_bits(rng.integers(-3, 4, size=(Lyr, H, n_q, d)).astype(np.float32) * 0.25)
    krow = rng.integers(-3, 4, size=(Hkv, 1, d)).astype(np.float32)
    k = [synth.f32_to_bf16_bits(np.repeat(krow, L, axis=1)) for _ in range(Lyr)]
    for mode in (0, 1):
        got = gpu_score(q, k, 0.125, mode)
        np.testing.assert_allclose(got, 1.0 / L, rtol=1e-5)
    # dominant key
    kz = np.zeros((Hkv, L, d), np.float32)
    kz[:, 123, :] = 8.0 * synth.bf16_bits_to_f32(q[0, 0, 0])[None, :]
    kd = [synth.f32_to_bf16_bits(kz) for _ in range(Lyr)]
    want = oracle.score(q, kd, 0.125, 1)
    got = gpu_score(q, kd, 0.125, 1)
    np.testing.assert_allclose(got, want, rtol=1e-3)
    assert got.argmax() == 123
    # shift invariance with a large shift (exact in bf16: |k + v| <= 67)
    kf = rng.integers(-3, 4, size=(Hkv, L, d)).astype(np.float32)
    v = rng.choice([-64.0, 64.0], size=(1, 1, d)).astype(np.float32)
    base = gpu_score(q, [synth.f32_to_bf16_bits(kf)] * Lyr, 0.125, 0)
    shifted = gpu_score(q, [synth.f32_to_bf16_bits(kf + v)] * Lyr, 0.125, 0)
    assert np.isfinite(shifted).all()
    np.testing.assert_allclose(shifted, base, rtol=2e-4)


def test_score_is_deterministic():
    from gpu_util import gpu_score
    say("[score] determinism")
    w = small_workload("det", 3, 8, 2, 64, 16, 2100, cfg_id=150)
    inp = synth.make_score_inputs(w)
    a = gpu_score(inp["q"][0], inp["k"], w.scale, 0)
    b = gpu_score(inp["q"][0], inp["k"], w.scale, 0)
    assert a.tobytes() == b.tobytes()


@pytest.mark.parametrize("layout", ["HND", "NHD"])
def test_score_batch_matches_oracle_per_prompt(layout):
    """Ragged batch with an empty prompt, a one-token prompt and lengths around
    the tile size; each prompt is softmaxed over its own keys only."""
    from gpu_util import assert_scores_close, gpu_score, gpu_score_batch
    say(f"[score_batch] layout={layout}")
    lengths = np.array([300, 1, 0, 513, 256, 77], dtype=np.int64)
    w = dataclasses.replace(small_workload("rag", 2, 8, 2, 64, 8, 0, cfg_id=160), batch=len(lengths))
    hh = synth.heavy_hitter_positions(w, lengths)
    q = synth.gen_q(w, len(lengths))
    ks = [synth.gen_k_layer(w, l, q, lengths, hh) for l in range(w.n_layers)]      # [Hkv][T][d]
    offsets = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    packed = ks if layout == "HND" else [np.ascontiguousarray(k.transpose(1, 0, 2)) for k in ks]
    for mode in (0, 1):
        got = gpu_score_batch(q, packed, offsets, w.scale, mode, layout=layout)
        for b, Lb in enumerate(lengths):
            if Lb == 0:
                continue
            sl = slice(int(offsets[b]), int(offsets[b + 1]))
            kb = [np.ascontiguousarray(k[:, sl, :]) for k in ks]
            want = oracle.score(q[b], kb, w.scale, mode)
            assert_scores_close(got[sl], want)
            if layout == "HND":
                single = gpu_score(q[b], kb, w.scale, mode)
                np.testing.assert_allclose(got[sl], single, rtol=1e-6)


FUSED_BATCHES = [
    # name, Lyr, H, Hkv, d, n_q, prompt lengths  (every prompt empty or >= 512 tokens: one launch or several)
    ("batch_one_launch", 2, 8, 2, 64, 8, [20000, 512, 700, 0, 15000, 9001]),
    ("batch_nq16_two_row_blocks", 1, 8, 2, 64, 16, [12000, 24000, 513]),
    ("batch_g8_two_gblocks", 1, 16, 2, 64, 8, [33000, 1024, 2047]),
    ("batch_several_launches", 1, 4, 1, 64, 8, [70000, 65000, 60000, 3000, 1500]),
    ("batch_single_prompt", 2, 8, 2, 64, 5, [40000]),
    ("batch_d128_one_launch", 2, 4, 2, 128, 8, [9000, 256, 300, 0, 7000, 4001]),
    # the kernel instantiations with a fixed model shape (16 layers, 32 / 8 heads) for several prompts a launch
    ("batch_draft_model_nq16", 16, 32, 8, 64, 16, [20000, 13000, 600]),
    ("batch_draft_model_nq8", 16, 32, 8, 64, 8, [15000, 18000, 512, 0, 1000]),
    ("batch_d128_several_launches", 1, 4, 2, 128, 8, [40000, 33000, 30000, 1500]),
]


@pytest.mark.parametrize("case", FUSED_BATCHES, ids=[c[0] for c in FUSED_BATCHES])
def test_score_batch_on_the_single_launch_kernel(case):
    """Ragged batches whose prompts are all at least one tile (512 keys; 256 at head_dim 128) long take the single-launch
    kernel, several prompts to a launch: every prompt against the oracle run on that prompt alone, both
    modes, both layouts, deterministic."""
    import paper_2603_02631_amd as sp
    from gpu_util import assert_scores_close, gpu_score_batch, make_desc
    name, Lyr, H, Hkv, d, n_q, lens = case
    lengths = np.array(lens, dtype=np.int64)
    say(f"[score_batch-fused] {name} Lyr={Lyr} H={H} Hkv={Hkv} n_q={n_q} lengths={lens}")
    w = dataclasses.replace(small_workload(name, Lyr, H, Hkv, d, n_q, 0, cfg_id=170 + FUSED_BATCHES.index(case), hh=(1, 1000)),
                            batch=len(lengths))
    hh = synth.heavy_hitter_positions(w, lengths)
    q = synth.gen_q(w, len(lengths))
    ks = [synth.gen_k_layer(w, l, q, lengths, hh) for l in range(w.n_layers)]
    offsets = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    T = int(offsets[-1])
    n_launch = sp.sp_score_batch_is_fused(make_desc(Lyr, H, Hkv, d, n_q, w.scale, 0, "HND", T), [int(v) for v in offsets])
    assert n_launch >= (2 if "several" in name else 1)
    got = None
    for mode in (0, 1):
        got = gpu_score_batch(q, ks, offsets, w.scale, mode)
        for b, Lb in enumerate(lengths):
            if Lb == 0:
                continue
            sl = slice(int(offsets[b]), int(offsets[b + 1]))
            want = oracle.score(q[b], [np.ascontiguousarray(k[:, sl, :]) for k in ks], w.scale, mode)
            assert_scores_close(got[sl], want)
        say(f"  mode {mode}: ok")
    again = gpu_score_batch(q, ks, offsets, w.scale, 1)
    assert again.tobytes() == got.tobytes()
    nhd = [np.ascontiguousarray(k.transpose(1, 0, 2)) for k in ks]
    assert gpu_score_batch(q, nhd, offsets, w.scale, 1, layout="NHD").tobytes() == got.tobytes()


def test_score_mid_size_config():
    """The 16-layer, 32/8-head, head_dim-64 shape at L = 8192 (second workload), full element-wise parity."""
    from gpu_util import assert_scores_close, gpu_score
    say("[score] llama1b-8k full")
    w = synth.get_config("llama1b-8k")
    inp = synth.make_score_inputs(w)
    for mode in (0, 1):
        want = oracle.score(inp["q"][0], inp["k"], w.scale, mode)
        got = gpu_score(inp["q"][0], inp["k"], w.scale, mode)
        assert_scores_close(got, want)
        say(f"  mode {mode}: max rel err {np.max(np.abs(got - want) / want):.2e}")


@pytest.mark.parametrize("Lyr,Hkv,tiles", [(2, 2, 1), (2, 2, 24), (2, 2, 25), (4, 1, 24), (5, 1, 24), (1, 4, 24)])
@pytest.mark.parametrize("d", [64, 128])
def test_score_of_few_phases_in_one_range(Lyr, Hkv, tiles, d):
    """Three-kernel path: up to four phases and 24 tiles the prob pass takes all layers in one workgroup, beyond in ranges."""
    from gpu_util import assert_scores_close, gpu_score, score_path
    L = tiles * (256 if d == 64 else 128) - 19
    say(f"[score] few phases Lyr={Lyr} Hkv={Hkv} d={d} L={L}")
    w = small_workload("few", Lyr, 2 * Hkv, Hkv, d, 8, L, cfg_id=190, hh=(1, 100))
    inp = synth.make_score_inputs(w)
    for mode in (0, 1):
        got = gpu_score(inp["q"][0], inp["k"], w.scale, mode)
        assert score_path() == "general"
        assert_scores_close(got, oracle.score(inp["q"][0], inp["k"], w.scale, mode))


# Long single prompts take the single-launch kernel that keeps K on chip (head_dim 64: up to 64 padded
# query rows and 128K tokens; head_dim 128: up to 32 rows and 64K tokens).
FUSED_SHAPES = [
    # name, Lyr, H, Hkv, d, n_q, L
    ("fused_g4_nq16_tail", 2, 8, 2, 64, 16, 40000),       # 79 workgroups, 64-key tail
    ("fused_g4_nq8", 2, 8, 2, 64, 8, 33000),
    ("fused_g2_nq8_rows32", 3, 4, 2, 64, 8, 36001),
    ("fused_g8_nq8_two_gblocks", 1, 16, 2, 64, 8, 34000),
    ("fused_g3_nq5_padding", 2, 6, 2, 64, 5, 35000),
    ("fused_single_phase_full_grid", 1, 4, 1, 64, 16, 131072),
    ("fused_20_phases", 5, 8, 4, 64, 16, 40000),
    # the two kernel instantiations with a fixed model shape (16 layers, 32 / 8 heads): 8 and 16 lookahead rows
    ("fused_draft_model_nq8", 16, 32, 8, 64, 8, 33000),
    ("fused_draft_model_nq16", 16, 32, 8, 64, 16, 32768 + 513),
    ("fused_draft_model_nq8_full_grid", 16, 32, 8, 64, 8, 131072 - 100),     # 256 workgroups, ragged last tile
    # head_dim 128 (up to 32 padded query rows): 256 keys per workgroup, from 96 workgroups up
    ("fused_d128_g2_nq8", 3, 4, 2, 128, 8, 25000),                           # 98 workgroups, 168-key tail
    ("fused_d128_g4_nq8_rows32", 2, 8, 2, 128, 8, 24576 + 1),                # 1-key tail
    ("fused_d128_g2_nq5_padding", 2, 4, 2, 128, 5, 26000),
    ("fused_d128_g3_nq8_padding", 2, 6, 2, 128, 8, 25500),
    ("fused_d128_full_grid", 2, 4, 2, 128, 8, 65536 - 100),                  # 256 workgroups, ragged last tile
    ("fused_d128_28_phases", 7, 8, 4, 128, 8, 24576),
    ("fused_d128_40k", 2, 4, 2, 128, 8, 40000),
]


def test_which_prompts_take_the_single_launch_kernel():
    """The lengths at which sp_score changes kernels (sp_score_is_fused): head_dim 64 from 64 workgroups of
    512 keys up to 256; head_dim 128 from 96 workgroups of 256 keys up to 256, and only with at most 32
    padded query rows."""
    import paper_2603_02631_amd as sp
    from gpu_util import make_desc
    def fused(d, G, n_q, L):
        return sp.sp_score_is_fused(make_desc(2, 2 * G, 2, d, n_q, 0.1, 0, "HND", L), L)
    assert [fused(64, 4, 16, L) for L in (63 * 512, 63 * 512 + 1, 131072, 131073)] == [0, 1, 1, 0]
    assert [fused(128, 2, 8, L) for L in (95 * 256, 95 * 256 + 1, 65536, 65537)] == [0, 1, 1, 0]
    assert fused(128, 4, 8, 40000) == 1 and fused(128, 4, 16, 40000) == 0 and fused(128, 8, 8, 40000) == 0
    assert fused(64, 8, 16, 40000) == 0          # 128 padded rows


def test_which_batches_take_the_single_launch_kernel():
    """sp_score_batch_is_fused: 90 workgroups with the duty blocks (8 a prompt of 32 padded rows) of 10 prompts, or of 30."""
    import paper_2603_02631_amd as sp
    from gpu_util import make_desc
    def fused(n, tiles, shorten=0):
        off = np.arange(n + 1) * tiles * 512
        off[-1] -= shorten
        return sp.sp_score_batch_is_fused(make_desc(2, 8, 2, 64, 8, 0.1, 0, "HND", int(off[-1])), off)
    assert [fused(10, 9), fused(11, 8), fused(12, 8), fused(30, 3), fused(7, 9)] == [1, 1, 1, 0, 0]
    assert fused(13, 7) == 0 and fused(90, 3) == 0              # 91 workgroups, 104 duty blocks; three launches
    assert fused(8, 64) == 2 and fused(8, 64, 64 * 512 - 1) == 0     # a prompt shorter than a tile


@pytest.mark.parametrize("shape", FUSED_SHAPES, ids=[s[0] for s in FUSED_SHAPES])
def test_fused_score_matches_oracle(shape):
    import paper_2603_02631_amd as sp
    from gpu_util import assert_scores_close, gpu_score, make_desc
    name, Lyr, H, Hkv, d, n_q, L = shape
    say(f"[score-fused] {name} Lyr={Lyr} H={H} Hkv={Hkv} d={d} n_q={n_q} L={L}")
    w = small_workload(name, Lyr, H, Hkv, d, n_q, L, cfg_id=200 + FUSED_SHAPES.index(shape), hh=(1, 1000))
    assert sp.sp_score_is_fused(make_desc(Lyr, H, Hkv, d, n_q, w.scale, 0, "HND", L), L) == 1
    inp = synth.make_score_inputs(w)
    for mode in (0, 1):
        want = oracle.score(inp["q"][0], inp["k"], w.scale, mode)
        got = gpu_score(inp["q"][0], inp["k"], w.scale, mode)
        assert_scores_close(got, want)
        say(f"  mode {mode}: max rel err {np.max(np.abs(got - want) / want):.2e}")
    again = gpu_score(inp["q"][0], inp["k"], w.scale, 1)
    assert again.tobytes() == got.tobytes()          # deterministic
    nhd = [np.ascontiguousarray(k.transpose(1, 0, 2)) for k in inp["k"]]
    got_nhd = gpu_score(inp["q"][0], nhd, w.scale, 1, layout="NHD")
    assert got_nhd.tobytes() == got.tobytes()        # same keys through token-major strides


@pytest.mark.parametrize("workgroups", [64, 65, 66, 67, 68, 69, 70, 71])
def test_tiles_of_a_prompt_on_its_dies(workgroups):
    """Workgroups of a whole prompt take tiles by die: every remainder of the workgroup count by eight."""
    from gpu_util import assert_scores_close, gpu_score
    w = small_workload("dies", 1, 4, 1, 64, 8, workgroups * 512 - 77, cfg_id=240 + workgroups, hh=(1, 1000))
    inp = synth.make_score_inputs(w)
    assert_scores_close(gpu_score(inp["q"][0], inp["k"], w.scale, 0), oracle.score(inp["q"][0], inp["k"], w.scale, 0))


# Prompts that fill only part of the device: the layers run in ranges side by side and a last launch adds them up.
RANGE_SHAPES = [
    # name, Lyr, H, Hkv, d, n_q, lengths  (one: sp_score; several: sp_score_batch)
    ("ranges_16_of_1_layer", 16, 32, 8, 64, 8, [6200]),              # 13 workgroups, 56-key tail
    ("ranges_8_of_2_layers_rows64", 16, 32, 8, 64, 16, [8200]),      # 17 workgroups, 8-key tail
    ("ranges_two_gblocks", 12, 32, 4, 64, 8, [14000]),               # 28 workgroups: 6 ranges of 2 layers
    ("ranges_uneven_d128", 7, 8, 4, 128, 8, [13001]),                # 51 workgroups: layers 2 + 2 + 2 + 1
    ("ranges_d128_padding", 14, 8, 4, 128, 5, [4097]),               # 17 workgroups, 1-key tail
    ("ranges_batch", 12, 16, 4, 64, 8, [7600, 0, 2600, 3500]),       # 28 workgroups of three prompts: 9 -> 6 ranges
    ("ranges_batch_d128", 9, 8, 4, 128, 8, [9000, 300, 5000]),       # 58 workgroups: layers 3 + 3 + 3
    # prompts shorter than a tile: their tile starts with them, or ends with the packed keys (last prompt)
    ("ranges_short_prompts", 16, 32, 8, 64, 8, [4700, 60, 3000, 1, 511]),
    ("ranges_short_prompts_rows64", 14, 16, 4, 64, 16, [11000, 77, 600, 300]),
    ("ranges_short_prompts_d128", 14, 8, 4, 128, 8, [255, 3000, 2049, 64, 1500, 1]),
    # head_dim 128 with two blocks of query rows (five to eight heads a kv head)
    ("ranges_d128_g8", 24, 32, 4, 128, 8, [6001]),                   # 24 workgroups: 8 ranges of 3 layers
    ("ranges_d128_g5_padding", 24, 20, 4, 128, 5, [6200]),
    ("whole_d128_g8", 12, 8, 1, 128, 8, [45000]),                    # 176 workgroups, one range
    ("ranges_batch_d128_g8", 24, 32, 4, 128, 8, [6000, 300, 2000]),
    # further from the lines between the kernels
    ("ranges_6_rows64", 16, 32, 8, 64, 16, [17001]),
    ("ranges_16_rows64", 16, 32, 8, 64, 16, [8190]),
    ("ranges_4_two_gblocks", 16, 32, 4, 64, 8, [26000]),
    ("ranges_7_d128_padding", 14, 8, 4, 128, 5, [6145]),
    ("whole_d128_g8_long", 16, 8, 1, 128, 8, [57000]),
]
# The kernels these take: (tiles a workgroup, layer ranges, launches, "stand-in") of the single-launch kernel.
RANGE_PATHS = {
    "ranges_16_of_1_layer": (1, 16, 1, "stand-in"), "ranges_8_of_2_layers_rows64": "general", "ranges_two_gblocks": "general",
    "ranges_uneven_d128": (1, 4, 1, "stand-in"), "ranges_d128_padding": "general", "ranges_batch": (1, 6, 1, "stand-in"),
    "ranges_batch_d128": (1, 3, 1, "stand-in"), "ranges_short_prompts": (1, 8, 1, "stand-in"),
    "ranges_short_prompts_rows64": (1, 7, 1, "stand-in"), "ranges_short_prompts_d128": (1, 7, 1, "stand-in"),
    "ranges_d128_g8": (1, 8, 1, "stand-in"), "ranges_d128_g5_padding": (1, 8, 1, "stand-in"), "whole_d128_g8": (1, 1, 1, "stand-in"),
    "ranges_batch_d128_g8": (1, 6, 1, "stand-in"), "ranges_6_rows64": (1, 6, 1, "stand-in"), "ranges_16_rows64": (1, 16, 1, "stand-in"),
    "ranges_4_two_gblocks": (1, 4, 1, "stand-in"), "ranges_7_d128_padding": (1, 7, 1, "stand-in"),
    "whole_d128_g8_long": (1, 1, 1, "stand-in"),
}


@pytest.mark.parametrize("shape", RANGE_SHAPES, ids=[s[0] for s in RANGE_SHAPES])
def test_score_in_layer_ranges_matches_oracle(shape):
    from gpu_util import assert_scores_close, gpu_score, gpu_score_batch, score_path
    name, Lyr, H, Hkv, d, n_q, lens = shape
    lengths = np.array(lens, dtype=np.int64)
    say(f"[score-ranges] {name} Lyr={Lyr} H={H} Hkv={Hkv} d={d} n_q={n_q} lengths={lens}")
    w = dataclasses.replace(small_workload(name, Lyr, H, Hkv, d, n_q, 0, cfg_id=500 + RANGE_SHAPES.index(shape), hh=(1, 1000)),
                            batch=len(lengths))
    q = synth.gen_q(w, len(lengths))
    ks = [synth.gen_k_layer(w, l, q, lengths, synth.heavy_hitter_positions(w, lengths)) for l in range(Lyr)]
    offsets = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    run = (lambda mode, k, lay: gpu_score(q[0], k, w.scale, mode, layout=lay)) if len(lens) == 1 else \
          (lambda mode, k, lay: gpu_score_batch(q, k, offsets, w.scale, mode, layout=lay))
    for mode in (0, 1):
        got = run(mode, ks, "HND")
        assert score_path() == RANGE_PATHS[name]
        for b, Lb in enumerate(lengths):
            if Lb:
                sl = slice(int(offsets[b]), int(offsets[b + 1]))
                assert_scores_close(got[sl], oracle.score(q[b], [np.ascontiguousarray(k[:, sl, :]) for k in ks], w.scale, mode))
        assert run(mode, ks, "HND").tobytes() == got.tobytes()
        nhd = [np.ascontiguousarray(k.transpose(1, 0, 2)) for k in ks]
        assert run(mode, nhd, "NHD").tobytes() == got.tobytes()


def test_two_tiles_a_workgroup_want_room_for_the_exchange():
    """Two blocks of query rows at head_dim 128 exchange in the general path's buffers, which are too small with one phase."""
    from gpu_util import assert_scores_close, gpu_score, score_path
    w = small_workload("pair_no_room", 1, 8, 1, 128, 8, 70000, cfg_id=690, hh=(1, 1000))
    inp = synth.make_score_inputs(w)
    got = gpu_score(inp["q"][0], inp["k"], w.scale, 0)
    assert score_path() == "general"
    assert_scores_close(got, oracle.score(inp["q"][0], inp["k"], w.scale, 0))


@pytest.mark.parametrize("d,Lyr,H,Hkv,lens,path", [
    (64, 16, 32, 8, [4096], "general"), (64, 16, 32, 8, [4097], (1, 16, 1, "stand-in")), (128, 28, 16, 8, [1024], "general"),
    (128, 28, 16, 8, [1025], (1, 28, 1, "stand-in")), (64, 16, 32, 8, [2000, 60, 0, 1500, 800], (1, 16, 1, "stand-in")),
    (128, 28, 16, 8, [700, 1, 500, 257], (1, 14, 1, "stand-in"))])         # a launch's table holds 64 entries
def test_shortest_calls_on_the_single_launch_kernel(d, Lyr, H, Hkv, lens, path):
    """The last prompt on the three kernels, the first beyond it, and batches whose tiles hold as many keys."""
    from gpu_util import assert_scores_close, gpu_score, gpu_score_batch, score_path
    say(f"[score-line] d={d} Lyr={Lyr} lengths={lens}")
    lengths = np.array(lens, dtype=np.int64)
    w = dataclasses.replace(small_workload("line", Lyr, H, Hkv, d, 8, 0, cfg_id=560 + len(lens), hh=(1, 100)), batch=len(lengths))
    q = synth.gen_q(w, len(lengths))
    ks = [synth.gen_k_layer(w, l, q, lengths, synth.heavy_hitter_positions(w, lengths)) for l in range(Lyr)]
    offsets = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    for mode in (0, 1):
        got = gpu_score(q[0], ks, w.scale, mode) if len(lens) == 1 else gpu_score_batch(q, ks, offsets, w.scale, mode)
        assert score_path() == path
        for b, n in enumerate(lens):
            if n:
                sl = slice(int(offsets[b]), int(offsets[b + 1]))
                assert_scores_close(got[sl], oracle.score(q[b], [np.ascontiguousarray(k[:, sl, :]) for k in ks], w.scale, mode))


@pytest.mark.parametrize("d,Lyr,lens", [
    (64, 16, [316, 356, 455, 376, 1005, 1068, 2681, 888, 1599]), (128, 28, [163, 618, 402, 241, 331, 64, 131, 882]),
    (64, 16, [186, 323, 84, 2759, 1217, 154, 96, 117, 2021, 2796, 179, 1356, 838, 1508, 134, 734, 707, 264, 247, 317, 226, 82, 113, 680, 78,
              2689, 153, 446, 138, 124, 3477, 273, 244, 73, 751, 3359, 514, 955, 578])], ids=["one_launch", "d128", "two_launches"])
def test_batches_of_short_prompts_below_their_line(d, Lyr, lens):
    """Layer ranges of more than some 17 steps with several prompts: the three kernels take as many keys as they take of one
    prompt and more (19 to 28 % less time on these batches)."""
    from gpu_util import assert_scores_close, gpu_score_batch, score_path
    say(f"[score-line] batch of {len(lens)} prompts, d={d}")
    lengths = np.array(lens, dtype=np.int64)
    w = dataclasses.replace(small_workload("short_batch", Lyr, 32 if d == 64 else 16, 8, d, 8, 0, cfg_id=570 + d, hh=(1, 100)), batch=len(lens))
    q = synth.gen_q(w, len(lens))
    ks = [synth.gen_k_layer(w, l, q, lengths, synth.heavy_hitter_positions(w, lengths)) for l in range(Lyr)]
    offsets = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    got = gpu_score_batch(q, ks, offsets, w.scale, 0)
    assert score_path() == "general"
    for b in (0, len(lens) // 2, len(lens) - 1):
        sl = slice(int(offsets[b]), int(offsets[b + 1]))
        assert_scores_close(got[sl], oracle.score(q[b], [np.ascontiguousarray(k[:, sl, :]) for k in ks], w.scale, 0))


# More than one tile per compute unit: a workgroup owns two.
PAIR_SHAPES = [
    # name, Lyr, H, Hkv, d, n_q, L, page_tokens (0: contiguous keys, also with lookahead keys)
    ("pair_one_key_more", 1, 4, 1, 64, 8, 131073, 0),                # the last workgroup shifted back by 1023 keys
    ("pair_three_phases", 3, 2, 1, 64, 5, 140001, 0),
    ("pair_two_gblocks", 1, 8, 1, 64, 8, 150000, 0),
    ("pair_full_grid", 1, 4, 2, 64, 8, 262144, 0),
    ("pair_d128", 2, 4, 2, 128, 8, 65537, 0),
    ("pair_d128_full_grid", 1, 2, 1, 128, 8, 131072, 0),
    ("pair_paged_second_tile_empty", 2, 4, 1, 64, 8, 131072 + 500, 512),
    ("pair_paged_d128_tail", 1, 4, 2, 128, 8, 70000, 4096),
    ("pair_draft_model", 16, 32, 8, 64, 8, 131072 + 777, 0),
    # two blocks of query rows: more than eight lookahead rows, five to eight heads a kv head of 128
    ("pair_rows64", 2, 4, 1, 64, 16, 131073, 0),
    ("pair_rows64_padding", 1, 3, 1, 64, 11, 200001, 0),
    ("pair_rows64_paged", 2, 4, 1, 64, 9, 131072 + 500, 512),
    ("pair_rows64_full_grid", 1, 4, 2, 64, 16, 262144, 0),
    ("pair_rows64_draft_model", 16, 32, 8, 64, 16, 131072 + 777, 0),
    ("pair_d128_g8", 3, 8, 1, 128, 8, 65537, 0),
    ("pair_d128_g5_padding_full_grid", 4, 5, 1, 128, 5, 131072, 0),
    ("pair_d128_g8_paged", 3, 8, 1, 128, 8, 70000, 4096),
]


@pytest.mark.parametrize("shape", PAIR_SHAPES, ids=[s[0] for s in PAIR_SHAPES])
def test_score_with_two_tiles_a_workgroup_matches_oracle(shape):
    from gpu_util import assert_scores_close, gpu_score, gpu_score_look, gpu_score_paged, make_paged, score_path
    name, Lyr, H, Hkv, d, n_q, L, page = shape
    say(f"[score-pair] {name} Lyr={Lyr} H={H} Hkv={Hkv} d={d} n_q={n_q} L={L} page={page}")
    w = small_workload(name, Lyr, H, Hkv, d, n_q, L, cfg_id=600 + PAIR_SHAPES.index(shape), hh=(1, 1000))
    inp = synth.make_score_inputs(w)
    q, k = inp["q"][0], inp["k"]
    if page:
        pools, table = make_paged(k, page, "HND", seed=w.cfg_id)
        run = lambda mode: gpu_score_paged(q, pools, table, page, L, w.scale, mode, "HND")
    else:
        run = lambda mode: gpu_score(q, k, w.scale, mode)
    for mode in ((0,) if Lyr > 4 else (0, 1)):
        got = run(mode)
        assert score_path() == (2, 1, 1, "stand-in")
        assert_scores_close(got, oracle.score(q, k, w.scale, mode))
        assert run(mode).tobytes() == got.tobytes()
    if not page and Lyr <= 4:
        kl = synth.gen_look_keys(w, inp["q"])
        assert_scores_close(gpu_score_look(q, k, kl, 1, w.scale, 0), oracle.score_look(q, k, kl, 1, w.scale, 0))
        nhd = [np.ascontiguousarray(x.transpose(1, 0, 2)) for x in k]
        assert gpu_score(q, nhd, w.scale, mode, layout="NHD").tobytes() == got.tobytes()


def test_wide_query_groups_with_lookahead_and_paged_keys():
    """head_dim 128 with eight heads a kv head on the single-launch kernel: lookahead keys in the normaliser, paged keys."""
    from gpu_util import assert_scores_close, gpu_score_look, gpu_score_paged, make_paged, score_path
    Lyr, H, Hkv, d, n_q, L, page = 24, 32, 4, 128, 8, 6001, 512
    say(f"[score-wide] L={L}")
    w = small_workload("wide_group", Lyr, H, Hkv, d, n_q, L, cfg_id=650, hh=(1, 1000))
    inp = synth.make_score_inputs(w)
    q, k = inp["q"][0], inp["k"]
    kl = synth.gen_look_keys(w, inp["q"])
    for mode in (0, 1):
        assert_scores_close(gpu_score_look(q, k, kl, 1, w.scale, mode), oracle.score_look(q, k, kl, 1, w.scale, mode))
        assert score_path() == (1, 8, 1, "stand-in")
    pools, table = make_paged(k, page, "HND", seed=w.cfg_id)
    assert_scores_close(gpu_score_paged(q, pools, table, page, L, w.scale, 0, "HND"), oracle.score(q, k, w.scale, 0))
    assert score_path() == (1, 8, 1, "stand-in")


@pytest.mark.parametrize("Lyr,H,Hkv,n_q,L", [(1, 4, 1, 8, 191 * 256 + 1), (1, 2, 2, 8, 50000), (3, 3, 1, 5, 60001), (5, 4, 2, 8, 49152 + 77),
                                             (3, 8, 4, 8, 65536)])
def test_long_prompt_of_head_dim_128_with_its_probabilities_last(Lyr, H, Hkv, n_q, L):
    """From 192 workgroups on: fewer phases than are in flight, and several turns of the exchange ring; contiguous and paged
    keys, lookahead keys, both aggregation modes; a call that gives up."""
    import torch
    import paper_2603_02631_amd as sp
    from gpu_util import (DEV, assert_scores_close, dev_bits, gpu_score, gpu_score_look, gpu_score_paged, make_desc, make_paged, score_path,
                          status_word, workspace)
    say(f"[score-prob-last] Lyr={Lyr} H={H} Hkv={Hkv} n_q={n_q} L={L}")
    w = small_workload("prob_last", Lyr, H, Hkv, 128, n_q, L, cfg_id=660 + Lyr, hh=(1, 1000))
    inp = synth.make_score_inputs(w)
    q, k = inp["q"][0], inp["k"]
    pools, table = make_paged(k, 512, "HND", seed=w.cfg_id)
    kl = synth.gen_look_keys(w, inp["q"])
    for mode in (0, 1):
        want = oracle.score(q, k, w.scale, mode)
        got = gpu_score(q, k, w.scale, mode)
        assert score_path()[:3] == (1, 1, 1)
        assert_scores_close(got, want)
        assert gpu_score(q, k, w.scale, mode).tobytes() == got.tobytes()
        assert_scores_close(gpu_score_paged(q, pools, table, 512, L, w.scale, mode, "HND"), want)
        assert_scores_close(gpu_score_look(q, k, kl, 1, w.scale, mode), oracle.score_look(q, k, kl, 1, w.scale, mode))
    try:
        sp.sp_debug_fused_giveup(4, 1)
        desc = make_desc(Lyr, H, Hkv, 128, n_q, w.scale, 0, "HND", L)
        ws, scores = workspace(sp.sp_score_workspace(desc, L, 1)), torch.zeros(L, device=DEV)
        sp.sp_score(desc, dev_bits(q), [dev_bits(x) for x in k], L, scores, ws)
        torch.cuda.synchronize()
        assert status_word(ws) == 1 and bool(torch.isnan(scores).all())
    finally:
        sp.sp_debug_fused_giveup(1 << 20, 0)
    assert_scores_close(gpu_score(q, k, w.scale, 1), want)


def test_fused_score_gives_up_as_a_whole():
    """The bounded waits of the single-launch kernel, driven to give up from the host (the test hook
    makes the combining waves treat their partial results as never arriving, with a spin limit of a few
    polls, so every kernel still runs to its end): all scores NaN, status word 1; the next ordinary
    call on the same workspace is valid again."""
    import torch
    import paper_2603_02631_amd as sp
    from gpu_util import DEV, dev_bits, make_desc, status_word, workspace
    Lyr, H, Hkv, d, n_q, L = 2, 8, 2, 64, 16, 40000
    w = small_workload("fused_give_up", Lyr, H, Hkv, d, n_q, L, cfg_id=290, hh=(1, 1000))
    inp = synth.make_score_inputs(w)
    desc = make_desc(Lyr, H, Hkv, d, n_q, w.scale, 0, "HND", L)
    assert sp.sp_score_is_fused(desc, L) == 1
    qd = dev_bits(inp["q"][0])
    kd = [dev_bits(k) for k in inp["k"]]
    ws = workspace(sp.sp_score_workspace(desc, L, 1))
    scores = torch.zeros(L, dtype=torch.float32, device=DEV)
    say("[score-fused] give-up path: spin limit 4, partials treated as missing")
    try:
        sp.sp_debug_fused_giveup(4, 1)
        sp.sp_score(desc, qd, kd, L, scores, ws)
        torch.cuda.synchronize()
    finally:
        sp.sp_debug_fused_giveup(1 << 20, 0)
    assert status_word(ws) == 1
    assert bool(torch.isnan(scores).all())
    say("[score-fused] ordinary call on the same workspace")
    sp.sp_score(desc, qd, kd, L, scores, ws)
    torch.cuda.synchronize()
    assert status_word(ws) == 0
    from gpu_util import assert_scores_close
    assert_scores_close(scores.cpu().numpy(), oracle.score(inp["q"][0], inp["k"], w.scale, 0))


@pytest.mark.parametrize("Lyr,Hkv,tiles,launches,ranges,prompt", [(2, 2, [128, 128, 64], 2, 1, 0), (2, 2, [128, 128, 64], 2, 1, 2),
                                                                  (6, 8, [90, 70, 50, 40, 12], 3, 2, 0), (6, 8, [90, 70, 50, 40, 12], 3, 2, 4)])
def test_batch_of_several_launches_gives_up_as_a_whole(Lyr, Hkv, tiles, launches, ranges, prompt):
    """One launch gives up, the other ones' prompts lose their scores too: launches of all layers (128 + 128 workgroups and
    64) and of two layer ranges side by side, whose last launch adds the ranges up."""
    import torch
    import paper_2603_02631_amd as sp
    from gpu_util import DEV, score_path, status_word, workspace
    B, H, d, n_q = len(tiles), 4 * Hkv, 64, 8
    off = [512 * sum(tiles[:b]) for b in range(B + 1)]
    say(f"[score-batch] give-up of the launch that holds prompt {prompt}, {ranges} range(s)")
    g = torch.Generator(device=DEV).manual_seed(5)
    q = torch.randn((B, Lyr, H, n_q, d), device=DEV, generator=g).to(torch.bfloat16)
    k = [torch.randn((Hkv, off[-1], d), device=DEV, generator=g).to(torch.bfloat16) for _ in range(Lyr)]
    desc = sp.ScoreDesc(Lyr, H, Hkv, d, n_q, 0.125, sp.SP_LAYER_MEAN, d, off[-1] * d)
    assert sp.sp_score_batch_is_fused(desc, off) == launches
    ws = workspace(sp.sp_score_workspace(desc, off[-1], B))
    od = torch.tensor(off, dtype=torch.int64, device=DEV)
    scores = torch.zeros(off[-1], dtype=torch.float32, device=DEV)
    for _ in range(600):                        # one stream only, whatever ran before: nothing stands in
        sp.sp_score_batch(desc, q, k, off, od, scores, ws)
    assert score_path() == (1, ranges, launches)
    try:
        sp.sp_debug_fused_giveup(4, 2 + prompt)
        sp.sp_score_batch(desc, q, k, off, od, scores, ws)
        torch.cuda.synchronize()
    finally:
        sp.sp_debug_fused_giveup(1 << 20, 0)
    assert status_word(ws) == 1
    assert bool(torch.isnan(scores).all())
    sp.sp_score_batch(desc, q, k, off, od, scores, ws)
    torch.cuda.synchronize()
    assert status_word(ws) == 0
    for b in range(B):
        s = scores[off[b]:off[b + 1]]
        assert bool(torch.isfinite(s).all()) and 0.99 < float(s.double().sum()) < H


@pytest.mark.parametrize("tiles", [[150, 106, 100, 100, 56], [200, 3, 60, 17, 2, 30]],
                         ids=["only_first_fit_fits", "shared_out_evenly"])
def test_batch_of_several_launches_matches_oracle(tiles):
    """512 and 312 workgroups in two launches of at most 256: sharing them out evenly, longest prompt first, leaves no room
    for the last prompt of the first batch."""
    from gpu_util import assert_scores_close, gpu_score_batch, score_path
    say(f"[score-batch] tiles {tiles}")
    lengths = np.array([512 * t - 9 * i for i, t in enumerate(tiles)], dtype=np.int64)
    w = dataclasses.replace(small_workload("launches", 1, 4, 1, 64, 8, 0, cfg_id=470 + len(tiles), hh=(1, 1000)), batch=len(tiles))
    q = synth.gen_q(w, len(tiles))
    ks = [synth.gen_k_layer(w, 0, q, lengths, synth.heavy_hitter_positions(w, lengths))]
    offsets = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    got = gpu_score_batch(q, ks, offsets, w.scale, 0)
    assert score_path()[:3] == (1, 1, 2)
    for b in range(len(tiles)):
        sl = slice(int(offsets[b]), int(offsets[b + 1]))
        assert_scores_close(got[sl], oracle.score(q[b], [np.ascontiguousarray(ks[0][:, sl, :])], w.scale, 0))


@pytest.mark.parametrize("d,tiles,last,path", [(64, [90, 70, 50, 40, 12], 512, (1, 2, 3)),
                                               (128, [80, 60, 0, 50, 40, 35], 100, (1, 2, 3, "stand-in"))], ids=["announced", "short_prompt_d128"])
def test_batch_in_layer_ranges_on_several_launches(d, tiles, last, path):
    """Batches of a little more than one launch: three launches of two layer ranges instead of two of one; the second batch
    ends with a prompt shorter than a tile."""
    from gpu_util import assert_scores_close, gpu_score_batch, score_path
    say(f"[score-batch] ranges on several launches, d={d} tiles={tiles}")
    tile, Lyr, Hkv = 32768 // d, 6, 8
    lengths = np.array([tile * t - 5 * (t > 0) for t in tiles] + [last], dtype=np.int64)
    w = dataclasses.replace(small_workload("spread", Lyr, 2 * Hkv, Hkv, d, 8, 0, cfg_id=480 + d, hh=(1, 1000)), batch=len(lengths))
    q = synth.gen_q(w, len(lengths))
    ks = [synth.gen_k_layer(w, l, q, lengths, synth.heavy_hitter_positions(w, lengths)) for l in range(Lyr)]
    offsets = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    for mode in (0, 1):
        got = gpu_score_batch(q, ks, offsets, w.scale, mode)
        assert score_path() == path
        for b in ((0, len(lengths) - 1) if mode else range(len(lengths))):
            sl = slice(int(offsets[b]), int(offsets[b + 1]))
            if lengths[b]:
                assert_scores_close(got[sl], oracle.score(q[b], [np.ascontiguousarray(k[:, sl, :]) for k in ks], w.scale, mode))


def test_batch_of_one_launch_gives_up_as_a_whole():
    """Two prompts of 64 workgroups each and a single (layer, kv head); the last workgroup of the second prompt is missing.
    What waits for its partial results gives up after some milliseconds, when workgroups of the first prompt are
    finished; the first prompt loses its scores all the same."""
    import torch
    import paper_2603_02631_amd as sp
    from gpu_util import DEV, score_path, status_word, workspace
    Lyr, H, Hkv, d, n_q = 1, 4, 1, 64, 8
    off = [0, 32768, 65536]
    say("[score-batch] give-up of one prompt of a launch")
    g = torch.Generator(device=DEV).manual_seed(6)
    q = torch.randn((2, Lyr, H, n_q, d), device=DEV, generator=g).to(torch.bfloat16)
    k = [torch.randn((Hkv, off[-1], d), device=DEV, generator=g).to(torch.bfloat16) for _ in range(Lyr)]
    desc = sp.ScoreDesc(Lyr, H, Hkv, d, n_q, 0.125, sp.SP_LAYER_MEAN, d, off[-1] * d)
    assert sp.sp_score_batch_is_fused(desc, off) == 1
    ws = workspace(sp.sp_score_workspace(desc, off[-1], 2))
    od = torch.tensor(off, dtype=torch.int64, device=DEV)
    scores = torch.zeros(off[-1], dtype=torch.float32, device=DEV)
    for _ in range(600):                        # calls of one stream, whatever ran before: no stand-in
        sp.sp_score_batch(desc, q, k, off, od, scores, ws)
    assert score_path() == (1, 1, 1)
    try:
        sp.sp_debug_fused_giveup(1 << 12, -1)
        sp.sp_score_batch(desc, q, k, off, od, scores, ws)
        torch.cuda.synchronize()
    finally:
        sp.sp_debug_fused_giveup(1 << 20, 0)
    assert status_word(ws) == 1
    assert bool(torch.isnan(scores).all())
    sp.sp_score_batch(desc, q, k, off, od, scores, ws)
    torch.cuda.synchronize()
    assert status_word(ws) == 0
    for b in range(2):
        s = scores[off[b]:off[b + 1]]
        assert bool(torch.isfinite(s).all()) and 0.99 < float(s.double().sum()) < H


# Calls that take the single-launch kernel although sp_score_is_fused does not say so.
STAND_IN_SHAPES = [
    # name, entry, Lyr, H, Hkv, d, n_q, lengths
    ("ranges", "prompt", 16, 32, 8, 64, 8, [6200]),
    ("ranges_rows64", "prompt", 16, 32, 8, 64, 16, [20100]),
    ("ranges_two_gblocks", "prompt", 12, 32, 4, 64, 8, [24000]),
    ("ranges_d128_padding", "prompt", 14, 8, 4, 128, 5, [8000]),
    ("ranges_d128_g8", "prompt", 24, 32, 4, 128, 8, [6001]),
    ("whole_d128_g8", "prompt", 12, 8, 1, 128, 8, [50000]),
    ("direct_d128", "prompt", 28, 16, 8, 128, 8, [1700]),
    ("pair", "prompt", 2, 4, 1, 64, 8, [131073]),
    ("pair_d128", "prompt", 1, 4, 2, 128, 8, [70000]),
    ("batch_ranges_short_prompts", "batch", 16, 32, 8, 64, 8, [4700, 60, 0, 3000, 1, 511]),
    ("batch_one_range_short_prompt", "batch", 4, 8, 2, 64, 8, [110000, 100, 0, 3000]),
    ("batch_ranges_d128_g8", "batch", 24, 32, 4, 128, 8, [6000, 300, 2000]),
    ("look_ranges", "look", 16, 32, 8, 64, 8, [6200]),
    ("paged_ranges", "paged", 16, 32, 8, 64, 8, [6200]),
    ("paged_pair", "paged", 2, 4, 1, 64, 8, [131072 + 500]),
    ("fp8_ranges", "fp8", 16, 32, 8, 64, 8, [30000]),
    ("fp8_direct_d128", "fp8", 28, 16, 8, 128, 8, [1700]),
    ("fp8_pair", "fp8", 2, 4, 1, 64, 8, [147457]),
    ("pair_rows64", "prompt", 2, 4, 1, 64, 16, [131073]),
    ("pair_d128_g8", "prompt", 3, 8, 1, 128, 8, [70000]),
    ("fp8_pair_rows64", "fp8", 2, 4, 1, 64, 16, [147457]),
    ("batch_ranges_on_several_launches", "batch", 6, 16, 8, 128, 8, [20480, 15360, 0, 12800, 10240, 8960, 100]),
]


@pytest.mark.parametrize("shape", STAND_IN_SHAPES, ids=[s[0] for s in STAND_IN_SHAPES])
def test_calls_that_are_not_announced_as_fused_never_fail(shape):
    """sp_score_is_fused (sp_score_batch_is_fused) answers 0: where the single-launch kernel gives up, driven to it from
    the host, the call still ends with the scores and status 0; the same call without it does not need the stand-in."""
    import paper_2603_02631_amd as sp
    import gpu_util as u
    name, entry, Lyr, H, Hkv, d, n_q, lens = shape
    say(f"[score-stand-in] {name} {entry} Lyr={Lyr} H={H} Hkv={Hkv} d={d} n_q={n_q} lengths={lens}")
    lengths = np.array(lens, dtype=np.int64)
    total = int(lengths.sum())
    w = dataclasses.replace(small_workload(name, Lyr, H, Hkv, d, n_q, 0, cfg_id=700 + STAND_IN_SHAPES.index(shape), hh=(1, 1000)),
                            batch=len(lengths))
    q = synth.gen_q(w, len(lengths))
    ks = [synth.gen_k_layer(w, l, q, lengths, synth.heavy_hitter_positions(w, lengths)) for l in range(Lyr)]
    offsets = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    kl = synth.gen_look_keys(w, q)
    if entry == "fp8":
        codes, kscale = zip(*[synth.quantise_k_e4m3(k) for k in ks])
        codes, kscale = list(codes), np.stack(kscale)
    if entry == "paged":
        pools, table = u.make_paged(ks, 512, "HND", seed=w.cfg_id)
    desc = u.make_desc(Lyr, H, Hkv, d, n_q, w.scale, 0, "HND", total)
    query = {"batch": lambda: sp.sp_score_batch_is_fused(desc, offsets), "fp8": lambda: sp.sp_score_fp8_is_fused(desc, total)}
    assert query.get(entry, lambda: sp.sp_score_is_fused(desc, total))() == 0
    for mode in (0, 1):
        run = {"prompt": lambda: u.gpu_score(q[0], ks, w.scale, mode),
               "batch": lambda: u.gpu_score_batch(q, ks, offsets, w.scale, mode),
               "look": lambda: u.gpu_score_look(q[0], ks, kl, 1, w.scale, mode),
               "paged": lambda: u.gpu_score_paged(q[0], pools, table, 512, total, w.scale, mode),
               "fp8": lambda: u.gpu_score_fp8(q[0], codes, kscale, w.scale, mode)}[entry]
        try:
            sp.sp_debug_fused_giveup(4, 1)
            got = run()
            assert u.last_call_gave_up() and u.score_path()[3] == "stand-in"
        finally:
            sp.sp_debug_fused_giveup(1 << 20, 0)
        plain = run()
        assert not u.last_call_gave_up()
        for b, Lb in enumerate(lengths):
            if Lb:
                sl = slice(int(offsets[b]), int(offsets[b + 1]))
                part = [np.ascontiguousarray(k[:, sl, :]) for k in ks]
                want = oracle.score_look(q[b], part, kl, 1, w.scale, mode) if entry == "look" else \
                    oracle.score_fp8(q[b], codes, kscale.astype(np.float64), w.scale, mode) if entry == "fp8" else oracle.score(q[b], part, w.scale, mode)
                u.assert_scores_close(got[sl], want)
                u.assert_scores_close(plain[sl], want)


LOOK_SHAPES = [
    # name, Lyr, H, Hkv, d, n_q, L   (general path: short prompts, head_dim 128; fused path: long prompts)
    ("look_g4_nq16_d64", 3, 8, 2, 64, 16, 1500),
    ("look_g2_nq8_d128", 2, 4, 2, 128, 8, 777),
    ("look_g3_nq5_d64", 2, 6, 2, 64, 5, 333),
    ("look_nq1_d64", 2, 4, 2, 64, 1, 300),
    ("look_fused_g4_nq16", 3, 8, 2, 64, 16, 33000),
    ("look_fused_g3_nq5_padding", 2, 6, 2, 64, 5, 35000),
    ("look_fused_d128_g2_nq8", 2, 4, 2, 128, 8, 25000),
]


@pytest.mark.parametrize("shape", LOOK_SHAPES, ids=[s[0] for s in LOOK_SHAPES])
def test_score_with_lookahead_keys_matches_oracle(shape):
    """sp_score_look: the rows' normalisers include their visible lookahead keys
    (Algorithm 1, ForwardWithAttn at lookahead = i); both visibility settings and
    both aggregation modes, on both kernels."""
    import paper_2603_02631_amd as sp
    from gpu_util import assert_scores_close, gpu_score, gpu_score_look, make_desc
    name, Lyr, H, Hkv, d, n_q, L = shape
    say(f"[score-look] {name} Lyr={Lyr} H={H} Hkv={Hkv} d={d} n_q={n_q} L={L}")
    w = small_workload(name, Lyr, H, Hkv, d, n_q, L, cfg_id=300 + LOOK_SHAPES.index(shape), hh=(1, 1000))
    fused = sp.sp_score_is_fused(make_desc(Lyr, H, Hkv, d, n_q, w.scale, 0, "HND", L), L)
    assert fused == (1 if "fused" in name else 0)
    inp = synth.make_score_inputs(w)
    q = inp["q"][0]
    kl = synth.gen_look_keys(w, inp["q"])
    plain = oracle.score(q, inp["k"], w.scale, 0)
    for look_self in (0, 1):
        for mode in (0, 1):
            want = oracle.score_look(q, inp["k"], kl, look_self, w.scale, mode)
            got = gpu_score_look(q, inp["k"], kl, look_self, w.scale, mode)
            assert_scores_close(got, want)
            say(f"  self {look_self} mode {mode}: max rel err {np.max(np.abs(got - want) / want):.2e}")
    # the term matters on these inputs, well above the tolerance (a test that passes without it would prove nothing)
    assert np.max(np.abs(oracle.score_look(q, inp["k"], kl, 1, w.scale, 0) - plain) / plain) > 5e-3
    # and a call without lookahead keys afterwards is the plain result again (no state left behind)
    assert_scores_close(gpu_score(q, inp["k"], w.scale, 0), plain)


@pytest.mark.parametrize("Lyr,H,Hkv,n_q,L,tiles,in_ranges", [
    (2, 8, 2, 16, 33000, 1, False),         # all layers in one launch entry, most workgroups only clear
    (1, 4, 1, 16, 131072, 1, False),        # one phase, the largest area: more words than threads that clear
    (16, 32, 8, 8, 6200, 1, True),          # layer ranges: the area lies elsewhere
    (2, 4, 1, 8, 140001, 2, False),         # two tiles a workgroup
])
def test_lookahead_call_on_a_workspace_that_holds_an_earlier_call(Lyr, H, Hkv, n_q, L, tiles, in_ranges):
    """What an earlier call exchanged is well-formed data of the same phases: a call that finds any of it takes wrong
    normalisers. Same bits as on a fresh workspace (the reductions have a fixed order)."""
    import torch
    import paper_2603_02631_amd as sp
    from gpu_util import DEV, make_desc, score_path, workspace
    say(f"[look-stale] Lyr={Lyr} H={H} Hkv={Hkv} n_q={n_q} L={L}")
    desc = make_desc(Lyr, H, Hkv, 64, n_q, 0.125, 0, "HND", L)
    g = torch.Generator(device=DEV).manual_seed(L)

    def inputs(spread):
        make = lambda *shape: torch.randn(shape, device=DEV, generator=g).mul_(spread).to(torch.bfloat16)
        return make(Lyr, H, n_q, 64), [make(Hkv, L, 64) for _ in range(Lyr)], make(Lyr, Hkv, n_q, 64)

    def call(ws, q, k, kl):
        scores = torch.full((L,), float("nan"), device=DEV)
        sp.sp_score_look(desc, q, k, L, kl, 1, scores, ws)
        torch.cuda.synchronize()
        return scores.cpu()

    first, second = inputs(1.5), inputs(1.0)
    size = sp.sp_score_workspace(desc, L, 1)
    used = workspace(size)
    stale = call(used, *first)
    got = call(used, *second)
    path = score_path()
    assert path[0] == tiles and (path[1] > 1) == in_ranges, path
    want = call(workspace(size), *second)
    assert torch.isfinite(want).all() and not torch.equal(stale, want)
    assert torch.equal(got, want)


PAGED_SHAPES = [
    # name, Lyr, H, Hkv, d, n_q, L, page_tokens, layout
    ("paged_general_d64", 3, 8, 2, 64, 16, 1500, 512, "HND"),
    ("paged_general_d128_nhd", 2, 4, 2, 128, 8, 777, 512, "NHD"),
    ("paged_general_one_page", 2, 4, 2, 64, 8, 300, 1024, "HND"),
    ("paged_fused_4k_ragged_tail", 3, 8, 2, 64, 16, 33000 + 77, 4096, "HND"),
    ("paged_fused_4k_whole_pages", 2, 8, 2, 64, 8, 8 * 4096, 4096, "HND"),
    ("paged_fused_512_nhd", 2, 6, 2, 64, 5, 35000, 512, "NHD"),
    ("paged_fused_d128_2k_ragged_tail", 2, 4, 2, 128, 8, 25000 + 77, 2048, "HND"),
    ("paged_fused_d128_512_nhd", 2, 4, 2, 128, 5, 24600, 512, "NHD"),
    ("paged_fused_d128_40k_4k_pages", 1, 4, 2, 128, 8, 40000 + 5, 4096, "HND"),
]


@pytest.mark.parametrize("shape", PAGED_SHAPES, ids=[s[0] for s in PAGED_SHAPES])
def test_score_over_paged_keys_matches_oracle(shape):
    """sp_score_paged: the keys sit in shuffled pages of per-layer pools (Section 3.1: KV caches in
    fixed-size blocks); rows that hold no token are NaN. Oracle: the plain score of the keys gathered
    through the block table."""
    import paper_2603_02631_amd as sp
    from gpu_util import assert_scores_close, gpu_score_paged, make_desc, make_paged
    name, Lyr, H, Hkv, d, n_q, L, P, layout = shape
    say(f"[score-paged] {name} Lyr={Lyr} H={H} Hkv={Hkv} d={d} n_q={n_q} L={L} page={P} {layout}")
    w = small_workload(name, Lyr, H, Hkv, d, n_q, L, cfg_id=400 + PAGED_SHAPES.index(shape), hh=(1, 1000))
    fused = sp.sp_score_is_fused(make_desc(Lyr, H, Hkv, d, n_q, w.scale, 0, layout, P), L)
    assert fused == (1 if "fused" in name else 0)
    inp = synth.make_score_inputs(w)
    q = inp["q"][0]
    pools, table = make_paged(inp["k"], P, layout, seed=w.cfg_id)
    gathered = [oracle.gather_pages(pool, table, L, layout) for pool in pools]
    for l in range(Lyr):                      # the scatter of the test and the oracle's gather are inverse
        ref = inp["k"][l] if layout == "HND" else inp["k"][l].transpose(1, 0, 2)
        np.testing.assert_array_equal(gathered[l], ref)
    for mode in (0, 1):
        want = oracle.score(q, gathered, w.scale, mode, layout=layout)
        got = gpu_score_paged(q, pools, table, P, L, w.scale, mode, layout)
        assert_scores_close(got, want)
        say(f"  mode {mode}: max rel err {np.max(np.abs(got - want) / want):.2e}")


@pytest.mark.parametrize("n_streams", [2, 4])
def test_scores_on_several_streams_at_once(n_streams):
    """Single-launch kernels on different streams take turns: every call ends with the scores it has alone."""
    import torch
    import paper_2603_02631_amd as sp
    from gpu_util import score_path
    dev = "cuda:0"
    say(f"[score-streams] {n_streams} streams")
    calls = []
    for i, L in enumerate([8200, 20001, 6200, 33000][:n_streams]):
        g = torch.Generator(device=dev).manual_seed(i)
        q = torch.randn((16, 32, 8, 64), device=dev, generator=g).to(torch.bfloat16)
        k = [torch.randn((8, L, 64), device=dev, generator=g).to(torch.bfloat16) for _ in range(16)]
        desc = sp.ScoreDesc(16, 32, 8, 64, 8, 0.125, sp.SP_LAYER_MEAN, 64, L * 64)
        ws = torch.empty(sp.sp_score_workspace(desc, L, 1), dtype=torch.uint8, device=dev)
        out = torch.zeros(L, dtype=torch.float32, device=dev)
        sp.sp_score(desc, q, k, L, out, ws)
        assert score_path()[1] > 1
        calls.append((desc, q, k, L, out, ws, out.clone(), torch.cuda.Stream()))
    torch.cuda.synchronize()
    for _ in range(20):
        for desc, q, k, L, out, ws, _, stream in calls:
            with torch.cuda.stream(stream):
                out.fill_(-1.0)
                sp.sp_score(desc, q, k, L, out, ws)
    torch.cuda.synchronize()
    for *_, out, ws, want, _ in calls:
        assert torch.equal(out, want)


def test_calls_that_cannot_be_ordered_never_fail():
    """Calls of one stream leave nothing that another stream could wait for. Until that stream calls again, calls from
    another one have a stand-in, also where sp_score_is_fused answers 1; driven to give up from the host."""
    import torch
    import paper_2603_02631_amd as sp
    from gpu_util import DEV, assert_scores_close, dev_bits, make_desc, status_word, workspace
    Lyr, H, Hkv, d, n_q = 1, 4, 1, 64, 8
    calls = []
    for L in (70000, 40000):
        w = small_workload("unordered", Lyr, H, Hkv, d, n_q, L, cfg_id=291, hh=(1, 1000))
        inp = synth.make_score_inputs(w)
        desc = make_desc(Lyr, H, Hkv, d, n_q, w.scale, 0, "HND", L)
        assert sp.sp_score_is_fused(desc, L) == 1
        calls.append((desc, dev_bits(inp["q"][0]), [dev_bits(k) for k in inp["k"]], L, torch.zeros(L, dtype=torch.float32, device=DEV),
                      workspace(sp.sp_score_workspace(desc, L, 1)), oracle.score(inp["q"][0], inp["k"], w.scale, 0)))
    other = torch.cuda.Stream()

    def call(c, stream=None):
        with torch.cuda.stream(stream):
            sp.sp_score(*c[:6])
        torch.cuda.synchronize()

    def gives_up(c, stream=None):
        try:
            sp.sp_debug_fused_giveup(4, 1)
            call(c, stream)
        finally:
            sp.sp_debug_fused_giveup(1 << 20, 0)
        return status_word(c[5]) == 1 and bool(torch.isnan(c[4]).all())

    say("[score-unordered]")
    for _ in range(600):                        # one stream only, whatever ran before
        sp.sp_score(*calls[0][:6])
    assert gives_up(calls[0])
    for c in calls:
        assert not gives_up(c, other)
        assert status_word(c[5]) == 0
        assert_scores_close(c[4].cpu().numpy(), c[6])
    call(calls[0])                              # the first stream's earlier calls lie before this one's event
    for stream in (other, None):
        for c in calls:
            assert gives_up(c, stream)
            call(c, stream)
            assert status_word(c[5]) == 0
            assert_scores_close(c[4].cpu().numpy(), c[6])


@pytest.mark.parametrize("shape", [("short", 16, 32, 8, 64, 8, 6200), ("two_tiles", 1, 4, 1, 64, 8, 150000), ("announced", 2, 8, 2, 64, 8, 40000)],
                         ids=lambda s: s[0])
def test_scores_on_a_stream_with_a_compute_unit_mask(shape):
    """128 of the device's compute units: nothing is launched whose workgroups would have to wait for others to end."""
    import ctypes
    import torch
    import paper_2603_02631_amd as sp
    from gpu_util import DEV, assert_scores_close, dev_bits, last_call_gave_up, make_desc, status_word, workspace
    name, Lyr, H, Hkv, d, n_q, L = shape
    say(f"[score-mask] {name} L={L}")
    w = small_workload(name, Lyr, H, Hkv, d, n_q, L, cfg_id=292, hh=(1, 1000))
    inp = synth.make_score_inputs(w)
    desc = make_desc(Lyr, H, Hkv, d, n_q, w.scale, 0, "HND", L)
    qd, kd = dev_bits(inp["q"][0]), [dev_bits(k) for k in inp["k"]]
    scores, ws = torch.zeros(L, dtype=torch.float32, device=DEV), workspace(sp.sp_score_workspace(desc, L, 1))
    torch.cuda.synchronize()
    hip, stream = ctypes.CDLL("libamdhip64.so.7"), ctypes.c_void_p()
    mask = (ctypes.c_uint32 * 8)(*[0xFFFFFFFF] * 4, *[0] * 4)
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(stream), 8, mask) == 0
    try:
        sp.sp_score(desc, qd, kd, L, scores, ws, stream=stream.value)
        assert hip.hipStreamSynchronize(stream) == 0
    finally:
        assert hip.hipStreamDestroy(stream) == 0
    assert status_word(ws) == 0 and not last_call_gave_up()
    assert_scores_close(scores.cpu().numpy(), oracle.score(inp["q"][0], inp["k"], w.scale, 0))


def test_batch_on_a_stream_with_a_compute_unit_mask():
    """128 compute units and an announced batch whose first launch has more workgroups: neither even launches nor layer
    ranges, which would fit, put it on the single-launch kernel there."""
    import ctypes
    import torch
    import paper_2603_02631_amd as sp
    from gpu_util import DEV, assert_scores_close, dev_bits, gpu_score_batch, make_desc, score_path, status_word, workspace
    say("[score-mask] batch")
    lengths = np.array([512 * t - 5 for t in (90, 70, 50, 40, 12)], dtype=np.int64)
    w = dataclasses.replace(small_workload("mask", 6, 16, 8, 64, 8, 0, cfg_id=293, hh=(1, 1000)), batch=len(lengths))
    q, T = synth.gen_q(w, len(lengths)), int(lengths.sum())
    ks = [synth.gen_k_layer(w, l, q, lengths, synth.heavy_hitter_positions(w, lengths)) for l in range(6)]
    offsets = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    gpu_score_batch(q, ks, offsets, w.scale, 0)
    assert score_path()[:3] == (1, 2, 3)
    desc = make_desc(6, 16, 8, 64, 8, w.scale, 0, "HND", T)
    qd, kd, off_d = dev_bits(q), [dev_bits(k) for k in ks], torch.from_numpy(offsets).to(DEV)
    scores, ws = torch.zeros(T, dtype=torch.float32, device=DEV), workspace(sp.sp_score_workspace(desc, T, len(lengths)))
    torch.cuda.synchronize()
    hip, stream = ctypes.CDLL("libamdhip64.so.7"), ctypes.c_void_p()
    mask = (ctypes.c_uint32 * 8)(*[0xFFFFFFFF] * 4, *[0] * 4)
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(stream), 8, mask) == 0
    try:
        sp.sp_score_batch(desc, qd, kd, [int(v) for v in offsets], off_d, scores, ws, stream=stream.value)
        path = score_path()
        assert hip.hipStreamSynchronize(stream) == 0
    finally:
        assert hip.hipStreamDestroy(stream) == 0
    assert path == "general"
    assert status_word(ws) == 0
    for b in range(len(lengths)):
        sl = slice(int(offsets[b]), int(offsets[b + 1]))
        assert_scores_close(scores[sl].cpu().numpy(), oracle.score(q[b], [np.ascontiguousarray(k[:, sl, :]) for k in ks], w.scale, 0))


@pytest.mark.parametrize("tiles,launches,ranges", [([90, 70, 50, 40, 12], 3, 2), ([250, 249, 120], 3, 1)], ids=["ranges", "whole"])
def test_captured_batch_runs_as_it_is_announced(tiles, launches, ranges):
    """An announced batch of several launches: a recorded call makes the launches that sp_score_batch_is_fused counts, and every
    replay gives the eager call's scores bit for bit (mean over layers: the order of summation is the same)."""
    import torch
    import paper_2603_02631_amd as sp
    from gpu_util import DEV, score_path, status_word, workspace
    Lyr, H, Hkv, d, n_q, B = 6, 16, 8, 64, 8, len(tiles)
    off = [512 * sum(tiles[:b]) - 7 * b for b in range(B + 1)]
    say(f"[score-capture] batch of {launches} launches, {ranges} range(s)")
    g = torch.Generator(device=DEV).manual_seed(7)
    q = torch.randn((B, Lyr, H, n_q, d), device=DEV, generator=g).to(torch.bfloat16)
    k = [torch.randn((Hkv, off[-1], d), device=DEV, generator=g).to(torch.bfloat16) for _ in range(Lyr)]
    desc = sp.ScoreDesc(Lyr, H, Hkv, d, n_q, 0.125, sp.SP_LAYER_MEAN, d, off[-1] * d)
    assert sp.sp_score_batch_is_fused(desc, off) == launches
    ws = workspace(sp.sp_score_workspace(desc, off[-1], B))
    od = torch.tensor(off, dtype=torch.int64, device=DEV)
    eager, out = (torch.zeros(off[-1], dtype=torch.float32, device=DEV) for _ in range(2))
    sp.sp_score_batch(desc, q, k, off, od, eager, ws)
    assert score_path()[:3] == (1, ranges, launches)
    torch.cuda.synchronize()
    assert status_word(ws) == 0
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sp.sp_score_batch(desc, q, k, off, od, out, ws)
    assert score_path() == (1, ranges, launches)
    for _ in range(3):
        out.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert status_word(ws) == 0 and torch.equal(out, eager)
        sp.sp_score_batch(desc, q, k, off, od, eager, ws)
        torch.cuda.synchronize()


def test_captured_score_of_a_short_prompt():
    """A captured call takes the general path; every replay agrees with the eager call."""
    import torch
    import paper_2603_02631_amd as sp
    from gpu_util import score_path
    dev, L = "cuda:0", 8200
    say("[score-capture]")
    g = torch.Generator(device=dev).manual_seed(3)
    q = torch.randn((16, 32, 8, 64), device=dev, generator=g).to(torch.bfloat16)
    k = [torch.randn((8, L, 64), device=dev, generator=g).to(torch.bfloat16) for _ in range(16)]
    desc = sp.ScoreDesc(16, 32, 8, 64, 8, 0.125, sp.SP_LAYER_MEAN, 64, L * 64)
    ws = torch.empty(sp.sp_score_workspace(desc, L, 1), dtype=torch.uint8, device=dev)
    eager, out = torch.zeros(L, device=dev), torch.zeros(L, device=dev)
    sp.sp_score(desc, q, k, L, eager, ws)
    assert score_path()[1] > 1
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sp.sp_score(desc, q, k, L, out, ws)
    assert score_path() == "general"
    for _ in range(3):
        out.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        torch.testing.assert_close(out, eager, rtol=1e-4, atol=0.0)     # fp32 exponentials of two summation orders
        sp.sp_score(desc, q, k, L, eager, ws)
        torch.cuda.synchronize()
