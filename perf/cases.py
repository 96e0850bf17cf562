"""Performance cases of the token-importance path: what a serving program has this library do.

A case is one request, or one batch of requests, taken through the public entry points the way a program that
compresses prompts calls them: score the prompt's keys, select chunks, project the kept spans onto the target
tokenisation. `op` names the call sequence:

  prompt   sp_score        + sp_select + sp_project      one prompt, contiguous bf16 keys
  look     sp_score_look   + sp_select + sp_project      ... with the lookahead tokens' own keys in the softmax
  paged    sp_score_paged  + sp_select + sp_project      ... keys behind a block table
  fp8      sp_score_fp8    + sp_select + sp_project      ... 8-bit keys
  batch    sp_score_batch  + sp_select_batch + sp_project_batch     ragged batch
  budget   sp_select_budget + sp_project + sp_assemble   a scored prompt cut to a fixed number of target tokens

Inputs are made on the GPU from the seed: N(0, 1) queries and keys rounded to bf16, a small share of keys planted as
heavy hitters (three times a query vector, what attention sinks and retrieved passages look like to this path), and
two tokenisations of one text with geometric token lengths.
"""
from __future__ import annotations

import math
import random

import torch

import paper_2603_02631_amd as sp

DEV = "cuda:0"
POOL = 13                       # average-pool width used throughout
DRAFT_CHARS, TARGET_CHARS = 4.0, 3.5    # mean characters of a draft / target token

# Draft models: layers, query heads, kv heads, head_dim.
DRAFTS = {
    "tiny": (2, 4, 2, 64),
    "llama1b": (16, 32, 8, 64),         # 16-layer, head_dim 64 draft
    "qwen06b": (28, 16, 8, 128),        # 28-layer, head_dim 128 draft
    "group8": (24, 32, 4, 128),         # eight query heads to a kv head
}
MAX_K_BYTES = 4.4e9                     # drawn cases stay below the largest listed one


def listed():
    base = dict(draft="llama1b", n_q=8, layout="HND", agg="mean", chunk=32, keep=20)

    def case(name, op, **kw):
        return {"name": name, "op": op, **base, **kw}

    return [
        # the smallest call: a toy draft and a thousand tokens; launches and host work are all there is
        case("prompt-1k", "prompt", draft="tiny", L=1024, keep=25),
        # a typical short document (average inputs of the short suite are 8-9 thousand tokens)
        case("prompt-8k", "prompt", L=8192),
        # the head_dim 128 draft on a mid-size document
        case("prompt-32k-d128", "prompt", draft="qwen06b", L=32768, keep=15),
        # the long-context setting: 128K tokens, 16 lookahead rows
        case("prompt-128k", "prompt", n_q=16, L=131072, chunk=64, keep=10),
        # the longest prompts of the suites, a quarter of a million tokens
        case("prompt-256k", "prompt", L=262144, chunk=128, keep=10),
        # continuous batching: sixteen prompts of very different length
        case("batch-16", "batch", B=16, lo=2048, hi=65536, lens_seed=25),
        # many short requests at once, some of them tiny, head_dim 128
        case("batch-short-24", "batch", draft="qwen06b", B=24, lo=60, hi=4000, lens_seed=11),
        # a paged key cache of 4k-token blocks, ragged tail
        case("paged-50k", "paged", L=50021, page=4096, keep=15),
        # 8-bit key cache at the long-context length
        case("fp8-128k", "fp8", n_q=16, L=131072, chunk=64, keep=10),
        # lookahead keys in the normaliser, token-major keys, maximum over layers, odd length, code-debug chunk size
        case("look-12k-nhd", "look", L=12007, layout="NHD", agg="max", chunk=128, look_self=1),
        # a draft with wide query groups (64 padded rows at head_dim 128), odd length
        case("prompt-20k-g8", "prompt", draft="group8", L=20001),
        # a scored 128K prompt cut to a fixed length of 16K target tokens and assembled with delimiters
        case("budget-128k", "budget", L=131072, chunk=64, budget=16384, delim=3),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["prompt", "prompt", "prompt", "batch", "batch", "paged", "fp8", "look", "budget"])
    case = {"op": op, "draft": rng.choice(["llama1b", "llama1b", "qwen06b"]), "n_q": rng.choice([8, 8, 8, 5, 12, 16]),
            "layout": rng.choice(["HND", "HND", "NHD"]), "agg": rng.choice(["mean", "mean", "max"]),
            "chunk": rng.choice([32, 32, 64, 128]), "keep": rng.choice([10, 15, 20, 25, 45])}
    if op == "prompt" and rng.random() < 0.15:
        case["draft"] = "group8"
    if case["draft"] != "llama1b":
        case["n_q"] = min(case["n_q"], 8)       # wider lookahead is used with the head_dim 64 draft
    layers, _, kv, d = DRAFTS[case["draft"]]
    top = int(min(262144, MAX_K_BYTES / (2 * layers * kv * d)))
    if op == "batch":
        short = rng.random() < 0.4
        case["B"] = rng.randint(4, 32) if short else rng.randint(2, 16)
        case["lo"], case["hi"] = (60, 4000) if short else (2048, 32768)
        case["lens_seed"] = rng.randrange(1000)
        while sum(lengths(case)) > top:
            case["B"] -= 1
    else:
        case["L"] = _log_uniform(rng, 1000, top)
    if op == "paged":
        case["page"] = rng.choice([512, 1024, 4096])
    if op == "look":
        case["look_self"] = rng.randint(0, 1)
    if op == "budget":
        case["chunk"] = max(case["chunk"], 32)
        case["budget"] = max(64, int(case["L"] * case["keep"] / 100))
        case["delim"] = rng.randint(0, 5)
    return case


def lengths(case):
    """Prompt lengths of a batch, log-uniform in [lo, hi]."""
    rng = random.Random(case["lens_seed"])
    return [_log_uniform(rng, case["lo"], case["hi"]) for _ in range(case["B"])]


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def target_tokens(L):
    return int(L * DRAFT_CHARS / TARGET_CHARS)


def _offsets(g, L):
    """Character offsets of a draft tokenisation of L tokens and of an independent target one of the same text: draft
    lengths are geometric, target boundaries fall on characters drawn without replacement."""
    lens = torch.empty(L, device=DEV).geometric_(1.0 / DRAFT_CHARS, generator=g).to(torch.int64)
    draft = torch.cat([torch.zeros(1, dtype=torch.int64, device=DEV), torch.cumsum(lens, 0)])
    total, M = int(draft[-1].item()), target_tokens(L)
    inner = torch.sort(torch.randperm(total - 1, device=DEV, generator=g)[:M - 1] + 1).values
    ends = torch.tensor([0, total], dtype=torch.int64, device=DEV)
    return draft, torch.cat([ends[:1], inner, ends[1:]])


def _heavy_positions(g, L):
    """One percent of the positions; on long prompts a tenth of that, within eight bands of 512 tokens."""
    if L >= 65536:
        starts = torch.randint(0, L - 512, (8, 1), device=DEV, generator=g)
        pool = (starts + torch.arange(512, device=DEV)[None, :]).reshape(-1)
        return torch.unique(pool[torch.randperm(pool.numel(), device=DEV, generator=g)[:L // 1000]])
    return torch.randperm(L, device=DEV, generator=g)[:max(1, L // 100)]


def _keys(g, q, lens, kv, layer, heavy):
    """bf16 keys [kv][T][d] of one layer; q: [B][layers][H][n_q][d]."""
    H, n_q, d = q.shape[2:]
    k = torch.randn((kv, sum(lens), d), device=DEV, generator=g).to(torch.bfloat16)
    at = 0
    for b, L in enumerate(lens):
        pos = heavy[b]
        head = torch.randint(0, H // kv, (kv, pos.numel()), device=DEV, generator=g)
        row = torch.randint(0, n_q, (kv, pos.numel()), device=DEV, generator=g)
        first = (torch.arange(kv, device=DEV) * (H // kv))[:, None]
        k[:, at + pos] = (3.0 * q[b, layer, first + head, row].float()).to(torch.bfloat16)
        at += L
    return k


def _zeros(n, dtype):
    return torch.zeros(n, dtype=dtype, device=DEV)


def prepare(case, seed):
    g = _gen(seed)
    op, chunk = case["op"], case["chunk"]
    layers, H, kv, d = DRAFTS[case["draft"]]
    n_q, nhd = case["n_q"], case["layout"] == "NHD"
    lens = lengths(case) if op == "batch" else [case["L"]]
    B, T = len(lens), sum(lens)
    s = {"op": op, "case": case, "lens": lens, "T": T}
    texts = [_offsets(g, L) for L in lens]
    chunks = [-(-L // chunk) for L in lens]
    kept = [sp.sp_keep_count(C, case["keep"], 100) for C in chunks]
    if op == "budget":
        # scores as the score call leaves them: positive, heavy-tailed, a few bands far above the rest
        scores = torch.rand(T, device=DEV, generator=g).mul_(4.0).exp_().div_(float(T))
        scores[_heavy_positions(g, T)] *= 50.0
        s["scores"] = scores
        (s["doff"], s["toff"]), C = texts[0], chunks[0]
        M = s["M"] = s["toff"].numel() - 1
        cap = s["cap"] = case["budget"] + C * max(1, case["delim"])
        s["ids"] = torch.randint(0, 120000, (M,), device=DEV, generator=g, dtype=torch.int32)
        s["delim"] = torch.randint(0, 120000, (max(1, case["delim"]),), device=DEV, generator=g, dtype=torch.int32)
        s.update(sel=_zeros(C, torch.int32), spans=_zeros((C, 2), torch.int64), n_spans=_zeros(1, torch.int32),
                 k=_zeros(1, torch.int64), n_kept=_zeros(1, torch.int64), cs=_zeros(C, torch.float32),
                 tspans=_zeros((C, 2), torch.int64), n_t=_zeros(1, torch.int32), mask=_zeros(M, torch.uint8),
                 n_proj=_zeros(1, torch.int64), out_ids=_zeros(cap, torch.int32), out_pos=_zeros(cap, torch.int32),
                 out_src=_zeros(cap, torch.int64), out_len=_zeros(1, torch.int64), max_spans=C,
                 ws=_zeros(sp.sp_select_budget_workspace(T, chunk), torch.uint8),
                 ws2=_zeros(sp.sp_assemble_workspace(C), torch.uint8))
        return s
    q = torch.randn((B, layers, H, n_q, d), device=DEV, generator=g).to(torch.bfloat16)
    heavy = [_heavy_positions(g, L) for L in lens]
    stride_t, stride_h = (kv * d, d) if nhd else (d, T * d)
    if op == "paged":
        P = case["page"]
        pages = -(-T // P)
        table = torch.randperm(pages, device=DEV, generator=g)
        s["table"] = table.to(torch.int32)
        stride_t, stride_h = (kv * d, d) if nhd else (d, P * d)
    s["k"], scales = [], []
    for layer in range(layers):
        k = _keys(g, q, lens, kv, layer, heavy)
        if op == "fp8":
            scale = (k.float().abs().amax(dim=(1, 2)) / 448.0).clamp_min(1e-30)
            scales.append(scale)
            k = (k.float() / scale[:, None, None]).to(torch.float8_e4m3fn).view(torch.uint8)
        if op == "paged":
            padded = torch.zeros((kv, pages * P, d), dtype=torch.bfloat16, device=DEV)
            padded[:, :T] = k
            pool = torch.empty((pages, kv, P, d), dtype=torch.bfloat16, device=DEV)
            pool[table] = padded.view(kv, pages, P, d).transpose(0, 1)
            k = pool.transpose(1, 2).contiguous() if nhd else pool
        elif nhd:
            k = k.transpose(0, 1).contiguous()
        s["k"].append(k)
    s["q"] = q if op == "batch" else q[0]
    s["desc"] = sp.ScoreDesc(layers, H, kv, d, n_q, 1.0 / math.sqrt(d),
                             sp.SP_LAYER_MAX if case["agg"] == "max" else sp.SP_LAYER_MEAN, stride_t, stride_h)
    if op == "fp8":
        s["kscale"] = torch.stack(scales).contiguous()
    if op == "look":
        noise = torch.randn((layers, kv, n_q, d), device=DEV, generator=g)
        s["k_look"] = (noise + q[0][:, ::H // kv].float()).to(torch.bfloat16).contiguous()
    s["scores"] = _zeros(T, torch.float32)
    s["ws"] = torch.empty(sp.sp_score_workspace(s["desc"], T, B), dtype=torch.uint8, device=DEV)
    if op == "batch":
        def prefix(values):
            out = [0]
            for v in values:
                out.append(out[-1] + v)
            return out, torch.tensor(out, dtype=torch.int64, device=DEV)
        s["off"], s["off_dev"] = prefix(lens)
        s["koff"], s["koff_dev"] = prefix(kept)
        s["moff"], s["moff_dev"] = prefix([t.numel() - 1 for _, t in texts])
        s["doff"], s["toff"] = torch.cat([t for t, _ in texts]), torch.cat([t for _, t in texts])
        K, M, n_cs = s["koff"][-1], s["moff"][-1], T // chunk + B + 1
        s["ws2"] = torch.empty(sp.sp_select_batch_workspace(T, B, chunk), dtype=torch.uint8, device=DEV)
    else:
        (s["doff"], s["toff"]), K, n_cs = texts[0], kept[0], chunks[0]
        M = s["toff"].numel() - 1
        s["ws2"] = torch.empty(sp.sp_select_workspace(T, chunk), dtype=torch.uint8, device=DEV)
    s.update(K=K, M=M, sel=_zeros(K, torch.int32), spans=_zeros((K, 2), torch.int64), n_spans=_zeros(B, torch.int32),
             cs=_zeros(n_cs, torch.float32), tspans=_zeros((K, 2), torch.int64), n_t=_zeros(B, torch.int32),
             mask=_zeros(M, torch.uint8), n_kept=_zeros(B, torch.int64))
    return s


def run(s):
    op, case, T = s["op"], s["case"], s["T"]
    chunk = case["chunk"]
    if op == "budget":
        sp.sp_select_budget(s["scores"], T, POOL, chunk, s["doff"], s["toff"], s["M"], case["budget"], s["sel"],
                            s["spans"], s["n_spans"], s["k"], s["n_kept"], s["cs"], s["ws"])
        sp.sp_project(s["doff"], T, s["toff"], s["M"], s["spans"], s["n_spans"], s["max_spans"], s["tspans"], s["n_t"],
                      s["mask"], s["n_proj"])
        sp.sp_assemble(s["ids"], s["M"], s["tspans"], s["n_t"], s["max_spans"], s["delim"], case["delim"], s["cap"],
                       s["out_ids"], s["out_pos"], s["out_src"], s["out_len"], s["ws2"])
        # target ranges come back as what they select: the mask and the assembled prompt
        return {n: s[n] for n in ("sel", "spans", "n_spans", "k", "n_kept", "cs", "n_t", "mask", "n_proj", "out_ids",
                                  "out_pos", "out_src", "out_len")}
    desc, q, k, scores, ws = s["desc"], s["q"], s["k"], s["scores"], s["ws"]
    if op == "batch":
        sp.sp_score_batch(desc, q, k, s["off"], s["off_dev"], scores, ws)
        sp.sp_select_batch(scores, s["off"], s["off_dev"], POOL, chunk, s["koff"], s["koff_dev"], s["sel"], s["spans"],
                           s["n_spans"], s["cs"], s["ws2"])
        sp.sp_project_batch(s["doff"], s["off"], s["off_dev"], s["toff"], s["moff"], s["moff_dev"], s["spans"],
                            s["n_spans"], s["koff"], s["koff_dev"], s["tspans"], s["n_t"], s["mask"], s["n_kept"])
    else:
        if op == "prompt":
            sp.sp_score(desc, q, k, T, scores, ws)
        elif op == "look":
            sp.sp_score_look(desc, q, k, T, s["k_look"], case["look_self"], scores, ws)
        elif op == "paged":
            kv, d = desc.n_kv_heads, desc.head_dim
            sp.sp_score_paged(desc, q, k, s["table"], case["page"], kv * case["page"] * d, T, scores, ws)
        else:
            sp.sp_score_fp8(desc, q, k, s["kscale"], T, scores, ws)
        sp.sp_select(scores, T, POOL, chunk, s["K"], s["sel"], s["spans"], s["n_spans"], s["cs"], s["ws2"])
        sp.sp_project(s["doff"], T, s["toff"], s["M"], s["spans"], s["n_spans"], s["K"], s["tspans"], s["n_t"],
                      s["mask"], s["n_kept"])
    # the lists of chunks and spans come back as the mask of kept target tokens: a chunk that trades places with a
    # near-tie moves every later entry of a list, but only its own tokens of the mask
    return {"scores": scores, "chunk_scores": s["cs"], "mask": s["mask"]}


def _layer_keys(s, layer):
    """Keys of one layer in 64 bits, [kv][T][d], whatever the layout they are held in."""
    case, T = s["case"], s["T"]
    k = s["k"][layer]
    if case["op"] == "paged":
        k = k.transpose(1, 2) if case["layout"] == "NHD" else k             # [pages][kv][P][d]
        k = k[s["table"].long()].transpose(0, 1)
        return k.reshape(k.shape[0], -1, k.shape[-1])[:, :T].double()
    if case["op"] == "fp8":
        k = k.view(torch.float8_e4m3fn).float().double()
        scale = s["kscale"][layer].double()
        return (k.transpose(0, 1) if case["layout"] == "NHD" else k) * scale[:, None, None]
    return (k.transpose(0, 1) if case["layout"] == "NHD" else k).double()


def _exact_scores(s):
    case, lens = s["case"], s["lens"]
    layers, H, kv, d = DRAFTS[case["draft"]]
    n_q, G, take_max = case["n_q"], H // kv, case["agg"] == "max"
    q = s["q"] if case["op"] == "batch" else s["q"][None]
    out = [None] * len(lens)
    for layer in range(layers):
        keys, at = _layer_keys(s, layer), 0
        for b, L in enumerate(lens):
            if L == 0:
                continue
            rows = q[b, layer].double().reshape(kv, G * n_q, d)
            logits = torch.matmul(rows, keys[:, at:at + L].transpose(1, 2).contiguous()).mul_(s["desc"].scale)
            norm = torch.logsumexp(logits, dim=2)
            if case["op"] == "look":
                look = torch.matmul(rows, s["k_look"][layer].double().transpose(1, 2).contiguous()).mul_(s["desc"].scale)
                n = torch.arange(n_q, device=DEV)
                hidden = n[None, :] >= n[:, None] + case["look_self"]       # row n sees the keys generated before it
                look = look.view(kv, G, n_q, n_q).masked_fill(hidden, -math.inf).view(kv, G * n_q, n_q)
                norm = torch.logaddexp(norm, torch.logsumexp(look, dim=2))
            prob = logits.sub_(norm[:, :, None]).exp_().view(kv * G, n_q, L).amax(dim=0)
            if out[b] is None:
                out[b] = prob
            elif take_max:
                out[b] = torch.maximum(out[b], prob)
            else:
                out[b] += prob
            at += L
    div = n_q * (1 if take_max else layers)
    return [o.sum(dim=0) / div for o in out]


def _exact_chunk_scores(scores, chunk):
    L = scores.numel()
    pooled = torch.nn.functional.avg_pool1d(scores[None, None], POOL, stride=1, padding=POOL // 2)[0, 0]
    C = -(-L // chunk)
    sums = torch.nn.functional.pad(pooled, (0, C * chunk - L)).view(C, chunk).sum(dim=1)
    size = torch.full((C,), float(chunk), dtype=torch.float64, device=DEV)
    size[-1] = L - (C - 1) * chunk
    return sums / size


def exact(case, seed):
    """Scores and chunk scores in 64 bits, straight from the definition. What follows from them by comparing (kept
    chunks, spans, mask, assembled prompt) has no nearer value."""
    s = prepare(case, seed)
    chunk = case["chunk"]
    if case["op"] == "budget":
        out = {n: None for n in ("sel", "spans", "n_spans", "k", "n_kept", "cs", "n_t", "mask", "n_proj", "out_ids",
                                 "out_pos", "out_src", "out_len")}
        out["cs"] = _exact_chunk_scores(s["scores"].double(), chunk)
        return out
    parts = _exact_scores(s)
    cs, at = torch.zeros_like(s["cs"], dtype=torch.float64), 0
    for b, part in enumerate(parts):
        v = _exact_chunk_scores(part, chunk)
        first = at // chunk + b if case["op"] == "batch" else 0
        cs[first:first + v.numel()] = v
        at += part.numel()
    return {"scores": torch.cat(parts), "chunk_scores": cs, "mask": None}


def work(case):
    """Keys, queries and offsets read once, scores, chunk scores and mask written once; one product of every query row
    with every key."""
    layers, H, kv, d = DRAFTS[case["draft"]]
    lens = lengths(case) if case["op"] == "batch" else [case["L"]]
    T = sum(lens)
    M = sum(target_tokens(L) for L in lens)
    small = 4.0 * T + 4.0 * T / case["chunk"] + 8.0 * T + 8.0 * M + M       # scores, chunk scores, offsets, mask
    if case["op"] == "budget":
        return {"bytes": small + 4.0 * M + 16.0 * case["budget"], "flops": float(POOL * T)}
    elem = 1 if case["op"] == "fp8" else 2
    return {"bytes": float(layers * kv * d * elem) * T + 2.0 * len(lens) * layers * H * case["n_q"] * d + small,
            "flops": 2.0 * layers * H * case["n_q"] * d * T}


def tolerance(case):
    # About four times what the path differs from the same computation in 64 bits on the listed cases (scores: 2-norm
    # 7.7e-7, largest 5.2e-6; chunk scores of given scores: 5.2e-8 and 2.0e-7). The mask may trade a near-tie of chunks.
    if case["op"] == "budget":
        return {"rel": 4e-7, "max": 1e-6, "differ": 0.0}
    return {"rel": 4e-6, "max": 2e-5, "differ": 0.01}
