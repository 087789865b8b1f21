"""The work a user of this library has it do, as a list of timed cases and a generator of more of them.

Four kinds of case, each through the calls of paper_2601_12247_amd.binding:

  forward   Context.forward: the batched pass over S whole canvases of T tokens (backbone plus drafts, or many
            independent canvases), logits of R window rows each.  8B shape, bf16.
  round     Context.round_sync, the body of a decode loop: forward, decisions, next batch, status read.  8B shape,
            bf16; with the block-level K/V cache (only the window rows run through the layers) or without.
  epilogue  epilogue: the decision step alone over logits that lie in memory, decoding or calibration routes.
  decode    Context.decode: a whole decode of the small float32 model, state initialisation to the last token.

Prompts have any length in use, so canvases whose length is no multiple of a tile stand beside the even ones.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2601_12247_amd import binding as B
from paper_2601_12247_amd import workloads as W

# 2-layer float32 model of the small parity configuration
TINY = dict(n_layers=2, d_model=256, n_heads=4, d_ff=704, vocab=4096, mask_id=4095, rms_eps=1e-5, rope_theta=10000.0)
BIG = W.LLADA_8B
PRIOR = 5.0          # mean weight of the 512 raised tokens along the [MASK] embedding, in units of its root mean square
INT_FIELDS = ("canvas", "tok", "n_drafts", "draft_route", "fill_pos", "fill_tok", "k_active", "n_ws_blocks", "winner",
              "n_commit", "done")


def listed():
    return [
        # the small parity configuration: one canvas decoded to the end; launches of a few microseconds each
        {"name": "decode_f32_1x128", "kind": "decode", "G": 1, "prompt": 64, "gen": 64, "block": 32, "K": 2},
        # the same model, a batch of prompts of an odd length with more drafts each
        {"name": "decode_f32_8x229", "kind": "decode", "G": 8, "prompt": 101, "gen": 128, "block": 32, "K": 4},
        # threshold decoding without drafts, and every cache refresh: a single canvas
        {"name": "forward_1x512", "kind": "forward", "S": 1, "T": 512, "R": 64},
        # batch 1 with four drafts: the round the benchmark is quoted on
        {"name": "forward_5x512", "kind": "forward", "S": 5, "T": 512, "R": 64},
        # long generation with eight drafts
        {"name": "forward_9x1280", "kind": "forward", "S": 9, "T": 1280, "R": 128},
        # throughput mode: 16 canvases with four drafts each
        {"name": "forward_80x1024", "kind": "forward", "S": 80, "T": 1024, "R": 64},
        # a prompt as users have them: 181 tokens, 256 to generate, two drafts
        {"name": "forward_3x437", "kind": "forward", "S": 3, "T": 437, "R": 64},
        # K/V-cached threshold decoding: 64 rows, the weights are read for one block
        {"name": "cached_round_k0", "kind": "round", "cache": True, "G": 1, "prompt": 256, "gen": 256, "block": 32, "K": 0},
        # K/V-cached round with four drafts
        {"name": "cached_round_k4", "kind": "round", "cache": True, "G": 1, "prompt": 256, "gen": 256, "block": 32, "K": 4},
        # the paper's setting (512 to generate, blocks of 64, three drafts, cache) behind a prompt of 203 tokens
        {"name": "cached_round_odd_prompt", "kind": "round", "cache": True, "G": 1, "prompt": 203, "gen": 512, "block": 64, "K": 3},
        # the decision step on 8 row sets of 256 masked positions with four drafts to verify: 2.6 GB of logits
        {"name": "epilogue_8x5x256", "kind": "epilogue", "dtype": "bf16", "G": 8, "K": 4, "block": 256, "gen": 256,
         "vocab": 126464, "calibrate": False},
        # one step of a calibration trajectory: 32 candidates measured, entropies of all their rows
        {"name": "calibrate_1x33x64", "kind": "epilogue", "dtype": "bf16", "G": 1, "K": 32, "block": 32, "gen": 256,
         "vocab": 126464, "calibrate": True},
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _even(rng, n, unit):
    """n as it is, or as often the next multiple of `unit`: prompts come padded and unpadded."""
    return n if rng.random() < 0.5 else (n + unit - 1) // unit * unit


def draw(rng):
    kind = rng.choice(["forward", "forward", "forward", "round", "round", "round", "epilogue", "epilogue", "decode"])
    if kind == "forward":
        while True:
            S, T = _log(rng, 1, 80), _even(rng, _log(rng, 80, 1536), 64)
            # a pass on the longest canvases of odd length stays below two seconds
            if S * T <= (81920 if T % 64 == 0 else 4096) and (T % 64 == 0 or S * T * T <= 2_500_000):
                return {"kind": kind, "S": S, "T": T, "R": min(T, rng.choice([32, 64, 128]))}
    if kind == "round":
        while True:
            block, K = rng.choice([16, 32, 64]), rng.choice([0, 2, 3, 4, 8])
            G = rng.choice([1, 1, 2, 4])
            c = {"kind": kind, "cache": rng.random() < 0.75, "G": G, "prompt": _even(rng, _log(rng, 24, 512), 64),
                 "gen": block * rng.randint(4, max(4, 768 // block)), "block": block, "K": K}
            T = c["prompt"] + c["gen"]
            if T <= 1152 and G * (1 + K) * (2 * block if c["cache"] else T) <= 4096 and \
                    (c["cache"] or T % 64 == 0 or G * (1 + K) * T * T <= 2_500_000):
                return c
    if kind == "epilogue":
        while True:
            cal = rng.random() < 0.3
            block = rng.choice([16, 32, 64, 128, 256])
            c = {"kind": kind, "dtype": rng.choice(["bf16", "bf16", "f32"]), "G": _log(rng, 1, 16),
                 "K": rng.choice([8, 16, 32]) if cal else rng.choice([0, 2, 3, 4, 8]), "block": block, "gen": block * rng.choice([1, 4, 8]),
                 "vocab": _even(rng, _log(rng, 4000, 150000), 64), "calibrate": cal}
            rows = c["G"] * (1 + c["K"]) * min(2 * block, c["gen"])
            if rows * c["vocab"] <= 10240 * 126464 and (1 + c["K"]) * min(2 * block, c["gen"]) <= 5120:
                return c
    block = rng.choice([16, 32])
    return {"kind": kind, "G": _log(rng, 1, 12), "prompt": _even(rng, _log(rng, 16, 160), 16), "gen": block * rng.randint(2, 5),
            "block": block, "K": rng.choice([0, 2, 3, 4])}


# ---- inputs ----------------------------------------------------------------------------------------------------
def _norm_gains(w, seed):
    """Gains as trained models have them: around 1, none of them exactly."""
    rows = [lw[n] for lw in w["layers"] for n in ("attn_norm", "ffn_norm")] + [w["final_norm"]]
    for i, t in enumerate(rows):
        B.fill_normal(t, seed * 1009 + i, 1.0, 0.1)


def _big_model(seed):
    """8B-shaped weights whose predictions are separated the way a trained model's are: a token predicts itself, and
    at a masked position some of the planning tokens come first (a prior over the vocabulary in the output head,
    along the [MASK] embedding).  Returns the weights and the planning bitmap."""
    dims = BIG
    w = W.consistent_model(dims, seed=seed, mix=0.25)
    _norm_gains(w, seed)
    rng = np.random.default_rng(seed + 77)
    ids = np.sort(rng.choice(dims["mask_id"], size=512, replace=False))
    e = w["embed"][dims["mask_id"]].float()
    prior = torch.from_numpy(rng.exponential(PRIOR / e.numel() ** 0.5, size=512).astype(np.float32)).cuda()
    at = torch.from_numpy(ids).cuda()
    w["out_head"][at] = (w["out_head"][at].float() + prior[:, None] * (e / e.norm())).to(torch.bfloat16)
    return w, _bitmap(ids, dims["vocab"])


def _bitmap(ids, vocab):
    words = np.zeros((vocab + 31) // 32, dtype=np.uint32)
    np.bitwise_or.at(words, ids >> 5, np.uint32(1) << (ids & 31).astype(np.uint32))
    return torch.from_numpy(words.view(np.int32)).cuda()


def _tiny_model(seed):
    w = W.random_model(TINY, seed=seed, dtype=torch.float32)
    _norm_gains(w, seed)
    return w


def _packed_state(G, cfg, vocab):
    """A State whose whole-number members are views of one buffer, so that a program can save and restore it whole."""
    st = B.State(G, cfg, vocab=vocab)
    n = sum(getattr(st, f).numel() for f in INT_FIELDS)
    flat = torch.zeros(n + (st.accept.numel() + 3) // 4, dtype=torch.int32, device="cuda")
    o = 0
    for f in INT_FIELDS:
        t = getattr(st, f)
        v = flat[o:o + t.numel()].view(t.shape)
        v.copy_(t)
        setattr(st, f, v)
        o += t.numel()
    st.accept = flat[o:].view(torch.uint8)[:st.accept.numel()].view(st.accept.shape)
    return st, flat


def _fill_canvases(st, cfg, vocab, mask_id, rng, k, n_drafts, route, plan_ids):
    """The middle of a decode: prompt and the blocks before block k known, half of block k known, the rest masked,
    and n_drafts drafts per group, each one planning token filled into a masked position of block k."""
    G, K, P, bl, T = st.G, cfg.K, cfg.prompt_len, cfg.block_len, cfg.T
    base = rng.integers(0, vocab - 1, size=(G, T))
    base = np.where(base >= mask_id, base + 1, base)
    w0 = P + k * bl
    base[:, w0 + bl:] = mask_id
    pos, tok = np.full((G, max(K, 1)), -1), np.full((G, max(K, 1)), -1)
    canvas = np.empty((G, 1 + K, T), dtype=np.int64)
    for g in range(G):
        order = rng.permutation(bl)
        n_masked = max(bl // 2, min(bl, n_drafts))
        base[g, w0 + order[:n_masked]] = mask_id
        canvas[g] = base[g]
        for j in range(n_drafts):
            pos[g, j], tok[g, j] = w0 + order[j % n_masked], rng.choice(plan_ids)
            canvas[g, 1 + j, pos[g, j]] = tok[g, j]
    for t, a in ((st.canvas, canvas), (st.fill_pos, pos), (st.fill_tok, tok)):
        t.copy_(torch.from_numpy(a.astype(np.int32)))
    st.n_drafts.fill_(n_drafts)
    st.draft_route.fill_(route if n_drafts else B.PVF_ROUTE_NONE)
    st.k_active.fill_(k)


def _prepare_forward(c, seed):
    w, _ = _big_model(seed)
    ctx = W.make_context(BIG, w, max_seqs=c["S"], max_T=c["T"], max_rows=c["R"])
    tokens = W.random_prompts(c["S"], c["T"], BIG["vocab"], BIG["mask_id"], seed=seed)
    tokens[:, c["T"] // 2:] = BIG["mask_id"]
    first = min(c["T"] // 2, c["T"] - c["R"])
    rows = torch.arange(first, first + c["R"], dtype=torch.int32, device="cuda")[None].repeat(c["S"], 1).contiguous()
    return {"c": c, "ctx": ctx, "tokens": tokens, "rows": rows}


def _prepare_round(c, seed):
    w, bitmap = _big_model(seed)
    cfg = B.DecodeCfg(block_len=c["block"], prompt_len=c["prompt"], gen_len=c["gen"], K=c["K"], tau_high=0.9, kv_cache=int(c["cache"]))
    ctx = W.make_context(BIG, w, max_seqs=c["G"] * (1 + c["K"]), max_T=cfg.T, max_rows=cfg.R)
    rng = np.random.default_rng(seed + 5)
    st, flat = _packed_state(c["G"], cfg, None)
    words = bitmap.cpu().numpy().view(np.uint32)
    plan_ids = np.flatnonzero((words[np.arange(BIG["vocab"]) >> 5] >> (np.arange(BIG["vocab"]) & 31).astype(np.uint32)) & 1)
    _fill_canvases(st, cfg, BIG["vocab"], BIG["mask_id"], rng, 1, c["K"], B.PVF_ROUTE_PLAN, plan_ids)
    saved = flat.clone()
    if c["cache"]:                       # the round in which the block was entered: it fills the K/V cache
        ctx.round_sync(st, bitmap)
        flat.copy_(saved)
    return {"c": c, "ctx": ctx, "st": st, "flat": flat, "saved": saved, "bitmap": bitmap, "n_seq": c["G"] * (1 + c["K"])}


def _prepare_epilogue(c, seed):
    V = c["vocab"]
    mask_id = V - 128
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    cal = c["calibrate"]
    cfg = B.DecodeCfg(block_len=c["block"], prompt_len=0, gen_len=c["gen"], K=c["K"], tau_high=0.9, logit_scale=1.5,
                      routes=B.PVF_ROUTES_CAL if cal else 3)
    rng = np.random.default_rng(seed + 9)
    st, flat = _packed_state(c["G"], cfg, V)
    n_rows = c["G"] * (1 + c["K"]) * cfg.R
    logits = torch.empty(n_rows, V, dtype=dt, device="cuda")
    B.fill_normal(logits, seed * 7 + 1, 0.0, 1.0)
    # rows of N(0,1) with one raised entry, from near-uniform to near-one-hot; a position keeps its token in every
    # canvas of a group but for one position in sixteen
    shape = (c["G"], 1 + c["K"], cfg.R)
    ids = np.broadcast_to(rng.integers(0, mask_id, size=(c["G"], 1, cfg.R)), shape).copy()
    other = rng.random(shape) < 1 / 16
    ids[other] = rng.integers(0, mask_id, size=int(other.sum()))
    boost = np.broadcast_to(rng.uniform(0.0, 12.0, size=(c["G"], 1, cfg.R)), shape)
    ar, at = torch.arange(n_rows, device="cuda"), torch.from_numpy(ids.reshape(-1)).cuda()
    up = torch.from_numpy(boost.reshape(-1).astype(np.float32)).cuda()
    logits[ar, at] = (logits[ar, at].float() + up).to(dt)
    plan_ids = np.sort(np.unique(np.concatenate([rng.choice(mask_id, size=512, replace=False), ids[:, 0, ::4].reshape(-1)])))
    _fill_canvases(st, cfg, V, mask_id, rng, 0, c["K"], B.PVF_ROUTE_CAL if cal else B.PVF_ROUTE_PLAN, plan_ids)
    return {"c": c, "st": st, "flat": flat, "saved": flat.clone(), "logits": logits.view(*shape, V), "vocab": V, "mask_id": mask_id,
            "bitmap": _bitmap(plan_ids, V)}


def _prepare_decode(c, seed):
    cfg = B.DecodeCfg(block_len=c["block"], prompt_len=c["prompt"], gen_len=c["gen"], K=c["K"], tau_high=0.9, logit_scale=20.0)
    ctx = W.make_context(TINY, _tiny_model(seed), max_seqs=c["G"] * (1 + c["K"]), max_T=cfg.T, max_rows=cfg.R)
    rng = np.random.default_rng(seed + 3)
    ids = np.sort(rng.choice(TINY["mask_id"], size=64, replace=False))
    return {"c": c, "ctx": ctx, "st": B.State(c["G"], cfg), "bitmap": _bitmap(ids, TINY["vocab"]),
            "prompt": W.random_prompts(c["G"], c["prompt"], TINY["vocab"], TINY["mask_id"], seed=seed)}


def prepare(case, seed):
    return {"forward": _prepare_forward, "round": _prepare_round, "epilogue": _prepare_epilogue,
            "decode": _prepare_decode}[case["kind"]](case, seed)


def run(state):
    kind = state["c"]["kind"]
    if kind == "forward":
        return state["ctx"].forward(state["tokens"], state["rows"])
    if kind == "decode":
        out, stats = state["ctx"].decode(state["st"], state["prompt"], state["bitmap"])
        return {"tokens": out, "rounds": stats.rounds}
    st = state["st"]
    state["flat"].copy_(state["saved"])  # the same step again
    if kind == "round":
        state["ctx"].round_sync(st, state["bitmap"], state["n_seq"])
        return {"state": state["flat"], "conf": st.conf}
    if not state["c"]["calibrate"]:
        B.epilogue(state["logits"], st, state["bitmap"], state["vocab"], state["mask_id"])
        return {"state": state["flat"], "conf": st.conf}
    for t in (st.cal_n, st.cal_m, st.cal_a, st.cal_vig):
        t.zero_()
    B.epilogue(state["logits"], st, state["bitmap"], state["vocab"], state["mask_id"])
    return {"state": state["flat"], "conf": st.conf, "ent": st.ent, "dh": st.dh, "cal": [st.cal_n, st.cal_m, st.cal_a, st.cal_vig]}


# ---- what a pass cannot do without ---------------------------------------------------------------------------------
def _layers(dims, rows, last_rows, key_rows, esize):
    """flops and weight bytes of the layers and the head: `rows` rows through every layer, of which only the last_rows
    that logits are wanted for go on after the attention of the last one; key_rows = sum over rows of the keys each sees."""
    d, ff, V, L = dims["d_model"], dims["d_ff"], dims["vocab"], dims["n_layers"]
    flops = 2.0 * rows * L * 2 * d * d + 2.0 * (rows * (L - 1) + last_rows) * (2 * d * d + 3 * d * ff)
    flops += 4.0 * d * key_rows * ((L - 1) + last_rows / rows) + 2.0 * last_rows * d * V
    return flops, esize * (L * (4.0 * d * d + 3 * d * ff) + V * d + min(rows, V) * d)


def work(case):
    c, kind = case, case["kind"]
    if kind == "forward":
        M = c["S"] * c["T"]
        flops, nb = _layers(BIG, M, c["S"] * c["R"], M * c["T"], 2)
        return {"flops": flops, "bytes": nb + 4.0 * (M + c["S"] * c["R"]) + 2.0 * c["S"] * c["R"] * BIG["vocab"]}
    if kind == "decode":
        # one round per committed token is the most, one per block the least; this model commits one to three a round
        T, n = c["prompt"] + c["gen"], c["G"] * (1 + c["K"])
        rounds, R = c["gen"] / 2.0, min(2 * c["block"], c["gen"])
        flops, nb = _layers(TINY, n * T, n * R, n * T * T, 4)
        return {"flops": flops * rounds, "bytes": nb * rounds}
    R, n = min(2 * c["block"], c["gen"]), c["G"] * (1 + c["K"])
    if kind == "round":
        T = c["prompt"] + c["gen"]
        rows = n * (R if c["cache"] else T)
        flops, nb = _layers(BIG, rows, n * R, rows * T, 2)
        kv = 4.0 * BIG["n_layers"] * BIG["d_model"] * c["G"] * (T - R) if c["cache"] else 0.0
        return {"flops": flops, "bytes": nb + kv + 8.0 * n * (T + 2 * R)}
    es = 2 if c["dtype"] == "bf16" else 4
    return {"flops": n * R * c["vocab"] * (8.0 if c["calibrate"] else 4.0), "bytes": n * R * (c["vocab"] * es + 12.0)}


def tolerance(case):
    """Measured between the matrix-core kernels and the plain ones (PVF_FORCE_SIMPLE=1), which round at the same tensors
    but add in another order.  bf16 through 32 layers: logits 2.5e-2 apart in the 2-norm (64 roundings of the residual
    stream alone give 1.9e-2 between two pipelines) and 0.17 at most; a round's probabilities 1.5e-2 and 0.05 apart, and
    up to 0.4 % of its whole values different, where a runner-up or a threshold is that close."""
    kind = case["kind"]
    if kind == "forward":
        return {"rel": 0.03, "max": 0.5}
    if kind == "round":
        return {"rel": 0.03, "max": 0.2, "differ": 0.01}
    if kind == "decode":                 # float32 with float64 sums: a confidence moves by 1e-6, tokens hardly ever
        return {"rel": 0.0, "differ": 0.01}
    return {"rel": 1e-5, "max": 1e-3, "differ": 0.001}      # float32 sums over a vocabulary
