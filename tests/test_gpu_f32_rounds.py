"""float32 rounds with the norms inside the projections and with rounds enqueued one ahead."""
import numpy as np
import pytest
import torch

from paper_2601_12247_amd import binding as B
from paper_2601_12247_amd import workloads as W

pytestmark = pytest.mark.gpu
DIMS = dict(n_layers=2, d_model=128, n_heads=4, d_ff=344, vocab=1000, mask_id=999, rms_eps=1e-5, rope_theta=1e4)
FIELDS = ("canvas", "n_drafts", "draft_route", "fill_pos", "fill_tok", "k_active", "n_ws_blocks", "conf", "tok", "accept",
          "winner", "n_commit", "done")


def model(offset=0):
    """Weights with gains around 1; offset: every norm gain and wide matrix that many floats behind an aligned address."""
    w = W.random_model(DIMS, seed=5, dtype=torch.float32, std=0.08)
    g = torch.Generator(device="cuda").manual_seed(3)

    def moved(t):
        out = torch.empty(t.numel() + offset, device="cuda")[offset:].view(t.shape)
        return out.copy_(t)

    for lw in w["layers"]:
        for n in ("attn_norm", "ffn_norm"):
            lw[n] = 1 + 0.1 * torch.randn(DIMS["d_model"], device="cuda", generator=g)
    w["final_norm"] = 1 + 0.1 * torch.randn(DIMS["d_model"], device="cuda", generator=g)
    for lw in w["layers"]:
        lw.update({n: moved(t) for n, t in lw.items()})
    w["final_norm"], w["out_head"] = moved(w["final_norm"]), moved(w["out_head"])
    return w


# canvases in launches of up to 1280 rows (norms inside, 16-row tiles) against the same ones among more (a norm pass, 32-row
# tiles); rows of fewer and of more tiles in the last layer; whole canvases wanted (no cut)
@pytest.mark.parametrize("T,R,few,many", [(100, 37, 1, 13), (17, 16, 3, 90), (229, 64, 5, 6), (64, 64, 2, 40), (33, 1, 1, 39)])
def test_rows_do_not_depend_on_the_batch(T, R, few, many):
    ctx = W.make_context(DIMS, model(), max_seqs=many, max_T=T, max_rows=R)
    tokens = W.random_prompts(many, T, DIMS["vocab"], DIMS["mask_id"], seed=T)
    rows = torch.stack([torch.randperm(T, generator=torch.Generator().manual_seed(s))[:R] for s in range(many)]).int()
    rows[:, R // 2] = -1 if R > 1 else rows[:, 0]
    rows = rows.cuda()
    all_ = ctx.forward(tokens, rows)
    some = ctx.forward(tokens[:few].contiguous(), rows[:few].contiguous())
    assert torch.equal(some, all_[:few])
    assert R == 1 or not all_[:, R // 2].any()
    # weights that 16-byte loads cannot read take the unfused launches: the same sums and norms
    plain = W.make_context(DIMS, model(offset=1), max_seqs=many, max_T=T, max_rows=R).forward(tokens, rows)
    assert torch.equal(plain, all_)


@pytest.mark.parametrize("G,prompt,gen,block,K,routes", [(1, 20, 32, 16, 0, 3), (5, 33, 64, 16, 4, 3), (3, 0, 48, 16, 2, 1), (70, 5, 16, 16, 1, 3),
                                                        (4, 40, 48, 16, 8, 1)])      # room for many more drafts than there are
def test_decode_is_its_rounds(G, prompt, gen, block, K, routes):
    """pvf_decode leaves state, tokens and counts as the same rounds called one by one do, although a round more is enqueued."""
    cfg = B.DecodeCfg(block_len=block, prompt_len=prompt, gen_len=gen, K=K, tau_high=0.9, logit_scale=6.0, routes=routes)
    w = model()
    ctx = W.make_context(DIMS, w, max_seqs=G * (1 + K), max_T=cfg.T, max_rows=cfg.R)
    bitmap = W.random_plan_bitmap(64, DIMS["vocab"], DIMS["mask_id"], seed=1)
    p = W.random_prompts(G, prompt, DIMS["vocab"], DIMS["mask_id"], seed=2)
    a, b = B.State(G, cfg), B.State(G, cfg)
    ctx.state_init(b, p)
    n_seq, rounds, forwards, commits = G, 0, 0, 0
    while n_seq:
        forwards += n_seq
        st = torch.as_tensor(np.asarray(ctx.round_sync(b, bitmap, n_seq))).reshape(G, 5)
        rounds += 1
        commits += int(st[:, 2:].sum())
        n_seq = int(((1 - st[:, 0]) * (1 + st[:, 1])).sum())
    for _ in range(2):
        out, stats = ctx.decode(a, p, bitmap)
        assert (stats.rounds, stats.seq_forwards, stats.n_base + stats.n_plan + stats.n_ar) == (rounds, forwards, commits)
        assert commits == G * gen
        for f in FIELDS:
            assert torch.equal(getattr(a, f), getattr(b, f)), f
        assert torch.equal(out.view(G, -1), b.canvas[:, 0])
