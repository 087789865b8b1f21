"""The decision step and the batch list at the sizes where their work is shared by several waves and passes: working sets
longer than a workgroup, planning that finds no candidate and hands over to AR, equal and NaN confidences under the progress
rule, more than 64 groups."""
import numpy as np
import pytest
import torch

from oracle import pvf_oracle as O
from paper_2601_12247_amd import binding as B
from synth import inputs as S
from tests.gpu_util import assert_state_equals, make_context, oracle_decode_cfg, to_device

pytestmark = pytest.mark.gpu

V, MASK = 512, 511


def dev(a, dtype=torch.int32):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dtype)


def fresh_state(G, cfg):
    st = B.State(G, cfg)
    st.canvas.fill_(MASK)
    return st


@pytest.mark.parametrize("bl,gen,n_sparse,K", [(256, 256, 0, 4), (256, 512, 0, 8), (160, 640, 160, 3), (200, 800, 200, 4)])
def test_planning_without_candidates_hands_over_to_ar(bl, gen, n_sparse, K):
    """Both routes on; the planning vocabulary holds ids that are never a prediction, so every proposal is AR's: its candidates
    are counted after planning's were found to be none.  Working sets of up to 400 positions, 24 groups, two rounds (the second
    verifies the AR drafts).  Decisions bit for bit, but for groups whose oracle margin is below 1e-5 (confidences of 2e-6)."""
    G = 24
    cfg = B.DecodeCfg(block_len=bl, prompt_len=0, gen_len=gen, K=K, tau_high=0.9, tau_ar_lo=0.05, logit_scale=1.0, n_sparse=n_sparse)
    ocfg = oracle_decode_cfg(cfg)
    plan = np.array([V - 2], dtype=np.int32)
    bitmap = dev(S.plan_bitmap(plan, V).view(np.int32))
    st = fresh_state(G, cfg)
    ost = [O.initial_state(np.zeros(0, np.int32), ocfg, MASK) for _ in range(G)]
    R, checked, ar = cfg.R, 0, 0
    live = [True] * G
    for rnd in range(2):
        lg = np.repeat(S.make_boosted_logits(40 + rnd + bl, G * R, V, 10.0, MASK).reshape(G, 1, R, V), 1 + K, axis=1)
        lg[..., V - 2] = -9.0
        B.epilogue(dev(lg, torch.float32), st, bitmap, V, MASK)
        for g in range(G):
            if not live[g] or ost[g].done:
                continue
            n = ost[g].drafts.n
            ok = O.window_positions(ocfg, ost[g].k_active) < ocfg.T
            conf, tok = np.zeros((1 + n, R), np.float32), np.full((1 + n, R), -1, np.int32)
            for j in range(1 + n):
                conf[j, ok], tok[j, ok] = O.stage1(lg[g, j][ok], 1.0, MASK)
            new, info = O.decide(ost[g], conf, tok, ocfg, MASK, plan)
            live[g] = info.margin >= 1e-5
            if live[g]:
                assert_state_equals(st, g, new, info, cfg, where=f"round {rnd} group {g}")
                checked += 1
                ar += new.drafts.route == 2
            ost[g] = new
    assert checked >= 1.5 * G and ar >= G


@pytest.mark.parametrize("bl", [64, 256, 400])
def test_progress_rule_of_equal_and_nan_confidences(bl):
    """No confidence reaches the threshold: the most confident mask is committed, the first of equals, a NaN only where the first
    mask has it (nothing compares above it, and it compares above nothing).  Masks of one lane, of neighbouring lanes, of the last pass."""
    hi, nan = 4.0, float("nan")
    cases = [({}, []), ({5: hi, 37: hi, bl - 1: hi}, []), ({bl - 2: hi, bl // 2: hi}, []), ({0: nan, bl // 3: hi}, []),
             ({3: nan, bl // 3: hi, bl // 3 + 20: hi}, []), ({i: nan for i in range(bl)}, []), ({10: nan, 20: hi}, range(10)),
             ({bl - 2: hi, bl - 1: hi}, range(bl - 2)), ({bl // 2 + 1: nan, bl - 1: hi}, range(bl // 2)), ({bl - 1: nan}, range(bl - 1))]
    G = len(cases)
    cfg = B.DecodeCfg(block_len=bl, prompt_len=0, gen_len=bl, K=0, tau_high=0.9)
    ocfg = oracle_decode_cfg(cfg)
    logits = np.zeros((G, 1, bl, V), np.float32)
    canvas = np.full((G, bl), MASK, np.int32)
    for g, (level, known) in enumerate(cases):
        logits[g, 0, np.arange(bl), np.arange(bl) % 400 + g] = 3.0
        for i, x in level.items():
            logits[g, 0, i, i % 400 + g] = x
        canvas[g, list(known)] = 7
    st = fresh_state(G, cfg)
    st.canvas.copy_(dev(canvas)[:, None])
    B.epilogue(dev(logits, torch.float32), st, dev(np.zeros((V + 31) // 32)), V, MASK)
    conf, tok = st.conf.cpu().numpy(), st.tok.cpu().numpy()
    for g, (level, _) in enumerate(cases):
        old = O.State(canvas[g], O.Drafts(0, []), 0, False)
        assert np.array_equal(np.isnan(conf[g, 0]), [np.isnan(level.get(i, 0.0)) for i in range(bl)])
        new, info = O.decide(old, conf[g], tok[g], ocfg, MASK, [])
        assert info.n_base == 1
        assert_state_equals(st, g, new, info, cfg, where=f"group {g}")


TINY = S.ModelShape(n_layers=1, d_model=64, n_heads=2, d_ff=96, vocab=V, mask_id=MASK, logit_scale=20.0)


@pytest.mark.parametrize("G,first_live", [(63, 0), (65, 64), (70, 0), (130, 66), (130, 128)])
def test_batches_of_more_than_64_groups(G, first_live):
    """The list of live canvases is made 64 groups at a time: groups before first_live and every fifth one are done, the others have
    no, one or two drafts.  Every live slot's summary is that of its canvas, with a compact list, a padded one and one for the
    first half of the live canvases only, which leaves the others' summaries alone; finished groups stay as they are."""
    K = 2
    cfg = B.DecodeCfg(block_len=8, prompt_len=3, gen_len=16, K=K, tau_high=0.9, logit_scale=TINY.logit_scale)
    ctx = make_context(TINY, to_device(S.make_weights(TINY, seed=2)), max_seqs=G * (1 + K), max_T=cfg.T, max_rows=cfg.R)
    rng = np.random.default_rng(G + first_live)
    done = (np.arange(G) < first_live) | (np.arange(G) % 5 == 4) & (np.arange(G) != first_live)
    n_drafts = np.where(done, 0, rng.integers(0, K + 1, size=G))
    canvas = rng.integers(0, MASK, size=(G, 1 + K, cfg.T))
    canvas[:, :, 5:] = MASK                            # two known positions of the first block
    canvas[:, 1:, 5] = 9
    rows = torch.arange(cfg.prompt_len, cfg.T, dtype=torch.int32, device="cuda")[None].repeat(G * (1 + K), 1).contiguous()
    logits = ctx.forward(dev(canvas.reshape(-1, cfg.T)), rows)
    want_conf, want_tok = B.stage1(logits.view(-1, V), MASK, TINY.logit_scale)
    want_conf, want_tok = want_conf.view(G, 1 + K, cfg.R), want_tok.view(G, 1 + K, cfg.R)
    live = [(g, j) for g in range(G) if not done[g] for j in range(1 + n_drafts[g])]
    bitmap = dev(np.zeros((V + 31) // 32))
    for n_seq in (len(live), 0, len(live) // 2):
        st = fresh_state(G, cfg)
        st.canvas.copy_(dev(canvas)); st.done.copy_(dev(done)); st.n_drafts.copy_(dev(n_drafts))
        st.draft_route.fill_(B.PVF_ROUTE_PLAN); st.fill_pos.fill_(5); st.fill_tok.fill_(9); st.n_ws_blocks.fill_(1)
        st.conf.fill_(-1.0); st.tok.fill_(-2)
        ctx.round(st, bitmap, n_seq)
        torch.cuda.synchronize()
        seen = live[:n_seq] if n_seq else live
        at = tuple(np.array(seen).T)
        conf, tok = st.conf.cpu().numpy(), st.tok.cpu().numpy()
        assert np.array_equal(conf[at], want_conf.cpu().numpy()[at]) and np.array_equal(tok[at], want_tok.cpu().numpy()[at]), n_seq
        if n_seq:
            rest = np.ones((G, 1 + K), bool)
            rest[at] = False
            assert (conf[rest] == -1.0).all(), n_seq
        assert np.array_equal(st.canvas.cpu().numpy()[done], canvas[done]) and bool(st.done[torch.from_numpy(done).cuda()].all())
