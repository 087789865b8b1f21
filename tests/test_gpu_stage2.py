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
