"""Above 640 token rows in a launch a canvas's bf16 logits are the same bits whatever rides along: full-width rows, canvas
lengths on both sides of every choice that depends on the launch's rows (tile shapes, rotary embedding in the projection's
epilogue or in a pass of its own)."""
import numpy as np
import pytest
import torch

from paper_2601_12247_amd import binding as B
from synth import inputs as S
from tests.gpu_util import make_context

pytestmark = pytest.mark.gpu

SHAPE = S.ModelShape(n_layers=2, d_model=4096, n_heads=32, d_ff=1024, vocab=2048, mask_id=2047, rope_theta=5e5)
N_MAX = 9


@pytest.fixture(scope="module")
def weights():
    g = torch.Generator(device="cuda").manual_seed(1)

    def mat(r, c, std=0.02):
        return (torch.randn(r, c, device="cuda", generator=g) * std).to(torch.bfloat16)

    def gain():
        return (1 + 0.1 * torch.randn(SHAPE.d_model, device="cuda", generator=g)).to(torch.bfloat16)

    d, ff, V = SHAPE.d_model, SHAPE.d_ff, SHAPE.vocab
    return {"embed": mat(V, d, 1.0), "final_norm": gain(), "out_head": mat(V, d),
            "layers": [dict(attn_norm=gain(), wqkv=mat(3 * d, d), wo=mat(d, d), ffn_norm=gain(), w_gate_up=mat(2 * ff, d),
                            w_down=mat(d, ff)) for _ in range(SHAPE.n_layers)]}


def batches_unlike_the_largest(weights, T, R):
    ctx = make_context(SHAPE, weights, max_seqs=N_MAX, max_T=T, max_rows=R)
    toks = torch.from_numpy(np.stack([S.make_prompt(s, T, SHAPE.vocab, SHAPE.mask_id) for s in range(N_MAX)])).cuda()
    rows = torch.arange(T - R, T, dtype=torch.int32, device="cuda")[None].repeat(N_MAX, 1).contiguous()
    want = ctx.forward(toks, rows)
    return [n for n in range(1, N_MAX) if n * T > 640 and not torch.equal(ctx.forward(toks[:n].contiguous(), rows[:n].contiguous()), want[:n])]


@pytest.mark.parametrize("T", [229, 437, 715])
def test_ragged_canvases(weights, T):
    assert batches_unlike_the_largest(weights, T, T) == []


@pytest.mark.parametrize("T,R", [(704, 704), (704, 64), (1280, 128), (832, 832), (192, 64)])
def test_canvases_of_whole_tiles(weights, T, R):
    """The norm folded into the projections: the tile shapes of the launches that write the rows' sums of squares differ."""
    assert batches_unlike_the_largest(weights, T, R) == []


@pytest.mark.parametrize("T,R", [(229, 64), (437, 32), (715, 100)])
def test_few_rows_behind_a_large_forward(weights, T, R):
    """At most 640 rows reach the last layer's projections and the head: they too take no share of K there."""
    assert batches_unlike_the_largest(weights, T, R) == []


@pytest.mark.parametrize("S_,T,H", [(5, 512, 32), (3, 512, 32), (9, 1280, 32), (1, 64, 2), (2, 320, 4), (7, 192, 8)])
def test_rotation_in_the_projection_is_the_separate_pass(S_, T, H):
    d = H * 128
    g = torch.Generator(device="cuda").manual_seed(S_ * T + H)
    x = torch.randn(S_ * T, d, device="cuda", generator=g).to(torch.bfloat16)
    w = (torch.randn(3 * d, d, device="cuda", generator=g) * (1.6 / d ** 0.5)).to(torch.bfloat16)
    qkv, out = B.qkv_attention(x, w, S_, T, H, 128, 5e5)
    ref = B.gemm(x, w)
    ref_out = B.rope_attention(ref, S_, T, H, 128, 5e5)
    assert torch.equal(qkv, ref) and torch.equal(out, ref_out)
