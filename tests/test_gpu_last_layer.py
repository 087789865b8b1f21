"""Behind the attention of the last layer only the rows that logits are wanted for go on: their logits are those of a
forward that asks for every row, whatever rows are asked for, in whatever order."""
import numpy as np
import pytest
import torch

from oracle import pvf_oracle as O
from synth import inputs as S
from tests.gpu_util import make_context, oracle_model_cfg, to_device

pytestmark = pytest.mark.gpu

ROWS = {"one": [5], "shuffled, repeated, padding": [40, 3, -1, 40, 39, 0], "all but one": list(range(47))}


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", torch.int32)


@pytest.mark.parametrize("layers", [1, 2])
@pytest.mark.parametrize("rows", list(ROWS))
def test_rows_of_a_float32_forward(rows, layers):
    shape = S.TINY
    T, S_ = 48, 2
    w = S.make_weights(shape, seed=0)
    w["layers"] = w["layers"][:layers]
    ctx = make_context(shape, to_device(w), max_seqs=S_, max_T=T, max_rows=T, n_layers=layers)
    toks = dev(np.stack([S.make_prompt(s, T, shape.vocab, shape.mask_id) for s in range(S_)]))
    whole = ctx.forward(toks, dev(np.tile(np.arange(T), (S_, 1))))
    r = np.array(ROWS[rows])
    got = ctx.forward(toks, dev(np.tile(r, (S_, 1))))
    assert torch.equal(got[:, r >= 0], whole[:, r[r >= 0]]) and not got[:, r < 0].any()


@pytest.mark.parametrize("S_,T,R", [(2, 128, 1), (3, 64, 63), (6, 128, 40), (7, 100, 128 - 28)])
def test_rows_of_a_bf16_forward(S_, T, R):
    """Up to 640 rows (K may be divided) and above (it is not), few rows and all of them."""
    shape = S.ModelShape(n_layers=2, d_model=256, n_heads=2, d_ff=512, vocab=2048, mask_id=2047, rope_theta=5e5)
    w = S.make_weights(shape, seed=3, round_to_bf16=True)
    ctx = make_context(shape, to_device(w, torch.bfloat16), max_seqs=S_, max_T=T, max_rows=R)
    toks = np.stack([S.make_prompt(s, T, shape.vocab, shape.mask_id) for s in range(S_)])
    rows = np.tile(np.random.default_rng(R).permutation(T)[:R].astype(np.int32), (S_, 1))
    got = ctx.forward(dev(toks), dev(rows)).float().cpu().numpy()
    for s in range(S_):
        want = O.forward(toks[s], w, oracle_model_cfg(shape), rows=rows[s])
        assert np.abs(got[s] - want).max() <= 5e-2
