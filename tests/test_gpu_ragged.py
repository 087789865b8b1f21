"""bf16 canvases whose length is no multiple of a key tile, and decode windows that begin or end anywhere, on the matrix
cores (d_head = 128): the attention kernel alone against float64, whole forwards and K/V-cached rounds against the oracle."""
import numpy as np
import pytest
import torch

from oracle import pvf_oracle as O
from paper_2601_12247_amd import binding as B
from synth import inputs as S
from tests.gpu_util import make_context, oracle_model_cfg, to_device

pytestmark = pytest.mark.gpu

SHAPE = S.ModelShape(n_layers=2, d_model=256, n_heads=2, d_ff=512, vocab=2048, mask_id=2047, rope_theta=5e5, logit_scale=6.0)


def dev(a, dtype=torch.int32):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda", dtype)


@pytest.fixture(scope="module")
def model():
    w = S.make_weights(SHAPE, seed=3, round_to_bf16=True)
    return w, to_device(w, torch.bfloat16)


@pytest.mark.parametrize("T", [1, 15, 63, 65, 96, 127, 437])
def test_attention_of_any_length(T):
    """q, k come back rotated, so the float64 reference starts from what the kernel read.  An output is one bf16 rounding
    away (8 significant bits: at most 2^-8 of the value), plus the probabilities' 2^-16 and the float32 exponentials' and
    sums' 2^-18 of the largest value."""
    S_, H, dh = 2, 2, 128
    d = H * dh
    g = torch.Generator(device="cuda").manual_seed(T)
    qkv = (torch.randn(S_ * T, 3 * d, device="cuda", generator=g) * 1.5).to(torch.bfloat16)
    out = B.rope_attention(qkv, S_, T, H, dh, 5e5).double().cpu()
    q, k, v = qkv.double().cpu().view(S_, T, 3, H, dh).permute(2, 0, 3, 1, 4)
    want = (torch.softmax(q @ k.transpose(-1, -2) / dh ** 0.5, -1) @ v).permute(0, 2, 1, 3).reshape(S_ * T, d)
    tol = 2.0 ** -8 * want.abs() + 2.0 ** -15 * v.abs().max()
    assert ((out - want).abs() <= tol).all(), float(((out - want).abs() / tol).max())


@pytest.mark.parametrize("T", [65, 127, 437])
def test_probabilities_keep_24_bits(T):
    """Values of +1 and -1 under weights p and p (1 + delta), delta = 8.6e-5: what is left is 1e4 times smaller than the weights, so
    it shows their last bits.  An exponent below 4 rounds to 2^-22 / 2 (x ln 2), the hardware exponential to 2^-23, together 2.9e-7 a
    weight and 0.7 % of delta for two; the output's own rounding is 2^-9.  Weights of 16 bits (2^-18) are up to 12 % off here."""
    dh = 128
    qkv = torch.zeros(T, 3 * dh, dtype=torch.bfloat16)
    j = torch.arange(T)
    qkv[:, 60], qkv[:, 61] = 2.0 ** -3, 8 * (1 + (j % 64) / 64)           # a theta of 1e30 leaves these columns as they are
    qkv[:, dh + 60] = 1 + (j % 2) / 128
    qkv[:, 2 * dh:] = (2.0 * (j % 2) - 1)[:, None]
    qkv[0, dh + 61], qkv[0, dh + 60], qkv[0, 2 * dh:] = 2, 0, 0            # this key has the largest weight, and no value
    out = B.rope_attention(qkv.cuda(), 1, T, 1, dh, 1e30).double().cpu()
    q, k, v = qkv.double().split(dh, -1)
    want = torch.softmax(q @ k.T / dh ** 0.5, -1) @ v
    assert want.abs().max() <= 1e-3 and float(((out - want).abs() / want.abs()).max()) <= 0.009


@pytest.mark.parametrize("T", [1, 17, 65, 127, 437])
def test_infinite_values(T):
    """Every weight is above zero, so an infinite value of any key gives that infinity and no other column is touched."""
    H, dh = 2, 128
    d = H * dh
    g = torch.Generator(device="cuda").manual_seed(T)
    qkv = torch.randn(T, 3 * d, device="cuda", generator=g).to(torch.bfloat16)
    qkv[T - 1, 2 * d + 3], qkv[T - 1, 2 * d + dh + 5], qkv[0, 2 * d + 9] = float("inf"), float("-inf"), float("inf")
    got = B.rope_attention(qkv, 1, T, H, dh, 5e5)
    want = torch.zeros(d, device="cuda")
    want[3], want[dh + 5], want[9] = float("inf"), float("-inf"), float("inf")
    inf = torch.isinf(want)
    assert torch.equal(got[:, inf].float(), want[inf].expand(T, 3)) and bool(torch.isfinite(got[:, ~inf]).all())


@pytest.mark.parametrize("S_,T", [(3, 100), (2, 81), (3, 208), (5, 150), (1, 40), (1, 1)])
def test_forward_of_ragged_canvases(model, S_, T):
    """Also: what an earlier, longer call left in the workspace must not show."""
    w, wd = model
    R = min(T, 37)
    toks = np.stack([S.make_prompt(s, T, SHAPE.vocab, SHAPE.mask_id) for s in range(S_)])
    toks[:, T // 2:] = SHAPE.mask_id
    rows = np.tile(np.arange(T - R, T, dtype=np.int32), (S_, 1))
    ctx = make_context(SHAPE, wd, max_seqs=S_, max_T=T + 90, max_rows=64)
    long = dev(np.stack([S.make_prompt(50 + s, T + 90, SHAPE.vocab, SHAPE.mask_id) for s in range(S_)]))
    first = ctx.forward(dev(toks), dev(rows))
    ctx.forward(long, dev(rows))
    got = ctx.forward(dev(toks), dev(rows))
    assert torch.equal(first, got)
    for s in range(S_):
        want = O.forward(toks[s], w, oracle_model_cfg(SHAPE), rows=rows[s])
        assert np.abs(got[s].float().cpu().numpy() - want).max() <= 5e-2


@pytest.mark.parametrize("bl,pl,gl", [(16, 37, 64), (32, 203, 128), (64, 77, 192), (24, 65, 72), (10, 3, 50)])
def test_cached_round_with_a_window_anywhere(model, bl, pl, gl):
    """On the canvas that filled the cache a cached round is exact, so both rounds have the oracle's confidences and clear tokens;
    every block in turn is the active one, the last with its window cut by the end of the canvas."""
    w, wd = model
    G, mc = 2, oracle_model_cfg(SHAPE)
    cfg = B.DecodeCfg(block_len=bl, prompt_len=pl, gen_len=gl, K=0, tau_high=0.9, logit_scale=SHAPE.logit_scale, kv_cache=1)
    ctx = make_context(SHAPE, wd, max_seqs=G, max_T=cfg.T, max_rows=cfg.R)
    bitmap = torch.zeros((SHAPE.vocab + 31) // 32, dtype=torch.int32, device="cuda")
    for k in range(gl // bl):
        canvas = np.stack([S.make_prompt(9 * g + k, cfg.T, SHAPE.vocab, SHAPE.mask_id) for g in range(G)])
        canvas[:, pl + k * bl:] = SHAPE.mask_id
        confs = []
        for _ in range(2):                                   # fills the cache, then uses it
            st = confs[0][0] if confs else B.State(G, cfg)
            st.canvas.copy_(dev(canvas)[:, None]); st.k_active.fill_(k); st.done.zero_(); st.n_drafts.zero_(); st.n_ws_blocks.fill_(1)
            ctx.round(st, bitmap, 0)
            torch.cuda.synchronize()
            confs.append((st, st.conf[:, 0].cpu().numpy().copy(), st.tok[:, 0].cpu().numpy().copy()))
        n = min(cfg.R, cfg.T - (pl + k * bl))
        for g in range(G):
            logits = O.forward(canvas[g], w, mc, rows=np.arange(pl + k * bl, pl + k * bl + n))
            conf, tok = O.stage1(logits.astype(np.float32), SHAPE.logit_scale, SHAPE.mask_id)
            for i, (_, c, t) in enumerate(confs):
                diff = np.abs(c[g][:n] - conf)
                assert diff.max() <= 2e-2 and diff.mean() <= 4e-3, (k, i, float(diff.max()), float(diff.mean()))
                # bf16 logits hold to 5e-2: a best one that leads by twice that stays the best
                live = np.delete(logits, SHAPE.mask_id, axis=1)
                top = -np.sort(-live, axis=1)[:, :2]
                sure = top[:, 0] - top[:, 1] > 0.1
                assert np.array_equal(t[g][:n][sure], tok[sure]), (k, i)
