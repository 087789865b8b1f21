"""The float32 norm of a row is one and the same on every route: here as a pass, at any alignment, and in cached rounds."""
import pytest
import torch

from paper_2601_12247_amd import binding as B
from paper_2601_12247_amd import workloads as W
from tests.test_gpu_f32_rounds import DIMS, model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,d", [(1, 8), (33, 255), (70, 256), (5, 1000), (64, 1023), (31, 1024)])
@pytest.mark.parametrize("shift", [0, 1, 2])
def test_rows_against_float64(M, d, shift):
    """A float32 norm is its float64 value within a rounding of 1 / rms, of x / rms and of the product with the gain."""
    g = torch.Generator(device="cuda").manual_seed(d)
    x = torch.randn(M, d, device="cuda", generator=g) * 10 ** (4 * torch.rand(M, 1, device="cuda", generator=g) - 2)
    gain = 1 + 0.1 * torch.randn(d, device="cuda", generator=g)
    want = x.double() / (x.double().square().mean(1, keepdim=True) + float(torch.tensor(1e-5))).sqrt() * gain
    buf = torch.empty(M * d + d + 8, device="cuda")
    a, b = buf[shift:shift + M * d].view(M, d).copy_(x), torch.empty(d + 4, device="cuda")[shift:shift + d].copy_(gain)
    got = B.rmsnorm(a, b, 1e-5)
    assert bool(((got.double() - want).abs() <= 3 * 2.0 ** -24 * want.abs() + 1e-44).all())
    assert torch.equal(got, B.rmsnorm(x, gain, 1e-5))


@pytest.mark.parametrize("shift", [0, 1])
def test_cached_round_follows_the_forward(shift):
    """The window rows of a cached round with the cache just filled are the rows of the full forward, up to the order of the
    attention's keys (all of them in float64 sums; the softmax sums in float32): a few 2^-24 through two layers."""
    cfg = B.DecodeCfg(block_len=16, prompt_len=20, gen_len=64, K=0, tau_high=0.9, logit_scale=6.0, kv_cache=1)
    plain = B.DecodeCfg(block_len=16, prompt_len=20, gen_len=64, K=0, tau_high=0.9, logit_scale=6.0)
    ctx = W.make_context(DIMS, model(offset=shift), max_seqs=1, max_T=cfg.T, max_rows=cfg.R)
    bitmap = W.random_plan_bitmap(64, DIMS["vocab"], DIMS["mask_id"], seed=1)
    prompt = W.random_prompts(1, 20, DIMS["vocab"], DIMS["mask_id"], seed=2)
    a, b = B.State(1, cfg), B.State(1, plain)
    for st in (a, b):
        ctx.state_init(st, prompt)
    ctx.round_sync(a, bitmap)                                # fills the cache
    for t, u in ((a.canvas, b.canvas), (a.k_active, b.k_active)):
        t.copy_(u)                                           # the first round again, from the cache
    for t, u in ((a.done, b.done), (a.n_ws_blocks, b.n_ws_blocks)):
        t.copy_(u)
    ctx.round_sync(a, bitmap)
    ctx.round_sync(b, bitmap)
    assert torch.equal(a.tok, b.tok)
    assert (a.conf - b.conf).abs().max() <= 2e-5 * b.conf.abs().max()
