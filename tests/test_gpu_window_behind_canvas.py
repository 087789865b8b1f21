"""K/V-cached rounds, bf16, d_head = 128, of a group that is not done but whose active block lies behind the canvas: its window has
no positions, the decision step answers with an empty round, and nothing of the groups beside it changes."""
import numpy as np
import pytest
import torch

from paper_2601_12247_amd import binding as B
from tests.gpu_util import make_context
from tests.test_gpu_window_shapes import dev, models  # noqa: F401

pytestmark = pytest.mark.gpu


# QKV that splits K (partial sums go to the rotary pass), the rotary pass behind whole sums, the rotation in the epilogue of small and of
# large tiles; canvases of whole 16-key groups and not
@pytest.mark.parametrize("d,K,bl,pl,gl", [(512, 4, 16, 48, 96), (512, 2, 16, 37, 96), (512, 4, 36, 45, 144), (512, 5, 48, 90, 144),
                                          (2048, 1, 16, 32, 96), (512, 4, 48, 96, 144)])
@pytest.mark.parametrize("behind", [0, 1, 5])
def test_empty_round(models, d, K, bl, pl, gl, behind):  # noqa: F811
    shape, w, wd = models(d)
    cfg = B.DecodeCfg(block_len=bl, prompt_len=pl, gen_len=gl, K=K, tau_high=0.9, logit_scale=shape.logit_scale, kv_cache=1)
    ctx = make_context(shape, wd, max_seqs=2 * (1 + K), max_T=cfg.T, max_rows=cfg.R)
    rng = np.random.default_rng(d + pl + behind)
    canvas = rng.integers(0, shape.mask_id, size=(2, 1, cfg.T)).repeat(1 + K, axis=1)
    at = pl + bl + np.arange(K)                              # block 1 lacks K positions; every draft fills one of them
    canvas[:, :, at] = shape.mask_id
    canvas[:, 1 + np.arange(K), at] = 11
    st = B.State(2, cfg)

    def round_of(active):
        st.canvas.copy_(dev(canvas)); st.fill_pos.copy_(dev(np.tile(at, (2, 1)))); st.fill_tok.fill_(11)
        st.n_drafts.fill_(K); st.draft_route.fill_(B.PVF_ROUTE_PLAN); st.n_ws_blocks.fill_(1); st.done.zero_()
        st.k_active.copy_(dev(np.array(active)))
        status = ctx.round_sync(st, dev(np.zeros((shape.vocab + 31) // 32)))
        return status, [t.clone() for t in (st.conf, st.tok, st.canvas, st.n_drafts, st.winner, st.accept)]

    end = gl // bl + behind
    round_of([1, 1])                                         # fills both caches
    status, want = round_of([1, 1])
    assert status[0][0] == 0
    first, got1 = round_of([1, end])                         # the second group's backbone runs whole, its drafts' windows are empty
    second, got2 = round_of([1, end])                        # every window
    assert first[1] == second[1] == (1, 0, 0, 0, 0)
    assert second[0] == status[0]
    for a, b in zip(want, got2):
        assert torch.equal(a[0], b[0])
    for _, _, cv, *_ in (got1, got2):
        assert torch.equal(cv[1, 0].cpu(), torch.from_numpy(canvas[1, 0].astype(np.int32)))
    for conf, tok, *_ in (got1, got2):
        assert bool((conf[1] == 0).all()) and bool((tok[1] == -1).all())
