"""The counting kernel behind the entropies of long bf16 rows: every way a row can take through it, against float64."""
import numpy as np
import pytest
import torch

from paper_2601_12247_amd import binding as B
from tests.test_gpu_logit_rows import reference

pytestmark = pytest.mark.gpu
V = 28_011                                                   # just above the limit; rows begin anywhere



def rows_of(seed):
    """name -> row of V bf16 values"""
    rng = np.random.default_rng(seed)
    n = lambda s=1.0: rng.standard_normal(V).astype(np.float32) * np.float32(s)
    far = n(); far[4500:4520] = 4000.0 * np.abs(far[4500:4520]) + 100       # behind the sample, above the counters' range: listed
    many = n(); many[6000:8000] *= 5000.0                                   # more of them than the list holds
    tiny = n(); tiny[5000:5900] *= np.float32(2.0 ** -40)
    zeros = n(); zeros[::3] = 0.0
    masked = n(); masked[rng.random(V) < 0.9] = -np.inf
    lowest = n(); lowest[rng.random(V) < 0.9] = -3.3895314e38               # the type's lowest value
    late = np.full(V, -3.3895314e38, np.float32); late[V - 3:] = [1.0, 2.0, 0.5]
    flat = np.full(V, -3.3895314e38, np.float32)
    hot = n(); hot[V // 2] = 90.0
    return {"normal": n(), "wide": n(60.0), "narrow": n(1e-6), "huge": n(1e30), "listed": far, "overflow": many, "tiny": tiny,
            "zeros": zeros, "masked": masked, "lowest": lowest, "late": late, "flat": flat, "one-hot": hot,
            "constant": np.full(V, 1.5, np.float32), "few": np.round(n(2.0)) / 2, "negative": -40 + n(3.0),
            "neighbours": np.repeat(rng.standard_normal(V // 8 + 1), 8)[:V].astype(np.float32)}


@pytest.mark.parametrize("scale", [1.0, 1.5, 0.03])
def test_every_route(scale):
    rows = rows_of(3)
    for mask_id in (0, 4097, V - 1):
        x = torch.from_numpy(np.stack(list(rows.values()))).to(torch.bfloat16)
        x[:, mask_id] = 1e38                                 # never counts
        _, _, ent = reference(x.float().numpy(), scale, mask_id)
        got = B.entropy(x.cuda(), mask_id, scale).cpu().numpy()
        for name, g, w in zip(rows, got, ent):
            # float64 sums of terms that are 1.1e-10 off, one rounding to float32 (the bound of the neighbouring tests)
            # (lowest value times 1.5 is -inf: a row of nothing else has no entropy)
            assert (np.isnan(w) and np.isnan(g)) or abs(g - w) <= 2e-6 * abs(w) + 1e-38, (name, mask_id, g, w)


def test_scales_so_small_that_no_value_is_negligible():
    """At 2e-38 the type's lowest value lies 7 below the row's maximum."""
    rows = rows_of(4)
    x = torch.from_numpy(np.stack(list(rows.values()))).to(torch.bfloat16)
    for scale in (2e-38, 1e-37, 1e-36):
        _, _, ent = reference(x.float().numpy(), scale, 7)
        got = B.entropy(x.cuda(), 7, scale).cpu().numpy()
        for name, g, w in zip(rows, got, ent):
            assert abs(g - w) <= 2e-6 * abs(w) + 1e-38, (name, scale, g, w)


@pytest.mark.parametrize("listed", [2, 63, 64, 65, 900])
def test_listed_elements_are_added_in_one_order(listed):
    """Equal rows, whose elements beyond the counters' range reach the list in any order: one value above them, the others 30-33
    below it, so that the order of the sums shows in the entropy."""
    n = 28_032
    rng = np.random.default_rng(6)
    x = 0.1 * rng.standard_normal(n).astype(np.float32)
    at = np.arange(4096, n)
    at = rng.permutation(at[(at // 8 % 112 >= 12) & (at // 8 % 112 < 108)])[:listed]      # between the places that the range is taken from
    x[at] = 40 + rng.integers(0, 13, listed) / 4
    x[at[listed // 2]] = 73
    rows = torch.from_numpy(x).to(torch.bfloat16).cuda()[None].repeat(512, 1)
    first = B.entropy(rows, 3, 1.0)
    for _ in range(8):
        assert torch.equal(B.entropy(rows, 3, 1.0), first)
    assert (first == first[0]).all()
    _, _, ent = reference(rows[:1].float().cpu().numpy(), 1.0, 3)
    assert abs(first[0].item() - ent[0]) <= 1e-5 * ent[0]    # S is 1 and a few 1e-11, rounded at 2^-53


@pytest.mark.parametrize("n", [V, 28_032, 126_464])
def test_rows_that_change_along_the_way(n):
    """Rows whose front says nothing about what follows, and values in any number of the counters' ranges."""
    rng = np.random.default_rng(n)
    f = lambda: rng.standard_normal(n).astype(np.float32)
    behind, front, tiny, huge, off = f(), f(), f(), f(), f()
    behind[n // 2:] = -3.25
    front[:n // 2] = -3.25
    tiny[5000:] *= 1e-6
    huge[5000:] *= 1e4
    off[2000:] = -np.inf
    zeros = {p: f() for p in (0.002, 0.01, 0.2)}             # listed; about as many as the list holds; left at once
    for p, x in zeros.items():
        x[rng.random(n) < p] = 0.0
    ranges = f()
    at = rng.permutation(n)[:700]
    ranges[at] *= np.float32(2.0) ** rng.integers(-110, -27, 700)
    masked = f()
    masked[rng.random(n) < 0.3] = -1e9
    x = torch.from_numpy(np.stack([behind, front, tiny, huge, off, *zeros.values(), ranges, masked])).to(torch.bfloat16)
    for mask_id in (1, n - 1):
        _, _, ent = reference(x.float().numpy(), 1.0, mask_id)
        got = B.entropy(x.cuda(), mask_id, 1.0).cpu().numpy()
        np.testing.assert_allclose(got, ent, rtol=2e-6, atol=1e-38)      # the bound of the tests above


@pytest.mark.parametrize("n", [27_999, 28_000, 28_007, 28_008])
def test_limit_of_counting(n):
    """Rows of 3500 vectors are counted, shorter ones are not; rows begin anywhere."""
    x = torch.from_numpy(np.random.default_rng(n).standard_normal((9, n)).astype(np.float32)).to(torch.bfloat16)
    _, _, ent = reference(x.float().numpy(), 1.5, n // 3)
    np.testing.assert_allclose(B.entropy(x.cuda(), n // 3, 1.5).cpu().numpy(), ent, rtol=2e-6)


def test_rows_without_numbers():
    x = torch.from_numpy(np.stack([rows_of(5)["normal"]] * 5)).to(torch.bfloat16)
    x[0], x[1, 77], x[2, V - 1], x[3, 9] = float("-inf"), float("inf"), float("nan"), float("nan")
    got = B.entropy(x.cuda(), 9, 1.0).cpu()
    assert torch.isnan(got[:3]).all() and got[3] == got[4]   # the NaN of row 3 is the [MASK] column


def test_calibration_state_of_long_rows():
    """conf, tok and ent of one calibration step, with rows that are not there, ties and the mask column on top."""
    G, K, bl, gen = 2, 3, 16, 32
    cfg = B.DecodeCfg(block_len=bl, prompt_len=0, gen_len=gen, K=K, logit_scale=1.5, routes=B.PVF_ROUTES_CAL)
    rng = np.random.default_rng(8)
    lg = torch.from_numpy(rng.standard_normal((G, 1 + K, cfg.R, V)).astype(np.float32)).to(torch.bfloat16)
    mask_id = V - 5
    lg[..., mask_id] = 50.0
    lg[0, 0, 0, [17, 18_000]] = 9.0                          # a tie: the lowest id
    lg[1, 1, 3, [0, V - 1]] = 9.0
    st = B.State(G, cfg, vocab=V)
    st.canvas.fill_(mask_id)
    st.n_drafts.copy_(torch.tensor([K, 1]))
    st.draft_route.fill_(B.PVF_ROUTE_CAL)
    bitmap = torch.zeros((V + 31) // 32, dtype=torch.int32, device="cuda")
    B.epilogue(lg.cuda(), st, bitmap, V, mask_id)
    live = torch.tensor([[True] * 4, [True, True, False, False]])
    tok, conf, ent = reference(lg.float().numpy().reshape(-1, V), 1.5, mask_id)
    shape = (G, 1 + K, cfg.R)
    got_tok, got_conf, got_ent = st.tok.cpu()[live], st.conf.cpu()[live], st.ent.cpu()[live]
    assert np.array_equal(got_tok.numpy(), tok.reshape(shape)[live.numpy()])
    np.testing.assert_allclose(got_conf.numpy(), conf.reshape(shape)[live.numpy()], rtol=2e-7)
    np.testing.assert_allclose(got_ent.numpy(), ent.reshape(shape)[live.numpy()], rtol=2e-7)
    assert (st.tok.cpu()[~live] == -1).all() and not st.ent.cpu()[~live].any()
