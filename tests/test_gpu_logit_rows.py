"""Stage 1 and the entropy on rows that begin anywhere (a vocabulary that is no multiple of a 16-byte vector, a logits pointer
in the middle of one) and at the sizes where the block width changes, against float64."""
import numpy as np
import pytest
import torch

from paper_2601_12247_amd import binding as B

pytestmark = pytest.mark.gpu

# vectors a row: bf16 8, float32 4 elements; limits at 256 and 4096 vectors
CASES = [(V, dt) for dt, sizes in ((torch.bfloat16, (2047, 2048, 2049, 4101, 32767, 32768, 32775, 126461)),
                                   (torch.float32, (1023, 1025, 4099, 16383, 16386, 126467))) for V in sizes]


def reference(x, scale, mask_id):
    """x [rows, V] float32; logits scaled in float32 like the library, everything else in float64."""
    s = (x * np.float32(scale)).astype(np.float64)
    s[:, mask_id] = -np.inf
    m = s.max(1, keepdims=True)
    with np.errstate(invalid="ignore"):
        e = np.exp(s - m)
        te = np.where(e > 0, (s - m) * e, 0.0)
    Z = e.sum(1)
    return s.argmax(1), 1.0 / Z, np.log(Z) - te.sum(1) / Z


@pytest.mark.parametrize("V,dtype", CASES)
@pytest.mark.parametrize("shift", [0, 1, 3])
def test_rows_anywhere(V, dtype, shift):
    rows, scale = 9, 1.5
    rng = np.random.default_rng(V + shift)
    x = torch.from_numpy(rng.standard_normal((rows, V)).astype(np.float32)).to(dtype)
    for mask_id in (0, 5, V - 1, V - 9):
        y = x.clone()
        y[:, mask_id] = 60.0                                  # never counts
        for r, at in enumerate(((1, 2), (V - 2, V - 3), (6, V - 2), (1, V - 2), (V // 2, V // 2 + 1), (7, 8), (15, 16))):
            y[r, [at[0], at[1]]] = 4.0 + r                      # a tie: the lowest id
        y[7, 3:] = float("-inf")                                # three live ids at most
        y[8, V // 3] = 70.0                                     # one-hot to 40 digits
        buf = torch.empty(rows * V + 8, dtype=dtype, device="cuda")
        d = buf[shift:shift + rows * V].view(rows, V)
        d.copy_(y)
        tok, conf, ent = reference(y.float().numpy(), scale, mask_id)
        got_conf, got_tok = B.stage1(d, mask_id, scale)
        got_ent = B.entropy(d, mask_id, scale).cpu().numpy()
        assert np.array_equal(got_tok.cpu().numpy(), tok), mask_id
        # conf: float32 sums and exponentials (the bound of the stage 1 tests); entropy: x - max is rounded to float32, so a
        # term is off by |t| 2^-24 and the mean of t e^t by as much
        np.testing.assert_allclose(got_conf.cpu().numpy(), conf, rtol=5e-6)
        np.testing.assert_allclose(got_ent, ent, rtol=2e-6, atol=1e-38)


def test_entropy_of_rows_without_numbers():
    x = torch.zeros(4, 2050)
    x[0] = float("-inf")
    x[1, 5] = float("inf")
    x[2, 2049] = float("nan")
    got = B.entropy(x.cuda(), 7, 1.0).cpu()
    assert torch.isnan(got[:3]).all() and abs(got[3].item() - np.log(2049)) < 1e-5


@pytest.mark.parametrize("V", [2056, 4101, 126464])
def test_entropies_are_rounded_once(V):
    """One id far above the rest, which alternate between two values: every term but one then has the same error, and it shows.
    Exponentials of 1.1e-10 and float64 sums leave the final rounding to float32 as the only one, but where the exact value lies
    within 0.4 % of the middle between two floats (float32 exponentials: more than 3 % of the rows)."""
    rows, mask_id = 400, 11
    rng = np.random.default_rng(V)
    low, step = rng.uniform(2, 9, size=rows).astype(np.float32), rng.uniform(0.1, 6, size=rows).astype(np.float32)
    x = torch.from_numpy(np.where(np.arange(V)[None] % 2, -low[:, None], -(low + step)[:, None])).to(torch.bfloat16)
    x[torch.arange(rows), torch.from_numpy(rng.integers(12, V, size=rows))] = float(np.log(V))
    x[:, mask_id] = 60.0
    want = reference(x.float().numpy(), 1.0, mask_id)[2].astype(np.float32)
    got = B.entropy(x.cuda(), mask_id, 1.0).cpu().numpy()
    np.testing.assert_allclose(got, want, rtol=1.2e-7, atol=0)
    assert (got == want).mean() >= 0.97
