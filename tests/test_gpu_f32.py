"""The float32 matrix-core kernels (float64 sums) at the sizes where their tiling can go wrong, against float64 NumPy.

Tolerance: operands are float32, products exact and sums float64, so what is left is the one rounding of the result
to float32 (2^-24 relative) -- held at 2^-23; attention also rounds scores and probabilities to float32 (below)."""
import numpy as np
import pytest
import torch

from oracle import pvf_oracle as O
from paper_2601_12247_amd import binding as B

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# one row, tile edges +-1, K below one chunk / no multiple of 16 / of 4 (the unvectorised loads), more chunks than the four
# waves can share evenly
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (31, 33, 16), (32, 32, 64), (33, 31, 20), (64, 96, 7), (65, 65, 272), (3, 4096, 256),
                                   (1473, 1471, 68), (2050, 1030, 30)])
def test_gemm_f32(M, N, K):
    rng = np.random.default_rng(M + N + K)
    A, W, R = (rng.standard_normal(s, dtype=np.float32) for s in ((M, K), (N, K), (M, N)))
    want = A.astype(np.float64) @ W.astype(np.float64).T
    near = lambda got, ref: np.all(np.abs(got.cpu().numpy() - ref) <= 2.0 ** -23 * np.abs(ref) + 1e-12)
    assert near(B.gemm(dev(A), dev(W)), want)
    r = dev(R)
    assert near(B.gemm(dev(A), dev(W), residual=r, out=r), want + R)
    if N % 2 == 0:
        g, u = want[:, :N // 2], want[:, N // 2:]
        assert near(B.gemm_swiglu(dev(A), dev(W)), g / (1 + np.exp(-g)) * u)


# key tiles of 16 and their remainders, fewer tiles than waves, every head size, scores close to the LDS limit
@pytest.mark.parametrize("S,T,H,dh", [(1, 1, 1, 16), (2, 15, 2, 64), (1, 17, 3, 32), (2, 63, 2, 128), (1, 65, 2, 64), (3, 229, 4, 64),
                                      (1, 100, 2, 48), (1, 2304, 1, 16)])
def test_attention_f32(S, T, H, dh):
    rng = np.random.default_rng(T + dh)
    d = H * dh
    qkv = rng.standard_normal((S * T, 3 * d), dtype=np.float32)
    got = B.rope_attention(dev(qkv), S, T, H, dh, 1e4).cpu().numpy()
    for s in range(S):
        q, k, v = (qkv[s * T:(s + 1) * T, i * d:(i + 1) * d].astype(np.float64).reshape(T, H, dh) for i in range(3))
        want = O.attention(O.rope(q, 1e4), O.rope(k, 1e4), v).reshape(T, d)
        # |score| <= 20 rounded to float32 moves a weight by 20 * 2^-24 relative, the weight's own chain
        # (exp, sum, product) by a few 2^-24 more: 4e-6 of max |v| = 5
        assert np.abs(got[s * T:(s + 1) * T] - want).max() <= 2e-5


# the last tile of 16 keys whole, with one to three keys (fewer than the four a lane takes), with 15; values that are read again for the padding keys are infinite
@pytest.mark.parametrize("T,dh", [(16, 64), (17, 32), (18, 64), (35, 16), (31, 128), (229, 64)])
def test_attention_f32_of_infinite_values(T, dh):
    """Every weight is above zero, so an infinite value of any key gives that infinity and no other column is touched."""
    rng = np.random.default_rng(T)
    H, d = 2, 2 * dh
    qkv = rng.standard_normal((T, 3 * d), dtype=np.float32)
    qkv[T - 1, 2 * d + 3], qkv[T - 1, 2 * d + dh + 5], qkv[0, 2 * d + 9] = np.inf, -np.inf, np.inf
    got = B.rope_attention(dev(qkv), 1, T, H, dh, 1e4).cpu().numpy()
    q, k, v = (qkv[:, i * d:(i + 1) * d].astype(np.float64).reshape(T, H, dh) for i in range(3))
    want = O.attention(O.rope(q, 1e4), O.rope(k, 1e4), v).reshape(T, d)
    inf = np.isinf(want)
    assert inf.sum() == 3 * T and np.array_equal(got[inf], want[inf]) and np.abs(got[~inf] - want[~inf]).max() <= 2e-5


# 16- and 32-row tiles, chunks of 16 k (whole, cut at a multiple of 4, element by element) and their odd and even numbers per wave
@pytest.mark.parametrize("K", [16, 60, 64, 130, 192, 256, 260, 704])
@pytest.mark.parametrize("kind", ["store", "residual", "swiglu"])
def test_rows_of_launches_of_any_size(kind, K):
    """A row has the same bits whatever the launch: tile heights follow the number of workgroups, the order of k does not."""
    rng = np.random.default_rng(K)
    N = 352                                    # 1 100 rows: 11 (22) columns of tiles, 16 rows for the short launches and 32 for the long one
    A, W, R = (dev(rng.standard_normal(s, dtype=np.float32)) for s in ((1100, K), (2 * N, K), (1100, N)))

    def run(rows):
        a, r = A[rows].contiguous(), R[rows].clone()
        return B.gemm_swiglu(a, W) if kind == "swiglu" else B.gemm(a, W[:N].contiguous(), residual=r if kind == "residual" else None, out=r)

    whole = run(slice(0, 1100))
    for rows in (slice(0, 1), slice(3, 50), slice(1071, 1100), slice(500, 900)):
        assert torch.equal(run(rows), whole[rows])
    want = A.double() @ W.double().T
    want = torch.nn.functional.silu(want[:, :N]) * want[:, N:] if kind == "swiglu" else want[:, :N] + (R.double() if kind == "residual" else 0)
    assert bool(((whole.double() - want).abs() <= 2.0 ** -23 * want.abs() + 1e-12).all())
