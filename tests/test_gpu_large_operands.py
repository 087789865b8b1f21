"""GEMM operands between 2 and 4 GiB: the 256 x 256, 192 x 256 and 256 x 192 tiles address them by 32-bit offsets from a buffer
descriptor, and half of these offsets have the upper bit set."""
import pytest
import torch

from paper_2601_12247_amd import binding as B

pytestmark = pytest.mark.gpu

K = 12288
FAR = 2 ** 31 // (2 * K)                                       # the row behind the first 2 GiB


def normal(rows, seed, std=1.0):
    t = torch.empty(rows, K, dtype=torch.bfloat16, device="cuda")
    B.fill_normal(t, seed, 0.0, std)
    return t


def close(got, want, slack):
    """One bf16 rounding of the sum; float32 sums of 12288 products of |a w| ~ 0.01 are 1e-6 to 1e-5 apart by their order."""
    bad = (got.float() - want).abs() > 2.0 ** -8 * want.abs() + slack
    assert not bool(bad.any()), (int(bad.sum()), bad.nonzero()[:4].tolist())


def test_left_operand():
    M, N = 90112, 1024                                       # 256 x 256 tiles
    A, W = normal(M, 1), normal(N, 2, 0.01)
    out = B.gemm(A, W)
    Wt = W.float().T.contiguous()
    for rows in (slice(0, 64), slice(FAR - 64, FAR + 64), slice(M - 64, M)):
        close(out[rows], A[rows].float() @ Wt, 1e-4)


@pytest.mark.parametrize("swiglu,N", [(False, 90112), (True, 45056), (True, 45120)])        # 192 x 256 twice, 256 x 192
def test_weights(swiglu, N):
    M, rows = 768, torch.arange(0, 768, 13, device="cuda")
    A, W = normal(M, 3), normal(2 * N if swiglu else N, 4, 0.01)
    want = A[rows].float() @ W.float().T
    if not swiglu:
        close(B.gemm(A, W)[rows], want, 1e-4)
        return
    g, u = want[:, :N], want[:, N:]
    close(B.gemm_swiglu(A, W)[rows], torch.nn.functional.silu(g) * u, 1e-4 * (1 + g.abs() + u.abs()))
