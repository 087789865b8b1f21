"""Launches that leave CUs idle in their last round, whose extra workgroups touch weights ahead (K of 1024 or more, 16 MB of weights or more): every
element against float64 products, for tiles in one and several rounds, several bands of tile rows, columns that no prefetching
workgroup has, one stage past the first ones, and shapes with a single column."""
import numpy as np
import pytest
import torch

from tests.test_gpu_gemm_splitk import ctx, reference  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,kind", [(65, 8192, 1024, "store"), (128, 9216, 1088, "store"), (96, 8256, 1024, "store"),
                                        (130, 128, 65536, "residual"), (640, 8192, 1088, "residual"), (1311, 4096, 2048, "residual"),
                                        (2200, 1024, 8192, "residual"), (4100, 384, 22016, "store"), (3000, 1280, 6592, "store"),
                                        (192, 9216, 1024, "swiglu"), (700, 2752, 2048, "swiglu"), (1100, 5504, 1088, "swiglu"),
                                        (300, 9216, 1024, "swiglu"), (100, 4096, 1024, "swiglu")])
def test_every_element(ctx, M, N, K, kind):  # noqa: F811
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = torch.randn(M, K, device="cuda", generator=g).to(torch.bfloat16)
    W = (torch.randn(N * (2 if kind == "swiglu" else 1), K, device="cuda", generator=g) * 0.02).to(torch.bfloat16)
    Rz = torch.randn(M, N, device="cuda", generator=g).to(torch.bfloat16) if kind == "residual" else None
    out = ctx.gemm_swiglu(A, W) if kind == "swiglu" else ctx.gemm(A, W, residual=Rz)
    want = reference(A, W, kind, Rz, N)
    tol = 2.0 ** -8 * np.abs(want) + 2e-4                 # one bf16 rounding of a float32 sum
    assert (np.abs(out.float().cpu().numpy() - want) <= tol).all()
