"""Gate/up projections on 160 x 192 tiles, whose waves hold gate or up columns alone (257-320 rows), and undivided launches
of few rows whose columns of tiles start inside K, against float64 products of the same bf16 inputs: rows at the edges of the
tiles, one and several rounds, either side of the rule that takes them, with a context and without."""
import numpy as np
import pytest
import torch

from paper_2601_12247_amd import binding as B
from tests.test_gpu_gemm_splitk import ctx, reference  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(257, 3072, 512), (272, 9216, 1024), (319, 6144, 2048), (320, 12288, 4096), (300, 16512, 512),
                                   (264, 7680, 8192), (311, 1536, 512), (300, 9216, 1088), (260, 3072, 576), (256, 3072, 512), (321, 3072, 512),
                                   (500, 3072, 2048), (192, 9216, 2048), (576, 6144, 2112)])
def test_swiglu_every_element(ctx, M, N, K):  # noqa: F811
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = torch.randn(M, K, device="cuda", generator=g).to(torch.bfloat16)
    W = (torch.randn(2 * N, K, device="cuda", generator=g) * 0.02).to(torch.bfloat16)
    want = reference(A, W, "swiglu", None, N)
    tol = 2.0 ** -8 * np.abs(want) + 2e-4                 # one bf16 rounding of a float32 sum
    outs = [ctx.gemm_swiglu(A, W), B.gemm_swiglu(A, W), ctx.gemm_swiglu(A, W)]
    for got in outs[:2]:
        assert (np.abs(got.float().cpu().numpy() - want) <= tol).all()
    assert torch.equal(outs[0], outs[2])
