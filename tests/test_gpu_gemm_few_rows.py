"""Launches of few rows that take the whole of K (context GEMMs of wide projections), and the ones that divide it where the tile
shapes change: every element against float64
products of the same bf16 inputs, on both sides of the limits in rows, columns and K, with fewer stages than the rings hold, with
columns of tiles that start inside K, and last tiles with few rows."""
import pytest
import torch

from synth import inputs as S
from tests.gpu_util import make_context, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    shape = S.ModelShape(n_layers=1, d_model=256, n_heads=2, d_ff=512, vocab=512, mask_id=511)
    return make_context(shape, to_device(S.make_weights(shape, seed=3, round_to_bf16=True), torch.bfloat16), max_seqs=1, max_T=64, max_rows=64)


@pytest.mark.parametrize("M", [1, 16, 63, 64, 65, 96, 127, 128, 129])
@pytest.mark.parametrize("N,K", [(6144, 64), (6144, 320), (6144, 448), (8192, 1024), (8320, 704), (12288, 4096), (4096, 832), (6016, 512)])
def test_every_element(ctx, M, N, K):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = torch.randn(M, K, device="cuda", generator=g).to(torch.bfloat16)
    W = (torch.randn(2 * N, K, device="cuda", generator=g) * 0.05).to(torch.bfloat16)
    full = A.double() @ W.double().T
    gate, up = full[:, :N], full[:, N:]
    # one bf16 rounding of a float32 sum of K products, whose own error is below K^0.5 2^-24 of its terms' size
    slack = K ** 0.5 * 2.0 ** -22
    for got, want in ((ctx.gemm(A, W[:N]), gate), (ctx.gemm_swiglu(A, W), torch.nn.functional.silu(gate) * up)):
        bound = 2.0 ** -8 * want.abs() + slack * (1 + gate.abs() + up.abs())
        assert bool(((got.double() - want).abs() <= bound).all()), (M, N, K)


@pytest.mark.parametrize("M", [130, 160, 192, 193, 256, 257, 320, 321, 384, 385, 512, 513, 640, 641])
@pytest.mark.parametrize("N,K,kind", [(8192, 192, "swiglu"), (12288, 512, "swiglu"), (12288, 512, "store"), (8320, 1024, "store"),
                                      (4096, 4096, "residual"), (4096, 2048, "residual"), (1280, 6144, "residual")])
def test_every_element_of_more_rows(ctx, M, N, K, kind):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = torch.randn(M, K, device="cuda", generator=g).to(torch.bfloat16)
    W = (torch.randn(N * (2 if kind == "swiglu" else 1), K, device="cuda", generator=g) * 0.05).to(torch.bfloat16)
    R = torch.randn(M, N, device="cuda", generator=g).to(torch.bfloat16) if kind == "residual" else None
    full = A.double() @ W.double().T
    size = 1 + full.abs()
    if kind == "swiglu":
        got, want, size = ctx.gemm_swiglu(A, W), torch.nn.functional.silu(full[:, :N]) * full[:, N:], size[:, :N] + size[:, N:]
    else:
        got, want = ctx.gemm(A, W, residual=R), full + (R.double() if R is not None else 0)
    assert bool(((got.double() - want).abs() <= 2.0 ** -8 * want.abs() + K ** 0.5 * 2.0 ** -22 * size).all())


# rings of six stages with one, three and five of them to fill (128 x 64 store, 64 x 128 SwiGLU), an odd multiple of 64 columns, and
# the limits in columns and K between whole and divided launches
@pytest.mark.parametrize("M", [1, 64, 65, 128])
@pytest.mark.parametrize("N,K", [(12288, 64), (12288, 320), (9280, 192), (9280, 1088), (8320, 64), (8320, 320), (20480, 1024), (20480, 2048), (6144, 2112),
                                 (9216, 5120), (16384, 1024)])
def test_short_loops_and_limits(ctx, M, N, K):
    if N % 128 == 0:
        test_every_element(ctx, M, N, K)
        return
    g = torch.Generator(device="cuda").manual_seed(M + N + K)           # plain products take whole 128 columns
    A = torch.randn(M, K, device="cuda", generator=g).to(torch.bfloat16)
    W = (torch.randn(2 * N, K, device="cuda", generator=g) * 0.05).to(torch.bfloat16)
    full = A.double() @ W.double().T
    want, size = torch.nn.functional.silu(full[:, :N]) * full[:, N:], 1 + full[:, :N].abs() + full[:, N:].abs()
    assert bool(((ctx.gemm_swiglu(A, W).double() - want).abs() <= 2.0 ** -8 * want.abs() + K ** 0.5 * 2.0 ** -22 * size).all())


@pytest.mark.parametrize("M", [129, 192, 193, 256, 320, 321, 384, 385, 513, 576])
@pytest.mark.parametrize("N,K,kind", [(8192, 1024, "swiglu"), (8192, 1088, "swiglu"), (9216, 2048, "swiglu"), (9216, 4160, "swiglu"), (11008, 2112, "swiglu"),
                                      (16384, 3072, "swiglu"), (8192, 2048, "store"), (8192, 3072, "store"), (9216, 3072, "store"), (4096, 2048, "residual")])
def test_limits_of_more_rows(ctx, M, N, K, kind):
    test_every_element_of_more_rows(ctx, M, N, K, kind)


@pytest.mark.parametrize("M,N,K", [(64, 6144, 512), (128, 6144, 512), (128, 12288, 1024), (2, 8192, 2048), (384, 8192, 512), (256, 4096, 8192), (640, 4096, 4096)])
def test_equal_rows_stay_equal(ctx, M, N, K):
    g = torch.Generator(device="cuda").manual_seed(N)
    a = torch.randn(M // 2, K, device="cuda", generator=g).to(torch.bfloat16)
    W = torch.randn(2 * N, K, device="cuda", generator=g).to(torch.bfloat16)
    for out in (ctx.gemm(torch.cat([a, a]), W[:N]), ctx.gemm_swiglu(torch.cat([a, a]), W)):
        assert torch.equal(out[:M // 2], out[M // 2:])
