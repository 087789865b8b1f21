"""The GEMM tile shapes with a ring of two stages (256 x 256, 192 x 256 and, for SwiGLU, 256 x 192) take the 64-k stages in pairs: the smallest
number of stages (only the first and the last pass), one pair in the loop, and odd numbers, which the first two run on another
schedule and the last leaves to another shape."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# one bf16 rounding of a float32 sum (2^-8 relative; the residual is added before it) and the float32 sum's own error
CHILD = r"""
import sys, torch
sys.path.insert(0, %r)
from paper_2601_12247_amd import binding as B
g = torch.Generator(device="cuda").manual_seed(5)
for K in (64, 128, 192, 256, 384, 448):
    for M, N in ((1, 256), (193, 512), (257, 256), (511, 768), (449, 384)):
        A = torch.randn(M, K, device="cuda", generator=g).to(torch.bfloat16)
        W = torch.randn(2 * N, K, device="cuda", generator=g).to(torch.bfloat16)
        R = torch.randn(M, N, device="cuda", generator=g).to(torch.bfloat16)
        full = A.double().cpu() @ W.double().cpu().T
        gate, up = full[:, :N], full[:, N:]
        for got, want, slack in ((B.gemm(A, W[:N].contiguous()), gate, 0), (B.gemm(A, W[:N].contiguous(), residual=R), gate + R.double().cpu(), 0),
                                 (B.gemm_swiglu(A, W), torch.nn.functional.silu(gate) * up, 1e-5)):
            bound = (2.0 ** -8 + slack) * want.abs() + 1e-6 * K ** 0.5 * (1 + slack * 1e5 * (gate.abs() + up.abs()))
            bad = ((got.double().cpu() - want).abs() > bound).sum().item()
            assert bad == 0, (M, N, K, bad)
print("ok")
""" % ROOT


@pytest.mark.parametrize("tile", ["0", "4", "10"])
def test_stage_counts(tile):
    env = dict(os.environ, PVF_GEMM_TILE=tile)
    r = subprocess.run([sys.executable, "-c", CHILD], capture_output=True, text=True, env=env, timeout=110)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stderr[-2000:]
