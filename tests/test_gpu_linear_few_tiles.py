"""Products with few output tiles, whose contraction the wavefronts of a workgroup split: C = A W + bias + residual against
float64 at the edges of tiles (32 or 64 tokens, 32 or 64 columns), chunks (64) and wavefronts (8 chunks a round).

Operands are exact in fp16 (bf16 is widened exactly), sums are fp32 over K terms of magnitude 1 / sqrt(K): 1e-5 of the RMS;
fp32 output, so nothing else is rounded."""
import numpy as np
import pytest
import torch

from fsvd_testing import rel_err

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("T,K,N,dt,tiled", [
    (1, 16, 16, "fp16", True), (1, 4096, 1040, "bf16", True), (31, 80, 48, "bf16", False), (32, 2112, 8208, "fp16", True),
    (33, 64, 64, "fp16", False), (64, 528, 144, "bf16", True), (65, 2064, 336, "fp16", True), (300, 1040, 80, "bf16", False),
    (1000, 192, 1024, "fp16", True),
])
def test_linear_split_contraction(T, K, N, dt, tiled):
    from paper_2508_01506_amd import binding as fb
    g = torch.Generator().manual_seed(T + K + N)
    tdt = torch.float16 if dt == "fp16" else torch.bfloat16
    A = torch.randn(T, K, generator=g).to(tdt)
    W = (torch.randn(K, N, generator=g) / K ** 0.5).to(tdt)
    b = torch.randn(N, generator=g).to(tdt)
    R = torch.randn(T, N, generator=g)
    ref = A.double().numpy() @ W.to(torch.float16).double().numpy() + b.double().numpy() + R.double().numpy()
    a, w, bb, rr = A.to(DEV), W.to(DEV), b.to(DEV), R.to(DEV)
    if tiled:
        run = lambda: fb.fsvd_linear_tiled(a, fb.fsvd_pack_tiled(w), N, bb, rr, torch.float32)
    else:
        run = lambda: fb.fsvd_linear(a, w, bb, rr, torch.float32)
    got = run()
    assert rel_err(got.cpu().numpy(), ref) < 1e-5
    assert torch.equal(got, run())
