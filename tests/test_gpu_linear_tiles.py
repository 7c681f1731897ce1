"""Products with few output tiles at the sizes where their tile shape changes (32 x 32, 32 x 64, 64 x 64: the smallest that makes one
round over the 256 compute units) and at ragged last tiles, row-major and fragment-major output.

Row-major: operands exact in fp16, fp32 sums and output: 1e-5 of the RMS.  Fragment-major output exists inside a layer only: a pre-LN layer
with the attention at zero, the feed-forward factors chosen so that the first product decides.  P1 and the hidden value are
rounded to fp16 (2^-11 / sqrt 3 each, 4e-4 in quadrature, and the normalised input 2.8e-4): 4.9e-4 RMS, 5 sigma at 10^5 outputs: 2.5e-3."""
import numpy as np
import pytest
import torch

from fsvd_testing import NORM, linear_few_pays, rel_err
from oracle import fsvd_oracle as O

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("T,K,N", [
    (33, 192, 4096), (64, 1040, 4096),      # 2 x 128 smallest tiles: one round
    (65, 192, 4096), (70, 320, 2736),       # 3 x 128, 3 x 86: tiles of 32 x 64
    (97, 128, 4112),                        # 4 x 65 of those: tiles of 64 x 64
    (250, 2064, 1008), (256, 80, 2064),     # ragged columns in either
])
@pytest.mark.parametrize("tiled", [True, False])
def test_row_major_output(T, K, N, tiled):
    from paper_2508_01506_amd import binding as fb
    g = torch.Generator().manual_seed(T + K + N)
    A, W, b = torch.randn(T, K, generator=g).half(), (torch.randn(K, N, generator=g) / K ** 0.5).half(), torch.randn(N, generator=g).half()
    ref = A.double().numpy() @ W.double().numpy() + b.double().numpy()
    a, w, bb = A.to(DEV), W.to(DEV), b.to(DEV)
    run = lambda: (fb.fsvd_linear_tiled(a, fb.fsvd_pack_tiled(w), N, bb, None, torch.float32) if tiled else
                   fb.fsvd_linear(a, w, bb, None, torch.float32))
    assert rel_err(run().cpu().numpy(), ref) < 1e-5


@pytest.mark.parametrize("T,D,r", [
    (40, 128, 80), (200, 256, 48),          # a last chunk of 64 columns that is half or mostly padding
    (96, 192, 2704), (130, 192, 1616),      # 3 x 86 smallest tiles, 5 x 52: tiles of 32 x 64
])
@pytest.mark.parametrize("tiled", [True, False])
def test_fragment_major_output(T, D, r, tiled):
    from paper_2508_01506_amd import binding as fb
    assert not linear_few_pays(NORM, T, D, min(r, 128))      # the LayerNorm in a launch of its own, its fragment-major result to this kernel
    g = torch.Generator().manual_seed(T + D + r)
    n = lambda *s, std=1.0: (torch.randn(*s, generator=g) * std).half()
    F = 128
    X, U1, V1, b1, U2, V2, b2 = n(T, D), n(D, r, std=D ** -0.5), n(r, F, std=r ** -0.5), n(F), n(F, 128, std=F ** -0.5), n(128, D, std=128 ** -0.5), n(D)
    f = lambda *a: fb.Factor(*(x.to(DEV) for x in a)).with_tiled(tiled, tiled)
    z = f(torch.zeros(D, 16).half(), torch.zeros(16, D).half(), torch.zeros(D).half())
    one, zero = torch.ones(D).half().to(DEV), torch.zeros(D).half().to(DEV)
    d = fb.make_desc(1, T, D, D // 64, F, torch.float16, torch.float32, norm="pre_ln")
    need = fb.fsvd_layer_workspace(d, 16, 16, 16, 16, r, 128)
    ws = torch.full((need // 2,), float("nan"), dtype=torch.float16, device=DEV).view(torch.uint8)   # padding must be written, not found
    got = fb.fsvd_layer(d, X.to(DEV).reshape(1, T, D), z, z, z, z, one, zero, f(U1, V1, b1), f(U2, V2, b2), one, zero, workspace=ws)
    x = X.double().numpy()
    ln = (x - x.mean(1, keepdims=True)) / np.sqrt(x.var(1, keepdims=True) + 1e-5)
    a = lambda t: t.double().numpy()
    want = O.activation(ln @ a(U1) @ a(V1) + a(b1), "gelu_erf") @ a(U2) @ a(V2) + a(b2)
    assert rel_err(got[0].cpu().numpy() - x, want) < 2.5e-3
