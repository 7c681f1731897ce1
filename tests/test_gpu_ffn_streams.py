"""The FFN core with wavefront-private weight streams (prepacked and row-major weights) at the sizes where its tiles, chunks and rank
groups end: Z = phi(P1 V_1 + b_1) U_2 against the plain definition in float64.

Tolerance, as for the FFN core elsewhere: P1 and the weights are exact in fp16, so the error is one rounding of the
activated hidden value (2^-11 relative, averaged over F terms) and one of Z itself; Z's largest values are about four times
its RMS, so half a unit in the last place of them is 4 * 2^-11 = 2.0e-3 of the RMS at worst; 2.5e-3 is the bound."""
import numpy as np
import pytest
import torch

from fsvd_testing import rel_err
from oracle import fsvd_oracle as O
from paper_2508_01506_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("T,r1,r2,F,dt,act,bias", [
    (1, 16, 16, 16, "fp16", "gelu_erf", True),            # the smallest of everything
    (33, 64, 64, 512, "bf16", "gelu_erf", True),          # one row past a token tile, exactly one chunk
    (65, 80, 144, 528, "fp16", "gelu_tanh", True),        # 16 features past a chunk, three rank groups
    (300, 512, 512, 1040, "fp16", "gelu_erf", False),     # P1 of 64 tokens just fits in LDS, no bias
    (300, 528, 272, 1040, "bf16", "relu", True),          # and just does not
    (97, 1280, 1040, 1552, "fp16", "gelu_erf", True),     # P1 of 32 tokens just fits, four groups per wavefront
    (97, 1296, 640, 1552, "bf16", "gelu_erf", True),      # and just does not: pieces, the last one a single chunk
    (40, 2048, 2064, 1024, "fp16", "gelu_erf", True),     # more groups than one workgroup holds
    (16500, 96, 208, 1536, "fp16", "gelu_erf", True),     # more than one round of 64-token workgroups
])
@pytest.mark.parametrize("tiled", [True, False])
def test_ffn_core_private_streams(T, r1, r2, F, dt, act, bias, tiled, monkeypatch):
    from paper_2508_01506_amd import binding as fb
    monkeypatch.setenv("FSVD_FFN_CORE", "wide")
    rng = np.random.default_rng(T + r1 + r2 + F)
    tdt = torch.float16 if dt == "fp16" else torch.bfloat16
    rnd = lambda a: W.round_to_storage(a.astype(np.float32), dt).astype(np.float64)
    V1, b1 = rnd(rng.standard_normal((r1, F)) / np.sqrt(r1)), rnd(0.3 * rng.standard_normal(F))
    U2 = rnd(rng.standard_normal((F, r2)) / np.sqrt(F))
    P1 = rng.standard_normal((T, r1)).astype(np.float16)
    up = lambda a: torch.from_numpy(np.asarray(a, dtype=np.float32)).to(device=DEV, dtype=tdt).contiguous()
    w1 = fb.Factor(up(np.zeros((128, r1))), up(V1), up(b1) if bias else None)
    w2 = fb.Factor(up(U2), up(np.zeros((r2, 128))), None)
    if tiled:
        w1, w2 = w1.with_tiled(v=True), w2.with_tiled(u=True)
    d = fb.make_desc(1, T, 128, 2, F, tdt, act=act)
    P1fm = fb.fsvd_pack_fm(torch.from_numpy(P1).to(DEV))
    run = lambda: fb.fsvd_unpack_fm(fb.fsvd_ffn_core(d, P1fm, w1, w2), T, r2, torch.float32).cpu().numpy()
    Z = run()
    rows = np.unique(np.concatenate([np.arange(min(T, 80)), np.arange(max(0, T - 80), T)]))
    ref = O.activation(P1[rows].astype(np.float64) @ V1 + (b1 if bias else 0.0), act) @ U2
    assert np.isfinite(Z).all()
    assert rel_err(Z[rows], ref) < 2.5e-3
    assert np.array_equal(Z, run())                        # sums are added in a fixed order
