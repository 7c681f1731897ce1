"""The decoding step's products in parts and its merge, at the edges of their rules: one sequence (four groups of threads merge) to 64, and 65
(the general projections); a last tile of 32 tokens with one in it; ranks that end inside a chunk of 64, a tile of 32 columns or a part;
both head widths, row-major factors and images.  Bound: that of the attention block's fp16 hand-offs (6e-3 of a sequence's RMS, or the
same absolute noise, 1e-3, where an average over many keys is small)."""
import numpy as np
import pytest
import torch

from fsvd_testing import rel_err
from oracle import fsvd_oracle as O
from paper_2508_01506_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B,D,H,ranks,t_max,dt,tiled", [
    (1, 4096, 32, (1024, 1024, 1024, 1024), 1100, "bf16", True),     # 4 and 8 parts; 32 parts of the keys
    (1, 256, 4, (16, 64, 32, 16), 40, "fp16", False),
    (3, 512, 8, (80, 128, 96, 144), 300, "fp16", True),
    (7, 512, 4, (336, 192, 352, 208), 90, "bf16", False),
    (8, 1280, 20, (272, 320, 288, 1008), 200, "fp16", True),         # 32 columns per workgroup from 8 sequences on
    (17, 768, 12, (256, 256, 256, 256), 130, "fp16", False),
    (33, 512, 4, (1024, 64, 1024, 48), 70, "bf16", True),
    (64, 256, 2, (48, 64, 32, 16), 50, "fp16", False),
    (65, 256, 4, (48, 64, 64, 16), 50, "fp16", True),
    (2, 2048, 16, (1040, 64, 64, 1040), 33, "fp16", True),           # ranks of q and of the output above 1024
])
def test_step(B, D, H, ranks, t_max, dt, tiled):
    from paper_2508_01506_amd import binding as fb
    rng = np.random.default_rng(B + D)
    tdt = torch.float16 if dt == "fp16" else torch.bfloat16
    store = lambda a: W.round_to_storage(a, dt)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(device=DEV, dtype=tdt)
    fac, dev = {}, {}
    for n, r in zip("qkvo", ranks):
        fac[n] = {"U": store(rng.standard_normal((D, r)) * D ** -0.5), "V": store(rng.standard_normal((r, D)) * r ** -0.5),
                  "b": store(rng.standard_normal(D) * 0.02)}
        f = fb.Factor(up(fac[n]["U"]), up(fac[n]["V"]), up(fac[n]["b"]))
        dev[n] = f.with_tiled(u=True, v=n in "qo") if tiled else f
    x = store(rng.standard_normal((B, D)))
    Pk, Pv = (W.round_to_storage(rng.standard_normal((B, t_max, r)), "fp16") for r in ranks[1:3])
    lens = rng.integers(0, t_max, B).astype(np.int32)
    lens[-1] = t_max - 1
    if B > 1:
        lens[0] = 0
    kc, vc = fb.fsvd_decode_new_caches(B, t_max, ranks[1], ranks[2], DEV)
    zero = torch.zeros(B, dtype=torch.int32, device=DEV)
    for which, (c, P) in enumerate(((kc, Pk), (vc, Pv))):
        fb.fsvd_decode_cache_write(c, which, t_max, torch.from_numpy(np.ascontiguousarray(P)).to(DEV, torch.float16), zero)
    d = fb.make_desc(B, t_max, D, H, 16, tdt, torch.float32)
    got = fb.fsvd_decode_attention(d, up(x), dev["q"], dev["k"], dev["v"], dev["o"], kc, vc, torch.from_numpy(lens).to(DEV)).cpu().numpy()
    ref, pk, pv = O.decode_attention(x, Pk, Pv, lens, fac["q"], fac["k"], fac["v"], fac["o"], H)
    for b in range(B):
        rms = float(np.sqrt(np.mean(np.asarray(ref[b]) ** 2)))
        assert rel_err(got[b], ref[b]) < max(6e-3, 1e-3 / rms), (b, lens[b])
    # the new rows of the caches: one rounding to fp16 of a 32-bit sum (2^-11 of the value, and 1e-5 for the sum)
    for c, new, which in ((kc, pk, 0), (vc, pv, 1)):
        r = ranks[1 + which]
        want = fb.fsvd_decode_new_caches(B, t_max, ranks[1], ranks[2], DEV)[which]
        fb.fsvd_decode_cache_write(want, which, t_max, torch.from_numpy(np.ascontiguousarray(Pk if which == 0 else Pv)).to(DEV, torch.float16), zero)
        fb.fsvd_decode_cache_write(want, which, t_max, torch.from_numpy(np.asarray(new).reshape(B, 1, r)).to(DEV, torch.float16), torch.from_numpy(lens).to(DEV))
        a, b = c.view(torch.float16).float(), want.view(torch.float16).float()
        assert bool(((a - b).abs() <= 2.0 ** -10 * b.abs() + 2e-5).all()), which
