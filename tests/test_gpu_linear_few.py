"""Products of few tokens that make their own operands (packing, LayerNorm, the FFN core's partial sums): the feed-forward block and the
layer at the edges of that route's rule - one token, a last tile of 32 tokens with one in it, sizes whose workgroups make just one round
(256) and the next ones, every number of wavefronts that share a contraction (8, 4, 2, 1) with one and with several chunks each, K of 1024
and above it, one part and several - against the oracle.  Each case states how many wavefronts its products get (0: another kernel) and
asserts it of the rules.  Bounds: those of the blocks' fp16 hand-offs (FFN 4e-3 of the RMS; post-LN layer 2e-3, the stated gate; in a
pre-LN layer nothing renormalises, and a row is the block input plus an attention row of up to unit RMS with 6e-3 of it, the rows that see few
keys, plus an FFN row of about half of that with 4e-3: 4e-3 of an output of 1.3.  Launches apart differ from the oracle by the same
2.4e-3 and 2.2e-3 in the two cases of bf16)."""
import numpy as np
import pytest
import torch

from fsvd_testing import NORM, NORM_TWICE, NOTHING, PACK, PARTS, ffn_plan, linear_few_pays, linear_few_plan, rel_err
from oracle import fsvd_oracle as O
from paper_2508_01506_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _factors(rng, shapes, dt, tiled):
    from paper_2508_01506_amd import binding as fb
    tdt = torch.float16 if dt == "fp16" else torch.bfloat16
    host, dev = {}, {}
    for n, (i, o, r) in shapes.items():
        h = {"U": rng.standard_normal((i, r)) * i ** -0.5, "V": rng.standard_normal((r, o)) * r ** -0.5, "b": rng.standard_normal(o) * 0.02}
        host[n] = {k: W.round_to_storage(v, dt) for k, v in h.items()}
        up = {k: torch.from_numpy(np.ascontiguousarray(v)).to(device=DEV, dtype=tdt) for k, v in host[n].items()}
        f = fb.Factor(up["U"], up["V"], up["b"])
        dev[n] = f.with_tiled(True, True) if tiled else f
    return host, dev


def _kw(pays, T, K, *N):
    return linear_few_plan(T, K, *N) if pays else 0


@pytest.mark.parametrize("T,D,F,r1,r2,dt,tiled,kw_first,kw_last", [
    (1, 256, 512, 16, 48, "fp16", True, 0, 0),
    (33, 1024, 2048, 240, 80, "bf16", False, 8, 2),
    (257, 768, 3072, 384, 384, "fp16", True, 8, 8),
    (2048, 768, 3072, 192, 192, "fp16", True, 4, 1),     # last product: one wavefront per column tile, three chunks
    (2048, 512, 2048, 144, 112, "bf16", True, 4, 2),     # 256 workgroups of two wavefronts a column tile, and one tile of tokens more
    (2049, 512, 2048, 144, 112, "bf16", True, 4, 1),
    (1000, 1024, 1024, 1024, 1024, "fp16", False, 2, 2), # 256 workgroups, K = 1024, and the next
    (1025, 1024, 4096, 1024, 1024, "fp16", False, 1, 1),
    (8192, 256, 512, 256, 256, "fp16", True, 1, 1),      # 256 workgroups of one wavefront a column tile, and one more: another kernel
    (8193, 256, 512, 256, 256, "fp16", True, 0, 0),
    (96, 2048, 1024, 80, 80, "fp16", True, 0, 2),        # D above 1024
])
def test_ffn_block(T, D, F, r1, r2, dt, tiled, kw_first, kw_last, monkeypatch):
    from paper_2508_01506_amd import binding as fb
    monkeypatch.delenv("FSVD_FFN_CORE", raising=False)
    assert _kw(linear_few_pays(NOTHING, T, D), T, D, r1) == kw_first
    assert _kw(linear_few_pays(PARTS, T, D, r2), T, r2, D) == kw_last
    rng = np.random.default_rng(T + D)
    host, dev = _factors(rng, {"w1": (D, F, r1), "w2": (F, D, r2)}, dt, tiled)
    X = W.round_to_storage(rng.standard_normal((1, T, D)), dt)
    tdt = torch.float16 if dt == "fp16" else torch.bfloat16
    d = fb.make_desc(1, T, D, D // 64, F, tdt, torch.float32)
    x = torch.from_numpy(np.ascontiguousarray(X)).to(device=DEV, dtype=tdt)
    got = fb.fsvd_ffn(d, x, dev["w1"], dev["w2"]).cpu().numpy()
    rows = np.unique(np.concatenate([np.arange(min(T, 40)), np.arange(max(0, T - 40), T)]))
    ref = O.ffn(X[:, rows], host["w1"], host["w2"])
    err = rel_err(got[:, rows], ref)
    print("parts", ffn_plan(T, r1, r2, F, (tiled, int(dt == "bf16"))).fsplit, "err", err)
    assert np.isfinite(got).all() and err < 4e-3


@pytest.mark.parametrize("B,M,D,F,ra,rf,norm,mask,dt,tiled,kw_in,kw_first,kw_last", [
    (1, 1, 256, 512, 16, 16, "post_ln", "none", "fp16", True, 4, 0, 0),
    (1, 1, 1024, 512, 16, 112, "post_ln", "none", "fp16", True, 8, 8, 2),
    (3, 21, 512, 1024, 48, 80, "pre_ln", "causal", "bf16", False, 8, 8, 2),
    (2, 128, 768, 3072, 192, 384, "post_ln", "padding", "fp16", True, 8, 8, 8),
    (5, 97, 1024, 1024, 96, 1024, "post_ln", "none", "bf16", True, 8, 4, 4),
    (1, 1100, 256, 1024, 64, 240, "pre_ln", "causal", "fp16", True, 4, 4, 4),
    (4, 256, 512, 2048, 128, 128, "post_ln", "none", "fp16", False, 4, 8, 2),
    (4, 256, 1024, 1024, 64, 1024, "pre_ln", "causal", "fp16", True, 8, 2, 2),     # 256 workgroups, and one tile of tokens more
    (5, 205, 1024, 1024, 64, 1024, "pre_ln", "causal", "fp16", True, 8, 1, 1),
    (1, 2331, 448, 512, 16, 688, "post_ln", "none", "fp16", False, 4, 1, 1),       # LayerNorm in the operands, and of the residual from its statistics
    (1, 2331, 384, 512, 16, 688, "pre_ln", "causal", "bf16", True, 4, 1, 2),
    (2, 300, 256, 512, 32, 48, "pre_ln", "none", "fp16", False, 0, 0, 0),          # where launches apart are faster
])
def test_layer(B, M, D, F, ra, rf, norm, mask, dt, tiled, kw_in, kw_first, kw_last):
    from paper_2508_01506_amd import binding as fb
    T, post = B * M, norm == "post_ln"
    assert _kw(linear_few_pays(PACK if post else NORM, T, D), T, D, ra, ra, ra) == kw_in
    pays = linear_few_pays(NORM_TWICE if post else NORM, T, D, rf) and linear_few_plan(T, D, rf) > 0 and linear_few_plan(T, rf, D) > 0
    assert (_kw(pays, T, D, rf), _kw(pays, T, rf, D)) == (kw_first, kw_last)
    rng = np.random.default_rng(B * M + D)
    shapes = {n: (D, D, ra) for n in "qkvo"}
    shapes.update(w1=(D, F, rf), w2=(F, D, rf))
    host, dev = _factors(rng, shapes, dt, tiled)
    tdt = torch.float16 if dt == "fp16" else torch.bfloat16
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(device=DEV, dtype=tdt)
    X = W.round_to_storage(rng.standard_normal((B, M, D)), dt)
    ln = [W.round_to_storage(1 + 0.02 * rng.standard_normal(D), dt) if i % 2 == 0 else W.round_to_storage(0.02 * rng.standard_normal(D), dt) for i in range(4)]
    lens = np.array([M if b == 0 else max(1, M - 7 * b) for b in range(B)], np.int32) if mask == "padding" else None
    H = D // 64
    dlens = None if lens is None else torch.from_numpy(lens).to(DEV)      # (the descriptor holds its address only)
    d = fb.make_desc(B, M, D, H, F, tdt, torch.float32, mask == "causal", dlens, 0.0, "gelu_erf", norm)
    g = [up(x) for x in ln]
    got = fb.fsvd_layer(d, up(X), *(dev[n] for n in "qkvo"), g[0], g[1], dev["w1"], dev["w2"], g[2], g[3]).cpu().numpy()
    ref = O.layer(X, host["q"], host["k"], host["v"], host["o"], (ln[0], ln[1]), host["w1"], host["w2"], (ln[2], ln[3]), H, norm, mask == "causal", lens)
    err = rel_err(got, ref)
    print("err", err)
    assert np.isfinite(got).all() and err < (2e-3 if post else 4e-3)
