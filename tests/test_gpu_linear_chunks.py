"""Products whose loops request operands past the end of the contraction: one 64-wide chunk, odd and even numbers of them and a ragged last one,
both weight layouts, every form of the activations, narrow and wide tiles, one set of wavefronts (two: test_gpu_linear_two_sets.py).

Row-major output: operands exact in fp16 (fp32 activations are rounded to it first), fp32 sums of K terms of 1 / sqrt(K): 1e-5 of the RMS.
Fragment-major: the attention block of sequences of one token, three roundings to fp16 (P_v, V, T_o) of 2^-11 / sqrt 3 each: 4.9e-4, the
largest of 4 10^6 outputs 5.2 sigma out: 2.6e-3 of its row's RMS, held to 2.8e-3; few ranks behind T_o make rows differ in scale.  The fused
LayerNorm: the stated gate of a post-LN layer, 2e-3."""
import ctypes as C

import numpy as np
import pytest
import torch

from fsvd_testing import rel_err, row_err
from oracle import fsvd_oracle as O
from paper_2508_01506_amd import workloads as W
from test_gpu_linear_two_sets import _attention, _f16, shared

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("T,K,N", [
    (9000, 16, 256), (9000, 64, 272), (9000, 128, 256), (9000, 192, 272), (9000, 1040, 144),         # narrow tiles
    (17000, 64, 1024), (17000, 192, 1040), (17000, 256, 1024), (2100, 2112, 4112),                  # wide ones, the last by its long contraction
])
@pytest.mark.parametrize("adt", [torch.float16, torch.bfloat16, torch.float32])
@pytest.mark.parametrize("wdt,tiled", [(torch.float16, False), (torch.bfloat16, False), (torch.bfloat16, True)])
def test_row_major(T, K, N, adt, wdt, tiled):
    from paper_2508_01506_amd import binding as fb
    g = torch.Generator(device=DEV).manual_seed(T + K + N)
    n = lambda *s: torch.randn(*s, generator=g, device=DEV)
    a, w, b = n(T, K).to(adt), (n(K, N) / K ** 0.5).to(wdt), n(N).to(wdt)
    ref = a.half().double() @ w.half().double() + b.double()
    got = (fb.fsvd_linear_tiled(a, fb.fsvd_pack_tiled(w), N, b, None, torch.float32) if tiled else
           fb.fsvd_linear(a, w, b, None, torch.float32))
    assert rel_err(got.cpu().numpy(), ref.cpu().numpy()) < 1e-5


@pytest.mark.parametrize("T,D,r_o", [
    (17000, 64, 64), (17000, 128, 64), (6000, 192, 192), (6000, 320, 192), (9000, 448, 512), (9000, 512, 512),
    (17000, 128, 1040), (17000, 192, 1040),                                                         # wide tiles
])
@pytest.mark.parametrize("dt,tiled", [("fp16", True), ("bf16", False)])
def test_fragment_major(T, D, r_o, dt, tiled):
    assert not shared(T, D, r_o)
    X, v, o, run = _attention(T, 1, D, 64, r_o, dt, tiled, T + D + r_o)
    want = (_f16(X[:, 0]) @ _f16(v[0]) @ _f16(v[1]) + v[2].double()) @ _f16(o[0]) @ _f16(o[1]) + o[2].double()
    assert row_err(run()[:, 0].double().cpu().numpy(), want.numpy()) < 2.8e-3


@pytest.mark.parametrize("D,r", [(256, 16), (512, 64), (768, 128), (1024, 144), (256, 320), (512, 448)])
def test_fused_layernorm(D, r):
    from paper_2508_01506_amd import binding as fb
    B, M = 60, 35                                          # 2100 tokens: both of the layer's LayerNorms are fused
    supported = fb.lib()._ZN4fsvd19linear_ln_supportedEi
    supported.restype = C.c_bool
    assert supported(D) and B * M >= 1024 + 2 * r
    rng = np.random.default_rng(D + r)
    store = lambda a: W.round_to_storage(a, "fp16")
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).half().to(DEV)
    F, host, dev = 512, {}, {}
    for n, (i, o, x) in {**{n: (D, D, 16) for n in "qkv"}, "o": (D, D, r), "w1": (D, F, 64), "w2": (F, D, r)}.items():
        h = host[n] = {"U": store(rng.standard_normal((i, x)) * i ** -0.5), "V": store(rng.standard_normal((x, o)) * x ** -0.5),
                       "b": store(rng.standard_normal(o) * 0.02)}
        dev[n] = fb.Factor(up(h["U"]), up(h["V"]), up(h["b"])).with_tiled(True, True)
    X = store(rng.standard_normal((B, M, D)))
    ln = [store((1 if i % 2 == 0 else 0) + 0.02 * rng.standard_normal(D)) for i in range(4)]
    g = [up(x) for x in ln]
    d = fb.make_desc(B, M, D, D // 64, F, torch.float16, torch.float32, norm="post_ln")
    got = fb.fsvd_layer(d, up(X), *(dev[n] for n in "qkvo"), g[0], g[1], dev["w1"], dev["w2"], g[2], g[3]).cpu().numpy()
    ref = O.layer(X, *(host[n] for n in "qkvo"), (ln[0], ln[1]), host["w1"], host["w2"], (ln[2], ln[3]), D // 64, "post_ln", False, None)
    assert rel_err(got, ref) < 2e-3
