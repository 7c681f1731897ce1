"""Fragment-major projections whose contraction two sets of wavefronts share (between a quarter and one 256 x 64 tile per compute unit, at
least six 64-wide chunks): an even and an odd number of chunks - with an odd one the second set's last step lies past the end and must
add nothing -, ragged tokens and columns, both weight layouts and types, against float64.  Every case asserts that the rules of the
dispatch send it to this kernel.

Tolerance: the feed-forward block rounds four tensors to fp16 on the way (the normalised input, P1, the hidden value, Z), each with a
relative RMS error of 2^-11 / sqrt(3); in quadrature 5.6e-4, and the largest of 10^6 outputs lies about 5 sigma out: 2.8e-3 of its row's
RMS (with few ranks behind the hidden value, 32, rows differ in scale).  The attention block of sequences of one token rounds three (P_v,
V, T_o): 4.9e-4, and the largest of 4 10^6 outputs 5.2 sigma out: 2.6e-3, held to the same bound."""
import ctypes as C

import numpy as np
import pytest
import torch

from fsvd_testing import linear_few_plan, row_err
from oracle import fsvd_oracle as O

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


class Group(C.Structure):
    _fields_ = [("W", C.c_void_p), ("bias", C.c_void_p), ("C", C.c_void_p), ("N", C.c_int), ("ldw", C.c_int), ("ldc", C.c_int),
                ("A", C.c_void_p), ("K", C.c_int), ("scale", C.c_float), ("v_tiles", C.c_int), ("C2", C.c_void_p)]


class Args(C.Structure):
    _fields_ = [("A", C.c_void_p), ("a_layout", C.c_int), ("lda", C.c_int), ("a_dt", C.c_int), ("T", C.c_int), ("K", C.c_int),
                ("w_dt", C.c_int), ("w_tiled", C.c_int), ("c_layout", C.c_int), ("c_dt", C.c_int), ("R", C.c_void_p),
                ("ldr", C.c_int), ("r_dt", C.c_int), ("ngroups", C.c_int), ("g", Group * 3)]


def shared(T, K, *N):
    """Whether a fragment-major [T, K] x [K, N..] product goes to the kernel under test (host functions of the library)."""
    from paper_2508_01506_amd import binding as fb
    a = Args(a_layout=1, c_layout=1, T=T, K=K, ngroups=len(N))
    for i, n in enumerate(N):
        a.g[i].N = n
    kwave, two = (getattr(fb.lib(), f"_ZN4fsvd{n}ERKNS_10LinearArgsE") for n in ("17linear_kwave_pays", "15linear_two_sets"))
    kwave.restype = two.restype = C.c_bool
    return two(C.byref(a)) and not kwave(C.byref(a))


def _f16(t):                   # stored values as the kernels use them
    return t.to(torch.float16).double() if t.dtype == torch.bfloat16 else t.double()


@pytest.mark.parametrize("T,D,r,dt,tiled", [
    (8200, 384, 272, "fp16", True),        # six chunks, the fewest; a last row tile of eight rows, a column tile of 16
    (8200, 448, 272, "bf16", False),       # seven
    (8200, 448, 400, "fp16", True),
    (8200, 512, 272, "fp16", True),
    (2331, 1088, 688, "bf16", True),       # 17, above the widths of the products that make their own operands
])
def test_projection_shared_by_two_sets(T, D, r, dt, tiled):
    from paper_2508_01506_amd import binding as fb
    assert shared(T, D, r) and linear_few_plan(T, D, r) == 0
    g = torch.Generator().manual_seed(T + D + r)
    tdt = torch.float16 if dt == "fp16" else torch.bfloat16
    n = lambda *s, std=1.0: (torch.randn(*s, generator=g) * std).to(tdt)
    F = 64
    X, U1, V1, b1 = n(T, D), n(D, r, std=D ** -0.5), n(r, F, std=r ** -0.5), n(F)
    U2, V2, b2 = n(F, 32, std=F ** -0.5), n(32, D, std=32 ** -0.5), n(D)
    f = lambda *a: fb.Factor(*(x.to(DEV) for x in a))
    w1, w2 = f(U1, V1, b1), f(U2, V2, b2)
    if tiled:
        w1, w2 = w1.with_tiled(True, True), w2.with_tiled(True, True)
    # the fragment-major input that selects this kernel exists inside a layer only: a pre-LN layer with the attention at zero
    z = f(torch.zeros(D, 16, dtype=tdt), torch.zeros(16, D, dtype=tdt), torch.zeros(D, dtype=tdt))
    if tiled:
        z = z.with_tiled(True, True)
    one, zero = torch.ones(D, dtype=tdt, device=DEV), torch.zeros(D, dtype=tdt, device=DEV)
    d = fb.make_desc(1, T, D, D // 64, F, tdt, torch.float32, norm="pre_ln")
    call = lambda: fb.fsvd_layer(d, X.to(DEV).reshape(1, T, D), z, z, z, z, one, zero, w1, w2, one, zero)
    got = call()
    assert torch.equal(got, call())
    x = X.double().numpy()
    ln = (x - x.mean(1, keepdims=True)) / np.sqrt(x.var(1, keepdims=True) + 1e-5)
    dd = lambda t: _f16(t).numpy()
    hidden = O.activation(ln @ dd(U1) @ dd(V1) + b1.double().numpy(), "gelu_erf")
    want = hidden @ dd(U2) @ dd(V2) + b2.double().numpy()
    have = got[0].double().cpu().numpy() - x
    err = row_err(have, want)
    assert err < 2.8e-3, err


def _attention(B, M, D, r, r_o, dt, tiled, seed):
    """Input, factors of v and o, and the call of an attention block with even attention (q and k are zero): what remains is products."""
    from paper_2508_01506_amd import binding as fb
    g = torch.Generator().manual_seed(seed)
    tdt = torch.float16 if dt == "fp16" else torch.bfloat16
    n = lambda *s, std=1.0: (torch.randn(*s, generator=g) * std).to(tdt)
    X = n(B, M, D)
    v, o = ([n(D, x, std=D ** -0.5), n(x, D, std=x ** -0.5), n(D, std=0.1)] for x in (r, r_o))
    z = [torch.zeros_like(t) for t in v]

    def run():
        q, k, vv, oo = (fb.Factor(*(t.to(DEV) for t in f)).with_tiled(tiled, tiled) for f in (z, z, v, o))
        return fb.fsvd_attention(fb.make_desc(B, M, D, D // 64, 16, tdt, torch.float32), X.to(DEV), q, k, vv, oo)
    return X, v, o, run


@pytest.mark.parametrize("T,D,r,r_o,dt,tiled", [
    (5500, 384, 16, 192, "fp16", True),    # six chunks
    (2331, 448, 16, 688, "fp16", True),    # seven
    (2331, 448, 16, 688, "bf16", False),
    (6000, 576, 64, 192, "bf16", True),    # nine
    (6000, 576, 64, 192, "fp16", False),
    (4100, 960, 64, 320, "fp16", True),    # fifteen
    (2304, 1600, 512, 512, "fp16", True),  # twenty-five, and the three projections into rank space take the same kernel
    (2304, 1600, 512, 512, "bf16", True),
    (2304, 1600, 512, 512, "bf16", False),
])
def test_context_projection_shared_by_two_sets(T, D, r, r_o, dt, tiled):
    assert shared(T, D, r_o) and (r < 512 or shared(T, D, r, r, r))
    X, v, o, run = _attention(T, 1, D, r, r_o, dt, tiled, T + D + r_o)       # sequences of one token: the context is V
    got = run()
    assert torch.equal(got, run())
    want = (_f16(X[:, 0]) @ _f16(v[0]) @ _f16(v[1]) + v[2].double()) @ _f16(o[0]) @ _f16(o[1]) + o[2].double()
    err = row_err(got[:, 0].double().cpu().numpy(), want.numpy())
    assert err < 2.8e-3, err


@pytest.mark.parametrize("tiled", [True, False])
def test_infinite_activation_in_the_last_chunk(tiled):
    """A step past the end multiplies zeros by zeros: an infinite context value in the last chunk stays an infinity (0 x inf would be NaN)."""
    B, M, D, r_o = 47, 128, 576, 192
    assert shared(B * M, D, r_o)
    X, v, o, run = _attention(B, M, D, 16, r_o, "fp16", tiled, 7)
    v[0][0, :], v[0][0, 0] = 0, 1
    v[1][0, :], v[1][0, D - 1] = 0, 4
    X[3, 5, :], X[3, 5, 0] = 0, 6e4              # P_v 6e4, V 2.4e5 in the last column: infinite in fp16 there, finite everywhere else
    o[0][:], o[1][:] = o[0].abs() + 2.0 ** -10, o[1].abs() + 2.0 ** -10
    got = run()
    assert bool((got[3] == float("inf")).all()) and bool(torch.isfinite(torch.cat([got[:3], got[4:]])).all())
