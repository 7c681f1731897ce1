"""The rules that choose between two kernels are host code of the library: its internal functions, called without a GPU."""
import ctypes as C
import random

import pytest

from fsvd_testing import NORM, NORM_TWICE, NOTHING, PACK, PARTS, ffn_plan, linear_few_pays, rebuilds_once
from paper_2508_01506_amd import binding as fb

TILED, ROW_F16, ROW_BF16 = (True, 0), (False, 0), (False, 1)


# the kernel that measures faster, where it does so by at least 3 %: private weight streams or loader wavefronts
@pytest.mark.parametrize("T,r1,r2,F,weights,streams", [
    (24, 16, 16, 768, ROW_BF16, False), (3000, 64, 64, 2048, ROW_BF16, False), (6000, 64, 64, 768, ROW_BF16, False),
    (6000, 128, 128, 1536, ROW_BF16, False), (1536, 48, 48, 4096, ROW_BF16, False), (11538, 800, 800, 5120, ROW_BF16, False),
    (256, 384, 384, 3072, ROW_BF16, True), (2331, 688, 688, 8192, ROW_BF16, True), (4096, 2048, 2048, 16384, ROW_BF16, True),
    (8192, 768, 768, 3072, ROW_BF16, True), (1536, 64, 64, 4096, ROW_F16, False), (2331, 688, 688, 8192, ROW_F16, True),
    (24000, 768, 768, 3072, TILED, False), (20000, 768, 768, 4096, TILED, False), (6000, 1024, 1024, 8192, TILED, False),
    (256, 384, 384, 3072, TILED, True), (8192, 768, 768, 3072, TILED, True), (16384, 256, 256, 4096, TILED, True),
    (4096, 2048, 2048, 16384, TILED, True),
])
def test_ffn_core_takes_the_faster_kernel(T, r1, r2, F, weights, streams, monkeypatch):
    monkeypatch.delenv("FSVD_FFN_CORE", raising=False)
    assert (ffn_plan(T, r1, r2, F, weights).stream_tt > 0) == streams


# prepacked, small ranks: the counted cycles alone would take the loader wavefronts, which measure 1.15 to 1.6 times slower
@pytest.mark.parametrize("T,r1,r2,F,streams", [
    (10301, 128, 48, 9712, True), (32311, 80, 80, 6800, True), (24, 256, 256, 1072, True),
    (9960, 640, 640, 560, False), (13397, 864, 864, 576, False), (24597, 128, 640, 1088, False),          # and where these are faster
])
def test_ffn_core_small_ranks(T, r1, r2, F, streams, monkeypatch):
    monkeypatch.delenv("FSVD_FFN_CORE", raising=False)
    assert (ffn_plan(T, r1, r2, F, TILED).stream_tt > 0) == streams


def test_ffn_plans_fit_the_workspace(monkeypatch):
    """Whichever kernel is chosen or forced, its partial sums fit what the size query (which knows no weight layout) asked for."""
    room = fb.lib()._ZN4fsvd22ffn_core_partial_bytesEiiii
    room.restype, room.argtypes = C.c_size_t, [C.c_int] * 4
    rng = random.Random(5)
    for _ in range(1500):
        T = int(2 ** rng.uniform(0, 15))
        r1, r2 = (16 * max(1, int(2 ** rng.uniform(0, 7))) for _ in "12")
        F = 16 * max(1, int(2 ** rng.uniform(0, 10)))
        for force in ("", "wide", "tworole"):
            monkeypatch.setenv("FSVD_FFN_CORE", force)
            for weights in (TILED, ROW_F16, ROW_BF16):
                p = ffn_plan(T, r1, r2, F, weights)
                assert p.partial_bytes <= room(T, r1, r2, F) <= T * F, (T, r1, r2, F, force, weights)
                assert (p.partial_bytes > 0) == (p.fsplit > 1) and p.nslices * p.slice_w >= r2


# products that make their own operands, where they measure faster than launches apart (here) or by at least 1.5 % slower (not)
@pytest.mark.parametrize("use,T,D,rank,here", [
    (PACK, 256, 768, 0, True), (PACK, 8, 128, 0, True), (PACK, 8, 64, 0, False),
    (NORM, 128, 256, 64, False), (NORM, 20, 256, 32, False), (NORM, 176, 512, 96, True), (NORM, 1676, 512, 48, True), (NORM, 4096, 256, 32, True),
    (NORM_TWICE, 2, 256, 48, False), (NORM_TWICE, 48, 768, 16, False), (NORM_TWICE, 256, 768, 384, True), (NORM_TWICE, 3452, 256, 272, True),
    (NOTHING, 6, 256, 48, False), (NOTHING, 2, 768, 48, False), (NOTHING, 3320, 256, 368, True), (NOTHING, 2048, 768, 192, True),
    (PARTS, 512, 512, 32, False), (PARTS, 18, 256, 32, False), (PARTS, 2048, 768, 192, True), (PARTS, 1792, 768, 160, True),
])
def test_products_of_few_tokens(use, T, D, rank, here):
    assert linear_few_pays(use, T, D, rank) == here


# 128 columns per workgroup where that measures faster: a long contraction and enough tiles that are not mostly padding
@pytest.mark.parametrize("T,K,N,wide", [
    (4096, 4096, (3072,), True), (4096, 4096, (2048,), True), (7636, 2768, (1728,), True), (13127, 3840, (592,), True),
    (4096, 4096, (1024,), False), (16384, 1024, (768,), False), (8192, 768, (1152,), False), (32768, 1024, (1024,), True),
    (22398, 3312, (288,), False), (14166, 2528, (192, 192, 192), False), (5057, 3360, (1584,), False), (29817, 3344, (64, 64, 64), False),
])
def test_column_tiles(T, K, N, wide):
    f = fb.lib()._ZN4fsvd19linear_narrow_tilesElli
    f.restype, f.argtypes = C.c_bool, [C.c_long, C.c_long, C.c_int]
    tiles = lambda n: -(-T // 256) * sum(-(-x // n) for x in N)
    assert f(tiles(128), tiles(64), K) != wide


# the faster way, where it measures so by at least 3 % of the whole layer: K and V once, or once per block of queries
@pytest.mark.parametrize("B,M,D,H,causal,r,once", [
    (1, 4096, 4096, 32, True, 1024, True), (4, 8192, 768, 12, False, 256, True), (3, 777, 2048, 16, True, 336, True),
    (16, 600, 1024, 8, True, 512, True), (1, 768, 768, 12, False, 256, True), (6, 3000, 768, 12, False, 256, True),
    (3, 8192, 1024, 8, False, 128, True), (1, 257, 1024, 8, False, 512, True),
    (16, 1100, 768, 12, True, 64, False), (16, 600, 1024, 8, True, 64, False), (16, 513, 768, 12, True, 64, False),
    (4, 513, 768, 12, False, 16, False), (16, 257, 1024, 8, True, 256, False), (16, 513, 256, 4, True, 64, False),
    (16, 1024, 768, 12, True, 16, False),
    (16, 512, 768, 12, False, 1024, False), (16, 256, 1024, 8, False, 1024, False),      # one block of queries
    (1, 520, 4096, 32, True, 64, False),                                                 # no room for V's last tiles over P_q
])
def test_layer_rebuilds_once_where_that_is_faster(B, M, D, H, causal, r, once):
    assert rebuilds_once(B, M, D, H, causal, r, r, r) == once


def test_rebuilding_once_has_room():
    """Where it is chosen, K and V fit the fp32 residual stream, the last token tiles of V the space of P_q."""
    rng = random.Random(9)
    chosen = 0
    for _ in range(20000):
        dh = rng.choice((64, 128))
        H, B, M = rng.randint(1, 32), rng.randint(1, 16), int(2 ** rng.uniform(5, 13))
        D, rq, rk, rv = H * dh, *(16 * rng.randint(1, 64) for _ in "qkv")
        if not rebuilds_once(B, M, D, H, rng.random() < 0.5, rq, rk, rv):
            continue
        T, tiles = B * M, (B * M + 31) // 32
        v_tiles = (4 * T * D - fb.fsvd_fm_bytes(T, D)) // (64 * D)
        assert v_tiles > 0 and (tiles - v_tiles) * 64 * D <= fb.fsvd_fm_bytes(T, rq)
        chosen += 1
    assert chosen > 5000
