"""Merging the parts of a pass over the cache (fsvd_decode_attention_core: one workgroup per head and sequence, 8 ranks per thread): the three
forms that request up to 4, up to 8 and 16 parts at once (with more than 16 a second round), at the part counts where they change; one
wavefront (up to 512 ranks) or two; a rank that ends inside one; more than 32 parts' worth of keys; equal parts above 64 sequences, one part
each, empty sequences.  Probabilities and u pass through fp16: the attention block's bound, 6e-3 of the RMS."""
import numpy as np
import pytest
import torch

from fsvd_testing import rel_err
from oracle import fsvd_oracle as O

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

EDGES = [32 * n for n in (1, 4, 5, 8, 9, 16, 17, 32)] + [0]      # one part per tile of 32 keys: so few tiles that every one is a part


def parts_of(lens):
    """How many parts every sequence is split into (up to 64 sequences: by its tiles of 32 keys, as few tiles per part as fit)."""
    B = len(lens)
    nsplit = min(32, max(1, 256 // B))
    if B > 64:
        return [nsplit] * B
    nt, G = [(n + 31) // 32 for n in lens], B * nsplit
    at = lambda t: [min(32, max(1, -(-x // t))) for x in nt]
    tpw = max(1, -(-sum(nt) // (G - B)))
    most = [min(32, max(1, x)) for x in nt]
    for _ in range(8):
        if tpw == 1 or at(tpw) == most or sum(at(tpw - 1)) > G:
            break
        tpw -= 1
    return at(tpw)


@pytest.mark.parametrize("r_v,lens,parts", [
    (32, EDGES, {1, 4, 5, 8, 9, 16, 17, 32}),
    (512, EDGES, {1, 4, 5, 8, 9, 16, 17, 32}),
    (544, EDGES, {1, 4, 5, 8, 9, 16, 17, 32}),
    (1024, EDGES, {1, 4, 5, 8, 9, 16, 17, 32}),
    (480, [2000], {32}),
    (1024, [1100] + [0, 3] * 23, {1, 32}),                         # 47 sequences
    (992, [1 + 17 * i for i in range(64)], set(range(1, 8))),
    (1024, [40 * (i % 9) for i in range(80)], {3}),                # equal parts, some without keys
    (288, [33 + i for i in range(256)], {1}),
])
def test_merge(r_v, lens, parts):
    assert set(parts_of(lens)) == parts
    from paper_2508_01506_amd import binding as fb
    rng = np.random.default_rng(r_v + len(lens))
    B, H, D, r_k, t_max = len(lens), 6, 384, 64, max(lens)
    Pk, Pv = (rng.standard_normal((B, t_max, r)).astype(np.float16) for r in (r_k, r_v))
    Wq = (rng.standard_normal((B, H, r_k)) * 0.15).astype(np.float16)
    kc, vc = fb.fsvd_decode_new_caches(B, t_max, r_k, r_v, DEV)
    zero = torch.zeros(B, dtype=torch.int32, device=DEV)
    fb.fsvd_decode_cache_write(kc, 0, t_max, torch.from_numpy(Pk).to(DEV), zero)
    fb.fsvd_decode_cache_write(vc, 1, t_max, torch.from_numpy(Pv).to(DEV), zero)
    Wpad = np.zeros((B, 32, r_k), np.float16)
    Wpad[:, :H] = Wq
    Wfm = torch.cat([fb.fsvd_pack_fm(torch.from_numpy(Wpad[b]).to(DEV)) for b in range(B)])
    d = fb.make_desc(B, t_max, D, H, 16, torch.float16)
    n_keys = torch.tensor(lens, dtype=torch.int32, device=DEV)
    got = fb.fsvd_decode_attention_core(d, r_k, r_v, Wfm, kc, vc, n_keys).cpu().numpy()
    for b, n in enumerate(lens):
        if n == 0:
            assert not got[b].any(), b
            continue
        s = Pk[b, :n].astype(np.float64) @ Wq[b].astype(np.float64).T * np.log(2.0)
        assert rel_err(got[b], O.softmax_rows(s.T) @ Pv[b, :n].astype(np.float64)) < 6e-3, (b, n)


@pytest.mark.parametrize("B,D,H,r", [(1, 256, 2, (48, 64, 32, 16)), (5, 512, 8, (80, 128, 96, 144)), (47, 256, 4, (16, 192, 1024, 32))])
def test_step_stays_in_its_workspace(B, D, H, r):
    """A workspace of exactly the size asked for: the step reads and writes nothing behind it."""
    from paper_2508_01506_amd import binding as fb
    g = torch.Generator().manual_seed(B + D)
    n = lambda *s, std=1.0: (torch.randn(*s, generator=g) * std).half().to(DEV)
    t_max = 200
    q, k, v, o = (fb.Factor(n(D, x, std=D ** -0.5), n(x, D, std=x ** -0.5), n(D, std=0.02)) for x in r)
    d = fb.make_desc(B, t_max, D, H, 16, torch.float16)
    x, lens = n(B, D), torch.randint(0, t_max, (B,), generator=g, dtype=torch.int32).to(DEV)
    rows = [n(B, t_max, c) for c in (r[1], r[2])]
    need = fb.fsvd_decode_attention_workspace(d, *r)
    outs = []
    for fill in (0x00, 0x7f):                   # 0x7f7f is a NaN in fp16 and in fp32: what is behind must not matter either
        kc, vc = fb.fsvd_decode_new_caches(B, t_max, r[1], r[2], DEV)
        for which, c in enumerate((kc, vc)):
            fb.fsvd_decode_cache_write(c, which, t_max, rows[which], torch.zeros(B, dtype=torch.int32, device=DEV))
        buf = torch.full((need + 65536,), fill, dtype=torch.uint8, device=DEV)
        outs.append(fb.fsvd_decode_attention(d, x, q, k, v, o, kc, vc, lens, workspace=buf[:need]).clone())
        assert (buf[need:] == fill).all()
    assert torch.isfinite(outs[0]).all() and torch.equal(outs[0], outs[1])
