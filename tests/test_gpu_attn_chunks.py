"""The attention core that rebuilds its tiles from the ranks, where its loops over 64-rank chunks can go wrong: one chunk, odd and even
numbers of them, ranks of k and v that end in different chunks (the shorter one's requests past its end must count as zeros), ranks that
are no multiple of a chunk, row-major weights (whose rows past the rank are cut by the resource) and prepacked ones (whose are zeros in the
image), numbers of heads that do and do not divide over the XCDs.

Against float64 on the same fp16 operands each row is held to 6e-3 of its own RMS: Q, K, V, the probabilities and the context are rounded
to fp16 (2^-11 each, of values up to about four times the RMS), which is the bound of the attention block elsewhere."""
import pytest
import torch

from fsvd_testing import row_err

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("B,M,H,r", [(1, 1, 1, (16, 16, 16)), (2, 33, 4, (64, 128, 16)), (3, 200, 3, (80, 48, 208)),
                                     (2, 257, 8, (192, 192, 64)), (1, 512, 8, (256, 320, 256)), (2, 545, 2, (384, 64, 144))])
def test_attention_core_over_rank_chunks(B, M, H, r, dh):
    from paper_2508_01506_amd import binding as fb
    D, T = H * dh, B * M
    g = torch.Generator().manual_seed(M + dh)
    n = lambda *s, std=1.0: (torch.randn(*s, generator=g) * std).to(device=DEV, dtype=torch.float16)
    fac = [fb.Factor(n(D, rk, std=D ** -0.5), n(rk, D, std=rk ** -0.5), n(D, std=0.1)) for rk in r]
    P = [n(T, rk) for rk in r]
    Pd = [fb.fsvd_pack_fm(p) for p in P]
    d = fb.make_desc(B, M, D, H, 16, torch.float16, torch.float32, M % 2 == 0, None, 0.0, "gelu_erf", "post_ln")
    core = lambda f: fb.fsvd_unpack_fm(fb.fsvd_attention_core(d, *Pd, *f), T, D)
    row, tiled = core(fac), core([f.with_tiled() for f in fac])
    assert torch.equal(row, tiled)
    heads = [(p.double() @ f.V.double() + f.b.double()).reshape(B, M, H, dh).transpose(1, 2).cpu() for p, f in zip(P, fac)]
    s = heads[0] @ heads[1].transpose(-1, -2).contiguous() * dh ** -0.5
    if M % 2 == 0:
        s = s.masked_fill(torch.ones(M, M).triu(1).bool(), float("-inf"))
    ref = (s.softmax(-1) @ heads[2]).transpose(1, 2).reshape(T, D)
    assert row_err(row.double().cpu().numpy(), ref.numpy()) < 6e-3
