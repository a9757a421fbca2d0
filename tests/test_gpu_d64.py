"""bf16 attention with D = 64, whose tiles go straight into LDS in two rows per 256
bytes: against fp64 at the edges of the 64-key tiles and the row tiles, with and
without a row list, and the log-sum-exp."""
import pytest
import torch

from paper_2605_07443_amd import ops

DEV = "cuda:0"


@pytest.mark.gpu
@pytest.mark.parametrize("B,N,Hq,Hkv,R", [
    (1, 1, 1, 1, 1), (2, 63, 4, 4, 63), (1, 64, 8, 2, 64), (3, 65, 8, 8, 9), (1, 127, 128, 1, 3), (1, 128, 2, 1, 128),
    (2, 129, 6, 3, 129), (1, 321, 12, 12, 130)])
def test_d64_against_fp64(B, N, Hq, Hkv, R):
    print(f"[d64] {B} {N} {Hq} {Hkv} {R}", flush=True)
    g = torch.Generator().manual_seed(N)
    q, k, v = (torch.randn((B, N, h, 64), generator=g).to(torch.bfloat16) for h in (Hq, Hkv, Hkv))
    rows = None if R == N else torch.stack([torch.randperm(N, generator=g)[:R].sort().values for _ in range(B)]).int()
    pos = torch.arange(N).expand(B, N) if rows is None else rows.long()
    dq, dk, dv = q.to(DEV), k.to(DEV), v.to(DEV)
    dr = None if rows is None else rows.to(DEV)
    out = ops.selective_attention(dq, dk, dv, dr).cpu().double()
    out_l, lse = (t.cpu().double() for t in ops.selective_attention_lse(dq, dk, dv, dr))
    G = Hq // Hkv
    qs = torch.gather(q.double(), 1, pos[:, :, None, None].expand(B, R, Hq, 64)).permute(0, 2, 1, 3)
    kk, vv = (t.double().repeat_interleave(G, 2).permute(0, 2, 1, 3) for t in (k, v))
    s = (qs @ kk.transpose(2, 3)) / 8
    s.masked_fill_(torch.arange(N)[None, None, None] > pos[:, None, :, None], float("-inf"))
    p = torch.softmax(s, -1)
    want, scale = (p @ vv).permute(0, 2, 1, 3), (p @ vv.abs()).permute(0, 2, 1, 3)
    # P and the output are rounded to bf16 (2^-9 of each addend, of the row sum
    # that divides them, and of the result) and P's reference maximum adds fp32 rounding
    for o in (out, out_l):
        assert ((o - want).abs() <= 3.2 * 2.0 ** -9 * scale + 1e-6).all()
    # scores: 64 fp32 additions whose absolute terms sum to t = sum |q k| / 8; the
    # log-sum-exp moves by no more than the worst score, plus exp2, the sum and log2
    t = ((qs.abs() @ kk.abs().transpose(2, 3)) / 8).amax(-1).permute(0, 2, 1)
    assert ((lse - torch.logsumexp(s, -1).permute(0, 2, 1)).abs() <= 64 * 2.0 ** -24 * t + 1e-5).all()
