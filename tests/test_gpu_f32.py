"""fp32 attention, log-sum-exp and attention mass at the edges of their tiles
(16 query vectors, chunks of 64 or 32 keys over 8 waves, 32 keys of the mass),
against the same in fp64."""
import math

import pytest
import torch

from paper_2605_07443_amd import ops

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# values of size 1: fp32 dot products of 128 terms and sums of up to 1,100
# weights stay below 1e-5 absolute (eps 6e-8 times about sqrt(128) and the
# score's size in the exponent, about 5)
ATOL = 1e-5


def _ref(q, k, v, rows):
    B, N, Hq, D = q.shape
    G = Hq // k.shape[2]
    q, k, v = q.double(), k.double().repeat_interleave(G, 2), v.double().repeat_interleave(G, 2)
    out, lse = [], []
    for b in range(B):
        pos = torch.arange(N, device=q.device) if rows is None else rows[b].long()
        s = torch.einsum("rhd,nhd->hrn", q[b][pos], k[b]) / math.sqrt(D)
        s.masked_fill_(torch.arange(N, device=q.device)[None, None] > pos[None, :, None], -math.inf)
        lse.append(torch.logsumexp(s, -1).t())
        p = torch.softmax(s, -1)
        out.append(torch.einsum("hrn,nhd->rhd", p, v[b]))
    return torch.stack(out), torch.stack(lse)


def _inputs(B, N, Hq, Hkv, D, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    rn = lambda *s: torch.randn(s, generator=g, device=DEV)  # noqa: E731
    return rn(B, N, Hq, D), rn(B, N, Hkv, D), rn(B, N, Hkv, D)


@pytest.mark.parametrize("B,N,Hq,Hkv,D,R", [
    (1, 1, 1, 1, 64, 1), (2, 15, 3, 1, 64, 7), (1, 16, 8, 8, 64, 16), (1, 17, 2, 2, 128, 5),
    (2, 63, 12, 4, 64, 33), (1, 65, 5, 5, 128, 65), (1, 416, 8, 8, 64, 90), (2, 513, 8, 2, 64, 47),
    (1, 1100, 6, 2, 128, 101)])
def test_f32_attention_selected_and_full(B, N, Hq, Hkv, D, R):
    print(f"[f32 attention] {B} {N} {Hq} {Hkv} {D} {R}", flush=True)
    q, k, v = _inputs(B, N, Hq, Hkv, D, N + R)
    g = torch.Generator().manual_seed(N)
    rows = torch.stack([torch.randperm(N, generator=g)[:R].sort().values for _ in range(B)]).to(torch.int32).to(DEV)
    for r in (rows, None):
        out, lse = ops.selective_attention_lse(q, k, v, r)
        plain = ops.selective_attention(q, k, v, r)
        want, wl = _ref(q, k, v, r)
        torch.cuda.synchronize()
        assert torch.equal(out, plain)
        assert (out.double() - want).abs().max().item() <= ATOL
        assert (lse.double() - wl).abs().max().item() <= ATOL
    mass = ops.attention_mass(q, k, lse)
    G = Hq // Hkv
    s = torch.einsum("bphd,bnhd->bhpn", q.double(), k.double().repeat_interleave(G, 2)) / math.sqrt(D)
    w = torch.exp(s - wl.permute(0, 2, 1)[..., None])
    w = w.masked_fill(torch.arange(N, device=DEV)[None, :] > torch.arange(N, device=DEV)[:, None], 0.0)
    want = w.sum(2).view(B, Hkv, G, N).sum(2)
    torch.testing.assert_close(mass.double(), want, rtol=2e-5, atol=1e-6)


@pytest.mark.parametrize("N,D", [(70, 64), (40, 128)])
def test_f32_attention_ignores_values_of_later_keys(N, D):
    """An infinity or NaN in K or V reaches only the rows that see its key."""
    q, k, v = _inputs(1, N, 4, 2, D, 5)
    clean = ops.selective_attention(q, k, v)
    bad = N - 9
    for value in (math.nan, math.inf, -math.inf):
        k2, v2 = k.clone(), v.clone()
        k2[:, bad, :, 0] = value
        v2[:, bad] = value
        out = ops.selective_attention(q, k2, v2)
        torch.cuda.synchronize()
        assert torch.isfinite(out[:, :bad]).all()
        assert (out[:, :bad] - clean[:, :bad]).abs().max().item() <= ATOL
        if math.isnan(value):
            assert torch.isnan(out[:, bad:]).all()


def test_f32_attention_bad_rows_are_nan():
    q, k, v = _inputs(2, 50, 4, 4, 64, 6)
    rows = torch.tensor([[0, 7, 49], [3, -1, 50]], dtype=torch.int32, device=DEV)
    out, lse = ops.selective_attention_lse(q, k, v, rows)
    torch.cuda.synchronize()
    want, _ = _ref(q, k, v, rows.clamp(0, 49))
    ok = torch.tensor([[True, True, True], [True, False, False]], device=DEV)
    assert (out[ok].double() - want[ok]).abs().max().item() <= ATOL
    assert torch.isnan(out[~ok]).all() and torch.isnan(lse[~ok]).all()
