"""rc_attention_mass with a workspace (query tiles divided over workgroups)
against fp64 and the undivided call."""
import ctypes
import math

import pytest
import torch

from paper_2605_07443_amd import _lib, ops

DEV = "cuda:0"


def _parts(B, N, Hq, Hkv, D, dtype=_lib.RC_BF16):
    b = _lib.load().rc_mass_workspace_bytes(ctypes.byref(_lib.RcShape(B, N, Hq, Hkv, D, dtype)))
    assert b % (4 * B * Hkv * N) == 0
    return b // (4 * B * Hkv * N)


def test_parts_rule():
    assert _parts(8, 3008, 32, 8, 128) == 2 and _parts(1, 3008, 32, 8, 128) == 16
    assert _parts(1, 100, 32, 8, 128) == 0 and _parts(64, 2080, 32, 8, 128) == 0
    assert _parts(1, 3008, 32, 8, 128, _lib.RC_F32) == 0 and _parts(1, 3008, 3, 1, 128) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("B,N,Hq,Hkv,D", [(1, 130, 8, 1, 64), (1, 255, 16, 2, 128), (1, 257, 64, 1, 64),
                                          (2, 750, 32, 8, 128), (1, 1999, 4, 4, 64), (1, 300, 128, 1, 128)])
def test_divided_mass(B, N, Hq, Hkv, D):
    print(f"[mass] {B} {N} {Hq} {Hkv} {D} parts={_parts(B, N, Hq, Hkv, D)}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(N)
    q = torch.randn((B, N, Hq, D), generator=g, device=DEV).to(torch.bfloat16)
    k = torch.randn((B, N, Hkv, D), generator=g, device=DEV).to(torch.bfloat16)
    G = Hq // Hkv
    want = torch.zeros((B, Hkv, N), dtype=torch.float64, device=DEV)
    lse = torch.empty((B, N, Hq), dtype=torch.float64, device=DEV)
    hide = torch.arange(N, device=DEV)[None, :] > torch.arange(N, device=DEV)[:, None]
    for b in range(B):
        for h in range(Hq):
            s = torch.mm(q[b, :, h].double(), k[b, :, h // G].double().t().contiguous()) / math.sqrt(D)
            s = s.masked_fill(hide, -math.inf)
            lse[b, :, h] = torch.logsumexp(s, -1)
            want[b, h // G] += torch.softmax(s, -1).sum(0)
    l32 = lse.float()
    mass, again = ops.attention_mass(q, k, l32), ops.attention_mass(q, k, l32)
    plain = torch.full_like(mass, 7.0)
    vp = ctypes.c_void_p
    _lib.check(_lib.load().rc_attention_mass(
        ctypes.byref(_lib.RcShape(B, N, Hq, Hkv, D, _lib.RC_BF16)), vp(q.data_ptr()), vp(k.data_ptr()),
        vp(l32.data_ptr()), ctypes.c_float(1 / math.sqrt(D)), vp(plain.data_ptr()),
        vp(torch.cuda.current_stream().cuda_stream)))
    torch.cuda.synchronize()
    assert torch.equal(mass, again)
    for got in (mass, plain):   # the bound of the oracle's mass test
        torch.testing.assert_close(got.double(), want, rtol=2e-5, atol=1e-6)
