"""Workloads that time the library through its public entry points (ops.*).

Kinds, and what each stands for in use:

  prefill   one layer of selective prefill of a batch of recommendation prompts
            (instruction + history block + item blocks, each block reused from
            a pool): gather + re-alignment + score, top-k + patch, attention of
            the fresh and selected rows. chain "vref": value rows by reference
            (bf16, D = 128); chain "copy": assembled V (every type and D).
  paged     the same step without an assembled copy.
  tokens    the same step with a token-granular history (one prototype row per
            position) through the per-position source map.
  full      the Full-Recompute baseline: causal attention of every row.
  eq3       selection by the full importance score: first layer in full with
            log-sum-exp, attention mass, gather, two-class top-k, patch.
  stack     selective prefill through decoder layers of Llama-3-8B dimensions
            (a whole call: projections, norms, attention, MLP).
  tail      the part of one decoder layer after attention for the recomputed
            rows: output projection + residual, RMSNorm, gate/up, SwiGLU, down.

Inputs. Block contents are N(0, 1) before rotation; cached keys are stored
rotated to block-local positions and the request's fresh keys are the block's
keys plus noise, rotated to the prompt positions. The noise of a position is
small (sigma about 0.05) except for the heavy hitters, whose number per request
is the recompute budget (the ratio is chosen to cover them) and whose noise is
8 to 12 times larger. Selection is then the same whatever the rounding of the
last bit, so outputs of two correct implementations can be compared row by row.
"""
from __future__ import annotations

import math

import torch

from paper_2605_07443_amd import inputs, ops

ITEM_MASK = inputs.ITEM_POOL_MASK
LAM = 0.5
EPS = 1e-5
STACK_H, STACK_I = 4096, 14336   # Llama-3-8B layer dimensions


# ------------------------------------------------------------------ the cases

def listed():
    llama = dict(dtype="bf16", Hq=32, Hkv=8, D=128, base=500000.0)
    return [
        # the headline workload: 8 prompts of 3,008 tokens, 15% recomputed
        dict(name="prefill_vref_b8_n3008", kind="prefill", chain="vref", B=8, F=64, hist=1024,
             items=20, item_len=96, pct=15, pool=1000, dist="zipf", **llama),
        # one request on its own, as an interactive server answers it
        dict(name="prefill_copy_b1_n2080", kind="prefill", chain="copy", B=1, F=32, hist=512,
             items=24, item_len=64, pct=15, pool=1000, dist="zipf", **llama),
        # the smallest: the fp32 workload, where latency and launches count
        dict(name="prefill_f32_b1_n416", kind="prefill", chain="copy", dtype="f32", B=1, Hq=8,
             Hkv=8, D=64, base=10000.0, F=32, hist=128, items=4, item_len=64, pct=15, pool=16,
             dist="zipf"),
        # long prompts
        dict(name="prefill_vref_b4_n8160", kind="prefill", chain="vref", B=4, F=64, hist=4096,
             items=50, item_len=80, pct=10, pool=1000, dist="zipf", **llama),
        # a full batch whose items are spread over the pool (gather-bound)
        dict(name="prefill_vref_b64_n2080", kind="prefill", chain="vref", B=64, F=32, hist=512,
             items=24, item_len=64, pct=15, pool=4096, dist="uniform", **llama),
        # multi-head attention with D = 64, odd sizes everywhere
        dict(name="prefill_mha64_b4_n1031", kind="prefill", chain="copy", dtype="bf16", B=4, Hq=16,
             Hkv=16, D=64, base=10000.0, F=7, hist=395, items=17, item_len=37, pct=30, pool=500,
             dist="zipf"),
        # few recomputed rows, without an assembled copy
        dict(name="paged_b8_n4096", kind="paged", B=8, F=96, hist=1024, items=31, item_len=96,
             pct=5, pool=1000, dist="zipf", **llama),
        # token-granular history
        dict(name="tokens_b8_n3008", kind="tokens", B=8, F=64, hist=1024, items=20, item_len=96,
             pct=15, pool=1000, dist="zipf", protos=16384, **llama),
        # the Full-Recompute baseline of the headline workload
        dict(name="full_b8_n3008", kind="full", B=8, F=64, hist=1024, items=20, item_len=96,
             pct=15, pool=0, dist="zipf", **llama),
        # selection by the full importance score
        dict(name="eq3_b8_n3008", kind="eq3", B=8, F=64, hist=1024, items=20, item_len=96, pct=15,
             pool=1000, dist="zipf", **llama),
        # two decoder layers, selected rows only after the first
        dict(name="stack_b4_n3008", kind="stack", B=4, F=64, hist=1024, items=20, item_len=96,
             pct=15, pool=0, dist="zipf", layers=2, **llama),
        # one request's recomputed rows through the rest of a layer
        dict(name="tail_m506", kind="tail", dtype="bf16", M=506),
    ]


def _loguniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost_us(c):
    w = work(c)
    return w["bytes"] / 4e6 + w["flops"] / (8e8 if c["dtype"] == "bf16" else 2e6)


def draw(rng):
    limit = _cost_us(next(c for c in listed() if c["kind"] == "stack"))
    while True:
        kind = rng.choice(["prefill"] * 5 + ["paged", "tokens", "full", "eq3", "stack", "tail"])
        if kind == "tail":
            return dict(kind="tail", dtype="bf16", M=_loguniform(rng, 48, 4200))
        c = dict(kind=kind, dtype="bf16", B=_loguniform(rng, 1, 64), F=_loguniform(rng, 4, 96),
                 hist=_loguniform(rng, 32, 4096), items=_loguniform(rng, 2, 50),
                 item_len=_loguniform(rng, 16, 96), pct=rng.choice([0, 5, 10, 15, 15, 25, 50, 100]),
                 pool=_loguniform(rng, 64, 2000), dist=rng.choice(["zipf", "uniform"]))
        heads = rng.choice([(32, 8, 128)] * 3 + [(16, 4, 128), (8, 2, 128), (16, 16, 64), (4, 4, 64)])
        if kind in ("prefill", "tokens", "eq3") and rng.random() < 0.2:   # the small fp32 shapes
            c.update(dtype="f32", B=rng.randint(1, 2), hist=_loguniform(rng, 32, 256),
                     items=rng.randint(2, 8))
            heads = rng.choice([(8, 8, 64), (8, 2, 64)])
        if kind == "prefill":
            c["chain"] = "vref" if heads[2] == 128 and rng.random() < 0.5 else "copy"
        if kind == "tokens":
            c["protos"] = _loguniform(rng, 256, 16384)
        if kind in ("full", "stack"):
            c["pool"] = 0
        if kind == "stack":
            heads = (32, 8, 128)
            c.update(B=rng.randint(1, 4), layers=2, pct=rng.choice([5, 10, 15, 25]))
        c["Hq"], c["Hkv"], c["D"] = heads
        c["base"] = 500000.0 if c["D"] == 128 else 10000.0
        c["pool"] = max(c["pool"], c["items"]) if c["pool"] else 0
        if _cost_us(c) <= limit and c["B"] * _N(c) <= 64 * 2080 and c["pool"] * c["item_len"] <= 300000:
            return c


# -------------------------------------------------------------------- sizes

def _N(c):
    return c["F"] + c["hist"] + c["items"] * c["item_len"]


def _budgets(c):
    """(history, item) positions and the budgets: one for both, or one each (eq3)."""
    nh, ni = c["hist"], c["items"] * c["item_len"]
    ceil = lambda n: (n * c["pct"] + 99) // 100  # noqa: E731
    return nh, ni, ceil(nh + ni), ceil(nh), ceil(ni)


def _k(c):
    _, _, k, kh, ki = _budgets(c)
    return kh + ki if c["kind"] == "eq3" else k


def work(c):
    if c["kind"] == "tail":
        m, h, i = c["M"], STACK_H, STACK_I
        w = h * h + 3 * h * i
        return {"bytes": 2.0 * (w + 4 * m * h), "flops": 2.0 * m * w}
    es = 2 if c["dtype"] == "bf16" else 4
    B, N, Hq, Hkv, D = c["B"], _N(c), c["Hq"], c["Hkv"], c["D"]
    row, qrow = Hkv * D * es, Hq * D * es
    k = _k(c)
    R, nr = c["F"] + k, N - c["F"]
    visible = c["F"] * (c["F"] + 1) / 2 + k * (N + c["F"] + 1) / 2   # keys seen by the rows, on average
    attend = 4.0 * D * Hq * visible
    full = 4.0 * D * Hq * N * (N + 1) / 2
    kind = c["kind"]
    if kind == "full":
        return {"bytes": B * (2.0 * N * row + 2.0 * N * qrow), "flops": B * full}
    if kind == "eq3":
        # q, fresh K/V, pool K/V read; output, lse, mass, assembled K/V, scores, rows written
        return {"bytes": B * (2.0 * N * qrow + 2.0 * N * row + 2.0 * nr * row + 2.0 * N * row
                              + 4.0 * N * (Hq + Hkv + 1) + 4.0 * R), "flops": B * 1.5 * full}
    if kind == "stack":
        h, i, L = STACK_H, STACK_I, c["layers"]
        qkv, rest = h * (Hq + 2 * Hkv) * D, h * Hq * D + 3 * h * i
        return {"bytes": 2.0 * L * (qkv + rest) + B * 2.0 * (N + R) * h
                + B * (nr * row + (L - 1) * 2.0 * nr * row),
                "flops": 2.0 * B * (N * qkv + (L - 1) * R * qkv + L * R * rest) + B * L * attend}
    # prefill, paged, tokens: q of the rows, pool K/V of cached positions, fresh
    # K of every position (score) and fresh V of the rows read; output, scores,
    # rows and (with an assembled copy) K, V written
    written = {"vref": 1.0, "copy": 2.0}[c["chain"]] if kind == "prefill" else 2.0 if kind == "tokens" else 0.0
    return {"bytes": B * (2.0 * R * qrow + (2.0 * nr + N + R) * row + written * N * row + 4.0 * N + 4.0 * R),
            "flops": B * attend}


def tolerance(c):
    # Measured against exact(): bf16 layers 2e-3 to 3e-3 (rounding of K, P and
    # the output), stack 5e-3, fp32 up to 3e-7; four times that, and a little
    # more in fp32, where the order of a sum decides.
    if c["dtype"] == "f32":
        return {"rel": 3e-6, "max": 1e-4}
    return {"rel": 0.02 if c["kind"] == "stack" else 0.01, "max": 0.3}


# -------------------------------------------------------------------- inputs

def _gen(seed, device, salt):
    g = torch.Generator(device=device)
    g.manual_seed((int(seed) * 1000003 + salt * 7919 + 17) & 0x7FFFFFFFFFFFFFFF)
    return g


def _angles(pos, D, base, dt):
    j = torch.arange(D // 2, dtype=torch.float64, device=pos.device)
    ang = pos.to(torch.float64)[..., None] * torch.pow(torch.tensor(base, dtype=torch.float64, device=pos.device), -2.0 * j / D)
    return torch.cos(ang).to(dt), torch.sin(ang).to(dt)


def _rope(x, pos, base):
    """Rotate-half RoPE of x [..., T, H, D] by pos [T] (or [..., T]), in x's type."""
    D = x.shape[-1]
    c, s = _angles(pos, D, base, x.dtype)
    c, s = c[..., None, :], s[..., None, :]
    a, b = x[..., : D // 2], x[..., D // 2:]
    return torch.cat([a * c - b * s, a * s + b * c], dim=-1)


def _dt(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _tables(c, hist_ids, item_ids):
    """Segment table [B, S, 4]: instruction (fresh), history (pool 0), items (pool 1)."""
    B, n = c["B"], c["items"]
    segs = torch.zeros((B, 2 + n, 4), dtype=torch.int32)
    segs[:, 0] = torch.tensor([0, c["F"], -1, 0])
    segs[:, 1, 0], segs[:, 1, 1], segs[:, 1, 2] = c["F"], c["hist"], 0
    segs[:, 1, 3] = hist_ids
    segs[:, 2:, 0] = c["F"] + c["hist"] + torch.arange(n, dtype=torch.int32) * c["item_len"]
    segs[:, 2:, 1], segs[:, 2:, 2] = c["item_len"], 1
    segs[:, 2:, 3] = item_ids
    return segs


def _ids(c, seed, hist_pool):
    g = _gen(seed, "cpu", 1)
    hist = torch.randint(0, hist_pool, (c["B"],), generator=g).to(torch.int32)
    if c["dist"] == "zipf":
        w = torch.arange(1, c["pool"] + 1, dtype=torch.float64).pow(-1.1)
    else:
        w = torch.ones(c["pool"], dtype=torch.float64)
    pick = torch.multinomial(w.expand(c["B"], -1), c["items"], replacement=False, generator=g)
    return hist, torch.randperm(c["pool"], generator=g)[pick].to(torch.int32)


def _sigma(c, seed, dev):
    """Noise of every cached position [B, N - F]: small, and 8 to 12 times larger
    at the heavy hitters (as many as the budget; of the history for eq3)."""
    g = _gen(seed, dev, 2)
    nh, ni, k, kh, _ = _budgets(c)
    n = nh + ni
    sig = 0.05 * torch.exp(0.1 * torch.randn((c["B"], n), generator=g, device=dev).clamp_(-3, 3))
    among, many = (nh, kh) if c["kind"] == "eq3" else (n, k)
    if many:
        at = torch.rand((c["B"], among), generator=g, device=dev).topk(many, dim=1).indices
        sig.scatter_(1, at, 0.4 + 0.2 * torch.rand((c["B"], many), generator=g, device=dev))
    return sig


def _prompts(c, seed, dev):
    """q, fresh K/V, pools and tables of a batch."""
    dt, B, N, F, Hkv, D = _dt(c), c["B"], _N(c), c["F"], c["Hkv"], c["D"]
    g = _gen(seed, dev, 3)
    rn = lambda *s: torch.randn(s, generator=g, device=dev)  # noqa: E731
    q = rn(B, N, c["Hq"], D).to(dt)
    kf, vf = torch.empty((B, N, Hkv, D), dtype=dt, device=dev), torch.empty((B, N, Hkv, D), dtype=dt, device=dev)
    kf[:, :F], vf[:, :F] = rn(B, F, Hkv, D).to(dt), rn(B, F, Hkv, D).to(dt)
    s = dict(c=c, q=q, kf=kf, vf=vf)
    if c["kind"] == "full":
        kf[:, F:], vf[:, F:] = rn(B, N - F, Hkv, D).to(dt), rn(B, N - F, Hkv, D).to(dt)
        return s
    sig = _sigma(c, seed, dev)[..., None, None]
    hist_pool = max(4, min(64, 65536 // c["hist"]))
    hist_ids, item_ids = _ids(c, seed, hist_pool)
    pos = torch.arange(N, device=dev)
    pools = []
    h1 = F + c["hist"]
    tokens = c["kind"] == "tokens"
    parts = [(c["protos"] if tokens else hist_pool, 1 if tokens else c["hist"], F, h1), (c["pool"], c["item_len"], h1, N)]
    proto = torch.randint(0, c["protos"], (B, c["hist"]), generator=_gen(seed, "cpu", 4)) if tokens else None
    for p, (count, length, a, b) in enumerate(parts):
        raw, val = rn(count, length, Hkv, D), rn(count, length, Hkv, D)
        at = (proto if tokens else hist_ids[:, None]) if p == 0 else item_ids
        at = at.to(device=dev, dtype=torch.int64)
        mine = lambda t: t[at].reshape(B, b - a, Hkv, D)  # noqa: E731
        noise = sig[:, a - F:b - F]
        kf[:, a:b] = _rope(mine(raw) + noise * rn(B, b - a, Hkv, D), pos[a:b], c["base"]).to(dt)
        vf[:, a:b] = (mine(val) + noise * rn(B, b - a, Hkv, D)).to(dt)
        pools.append((_rope(raw, pos[:length], c["base"]).to(dt), val.to(dt)))
        del raw, val
    segs = _tables(c, torch.zeros_like(hist_ids) if tokens else hist_ids, item_ids)
    s["segs"] = ops.prepare_segments(segs, N, pools, dev, check_blocks=not tokens)
    s["pools"] = pools
    if tokens:
        tmap = torch.zeros((B, N, 4), dtype=torch.int32)
        tmap[:, :F, 0] = -1
        tmap[:, F:h1, 1], tmap[:, F:h1, 2] = proto.to(torch.int32), torch.arange(F, h1, dtype=torch.int32)
        off = torch.arange(c["item_len"], dtype=torch.int32)
        tmap[:, h1:, 0] = 1
        tmap[:, h1:, 1] = (item_ids[..., None] * c["item_len"] + off).reshape(B, -1)
        tmap[:, h1:, 2] = (segs[:, 2:, 0, None].expand(-1, -1, c["item_len"])).reshape(B, -1)
        s["map"] = tmap.to(dev)
    return s


def prepare(case, seed):
    c = dict(case)
    dev = torch.device("cuda:0")
    if c["kind"] == "tail":
        layer = inputs.make_layers(1, STACK_H, 32, 8, 128, STACK_I, int(seed), dev)[0]
        g = _gen(seed, dev, 5)
        rn = lambda *s: torch.randn(s, generator=g, device=dev).to(torch.bfloat16)  # noqa: E731
        return dict(c=c, layer=layer, x=rn(c["M"], STACK_H), attn=rn(c["M"], STACK_H) * 0.5)
    B, N, Hq, Hkv, D = c["B"], _N(c), c["Hq"], c["Hkv"], c["D"]
    cos, sin = ops.rope_table(N, D, c["base"], dev)
    if c["kind"] == "stack":
        return dict(_stack(c, seed, dev), cos=cos, sin=sin)
    s = dict(_prompts(c, seed, dev), cos=cos, sin=sin)
    if c["kind"] == "full":
        s["out"] = torch.empty_like(s["q"])
    elif c["kind"] == "eq3":
        s["bufs"] = ops.Eq3Buffers.alloc(B, N, Hq, Hkv, D, c["F"] + _k(c), _dt(c), dev)
    else:
        vref = c["kind"] == "prefill" and c["chain"] == "vref"
        s["bufs"] = ops.PrefillBuffers.alloc(B, N, Hq, Hkv, D, c["F"] + _k(c), _dt(c), dev, v_copy=not vref, v_ref=vref)
    return s


def _stack(c, seed, dev):
    """Input states, layer weights and per-layer pools. The first layer's pools
    hold the prompt's own keys and values plus the position noise (its selection
    compares them with the projected ones); later layers' are independent."""
    B, N, F, Hq, Hkv, D, L = c["B"], _N(c), c["F"], c["Hq"], c["Hkv"], c["D"], c["layers"]
    g = _gen(seed, dev, 6)
    rn = lambda *s: torch.randn(s, generator=g, device=dev)  # noqa: E731
    x = rn(B, N, STACK_H).to(torch.bfloat16)
    layers = inputs.make_layers(L, STACK_H, Hq, Hkv, D, STACK_I, int(seed), dev)
    f = x.view(B * N, STACK_H).float()
    n = (f / torch.sqrt(f.square().mean(1, keepdim=True) + EPS) * layers[0].g_attn.float()).to(torch.bfloat16)
    kv = torch.mm(n, layers[0].w_qkv[Hq * D:].t()).float().view(B, N, 2, Hkv, D)
    sig = _sigma(c, seed, dev)[..., None, None]
    h1, pos, pools = F + c["hist"], torch.arange(N, device=dev), []
    for l in range(L):
        both = []
        for a, b, length in ((F, h1, c["hist"]), (h1, N, c["item_len"])):
            shape = (B * (b - a) // length, length, Hkv, D)
            k, v = ((kv[:, a:b, i] + sig[:, a - F:b - F] * rn(B, b - a, Hkv, D)).reshape(shape) if l == 0
                    else rn(*shape) for i in (0, 1))
            both.append((_rope(k, pos[:length], c["base"]).to(torch.bfloat16), v.to(torch.bfloat16).contiguous()))
        pools.append(both)
    ids = torch.arange(B * c["items"], dtype=torch.int32).view(B, c["items"])
    segs = ops.prepare_segments(_tables(c, torch.arange(B, dtype=torch.int32), ids), N, pools[0], dev)
    return dict(c=c, x=x, layers=layers, pools=pools, segs=segs)


# -------------------------------------------------------------------- one pass

def run(s):
    c, kind = s["c"], s["c"]["kind"]
    if kind == "tail":
        L = s["layer"]
        h = ops.gemm(s["attn"], L.w_o, residual=s["x"])
        act = ops.silu_mul(ops.gemm(ops.rmsnorm(h, L.g_mlp, EPS), L.w_gu))
        return {"h": h, "y": ops.gemm(act, L.w_down, residual=h)}
    if kind == "full":
        return {"out": ops.full_prefill(s["q"], s["kf"], s["vf"], out=s["out"])}
    if kind == "stack":
        hidden, rows, scores = ops.stack_prefill(s["x"], s["layers"], s["pools"], s["segs"], _k(c), s["cos"], s["sin"], EPS)
        return {"hidden": hidden, "rows": rows, "scores": scores}
    args = (s["q"], s["kf"], s["vf"], s["pools"], s["segs"])
    b = s["bufs"]
    if kind == "eq3":
        _, _, _, kh, ki = _budgets(c)
        ops.eq3_select(*args, ITEM_MASK, LAM, kh, ki, s["cos"], s["sin"], bufs=b)
        return {"k_asm": b.k_asm, "v_asm": b.v_asm, "out_full": b.out_full, "lse": b.lse, "mass": b.mass,
                "scores": b.scores, "rows": b.rows}
    if kind == "paged":
        ops.paged_prefill(*args, _k(c), s["cos"], s["sin"], bufs=b)
        return {"scores": b.scores, "rows": b.rows, "out": b.out}
    if kind == "tokens":
        ops.kv_gather_tokens(s["pools"], s["map"], s["kf"], s["vf"], s["cos"], s["sin"], b.k_asm, b.v_asm, scores_out=b.scores)
        ops.select_tokens(s["segs"], _k(c), s["kf"], s["vf"], b.k_asm, b.v_asm, scores_in=b.scores, rows_out=b.rows)
        ops.selective_attention(s["q"], b.k_asm, b.v_asm, b.rows, out=b.out)
    elif c["chain"] == "vref":   # the table of row addresses is no output: addresses differ from run to run
        ops.selective_prefill_vref(*args, _k(c), s["cos"], s["sin"], bufs=b)
        return {"k_asm": b.k_asm, "scores": b.scores, "rows": b.rows, "out": b.out}
    else:
        ops.selective_prefill(*args, _k(c), s["cos"], s["sin"], bufs=b)
    return {"k_asm": b.k_asm, "v_asm": b.v_asm, "scores": b.scores, "rows": b.rows, "out": b.out}


# -------------------------------------------------------- the same in 64 bits

def _attention64(q, k, v, pos, lse=False):
    """One request: q [R, Hq, D] at positions pos, k/v [N, Hkv, D] -> out [R, Hq, D] (and lse [R, Hq])."""
    R, Hq, D = q.shape
    N, Hkv = k.shape[:2]
    G = Hq // Hkv
    out, ls = torch.empty_like(q), torch.empty((R, Hq), dtype=q.dtype, device=q.device)
    key = torch.arange(N, device=q.device)
    step = max(1, 200_000_000 // (G * N))
    for r in range(0, R, step):
        hide = (key[None, :] > pos[r:r + step, None])[:, None, :]
        for h in range(Hkv):
            qs = q[r:r + step, h * G:(h + 1) * G]
            s = (torch.mm(qs.reshape(-1, D), k[:, h].t().contiguous()) / math.sqrt(D)).view(qs.shape[0], G, N)
            s.masked_fill_(hide, -math.inf)
            l = torch.logsumexp(s, dim=-1)
            ls[r:r + step, h * G:(h + 1) * G] = l
            s.sub_(l[..., None]).exp_()
            out[r:r + step, h * G:(h + 1) * G] = torch.mm(s.view(-1, N), v[:, h].contiguous()).view(qs.shape)
    return (out, ls) if lse else out


def _mass64(q, k, lse):
    """One request: the softmax weights that every key receives, [Hkv, N]."""
    N, Hq, D = q.shape
    Hkv = k.shape[1]
    G = Hq // Hkv
    mass = torch.zeros((Hkv, N), dtype=q.dtype, device=q.device)
    key = torch.arange(N, device=q.device)
    for h in range(Hq):
        s = torch.mm(q[:, h], k[:, h // G].t().contiguous()) / math.sqrt(D) - lse[:, h, None]
        s.masked_fill_(key[None, :] > key[:, None], -math.inf)
        mass[h // G] += s.exp_().sum(0)
    return mass


def _norm64(x, gamma):
    return x / torch.sqrt(x.square().mean(-1, keepdim=True) + EPS) * gamma.double()


def _mlp64(h, L):
    gu = _norm64(h, L.g_mlp) @ L.w_gu.double().t()
    half = gu.shape[1] // 2
    return (torch.nn.functional.silu(gu[:, :half]) * gu[:, half:]) @ L.w_down.double().t() + h


def _cached64(c, b, segs, pools, device, tmap=None):
    """The aligned K and V of request b's cached positions, [N - F, Hkv, D]."""
    N, F = _N(c), c["F"]
    k = torch.empty((N - F, c["Hkv"], c["D"]), dtype=torch.float64, device=device)
    v = torch.empty_like(k)
    for dst, length, p, blk in segs.host[b].tolist():
        if p < 0:
            continue
        at = slice(dst - F, dst - F + length)
        if tmap is not None and p == 0:
            rows = tmap[b, dst:dst + length, 1].long()
            k[at] = _rope(pools[0][0][rows, 0].double(), torch.arange(dst, dst + length, device=device), c["base"])
            v[at] = pools[0][1][rows, 0].double()
        else:
            k[at] = _rope(pools[p][0][blk, :length].double(), torch.full((length,), dst, device=device), c["base"])
            v[at] = pools[p][1][blk, :length].double()
    return k, v


def exact(case, seed):
    s = prepare(case, seed)
    c, kind = s["c"], s["c"]["kind"]
    if kind == "tail":
        L = s["layer"]
        h = s["attn"].double() @ L.w_o.double().t() + s["x"].double()
        return {"h": h, "y": _mlp64(h, L)}
    if kind == "stack":
        return _stack64(s)
    B, N, F = c["B"], _N(c), c["F"]
    dev = s["q"].device
    every = torch.arange(N, device=dev)
    if kind == "full":
        return {"out": torch.stack([_attention64(s["q"][b].double(), s["kf"][b].double(), s["vf"][b].double(), every) for b in range(B)])}
    got = {n: [] for n in ("k_asm", "v_asm", "scores", "out", "out_full", "lse", "mass")}
    for b in range(B):
        q, kf, vf = s["q"][b].double(), s["kf"][b].double(), s["vf"][b].double()
        k, v = (torch.cat([f[:F], t]) for f, t in zip((kf, vf), _cached64(c, b, s["segs"], s["pools"], dev, s.get("map"))))
        dk, dv = ((f - t).abs().sum((1, 2)) for f, t in ((kf, k), (vf, v)))
        if kind == "eq3":
            o, l = _attention64(q, kf, vf, every, lse=True)
            m = _mass64(q, kf, l)
            h1 = F + c["hist"]
            score = (1 - LAM) * m.sum(0) + LAM * torch.where(every < h1, dk + dv, torch.zeros_like(dk))
            _, _, _, kh, ki = _budgets(c)
            rows = torch.cat([every[:F], F + score[F:h1].topk(kh).indices, h1 + score[h1:].topk(ki).indices]).sort().values
            got["out_full"].append(o), got["lse"].append(l), got["mass"].append(m)
        else:
            score = dk
            rows = torch.cat([every[:F], F + score[F:].topk(_k(c)).indices]).sort().values
        k[rows], v[rows] = kf[rows], vf[rows]
        got["k_asm"].append(k), got["v_asm"].append(v), got["scores"].append(score)
        if kind != "eq3":
            got["out"].append(_attention64(q[rows], k, v, rows))
    got = {n: torch.stack(t) for n, t in got.items() if t}
    if kind == "paged" or c.get("chain") == "vref":
        got.pop("v_asm")
    if kind == "paged":
        got.pop("k_asm")
    return dict(got, rows=None)


def _stack64(s):
    c = s["c"]
    B, N, F, Hq, Hkv, D = c["B"], _N(c), c["F"], c["Hq"], c["Hkv"], c["D"]
    dev = s["x"].device
    every = torch.arange(N, device=dev)
    hidden, scores = [], []
    for b in range(B):
        x = s["x"][b].double()
        rows = every
        for l, L in enumerate(s["layers"]):
            qkv = (_norm64(x, L.g_attn) @ L.w_qkv.double().t()).view(len(rows), Hq + 2 * Hkv, D)
            q, k, v = _rope(qkv[:, :Hq], rows, c["base"]), _rope(qkv[:, Hq:Hq + Hkv], rows, c["base"]), qkv[:, Hq + Hkv:]
            ck, cv = _cached64(c, b, s["segs"], s["pools"][l], dev)
            if l == 0:
                dk = torch.cat([torch.zeros(F, dtype=torch.float64, device=dev), (k[F:] - ck).abs().sum((1, 2))])
                scores.append(dk)
                rows = torch.cat([every[:F], F + dk[F:].topk(_k(c)).indices]).sort().values
                q, x = q[rows], x[rows]
            else:
                ck, cv = (torch.cat([torch.zeros((F, Hkv, D), dtype=torch.float64, device=dev), t]) for t in (ck, cv))
                ck[rows], cv[rows] = k, v
                k, v = ck, cv
            a = _attention64(q.contiguous(), k.contiguous(), v.contiguous(), rows)
            x = _mlp64(a.reshape(len(rows), Hq * D) @ L.w_o.double().t() + x, L)
        hidden.append(x)
    return {"hidden": torch.stack(hidden), "rows": None, "scores": torch.stack(scores)}
