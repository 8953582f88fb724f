"""The calls this library is timed on: one pass of each public entry point a
program uses (attention prefill and decode, MLA decode, matrix and
matrix-vector products, the Mamba-2 chunked forward), from launch-bound to
large, with the arithmetic of each in 64 bits beside it.

Inputs are drawn on the GPU from the seed alone, with the distributions of
``paper_2504_17577_amd.gen``: unit normals in bf16 for activations, queries,
keys, values and caches (Q and K that give scores of unit variance), weight
matrices scaled by 1/sqrt(K), and Mamba-2's initialisation ranges for dt and A.
"""
from __future__ import annotations

import math

import torch

from paper_2504_17577_amd import gen, tileattn

CHUNK = tileattn.SSD_CHUNK


# ---------------------------------------------------------------------------
# The cases

def _attn(B, Hq, Hkv, Sq, Sk, D, causal, out, split=False):
    return dict(kind="attn", B=B, Hq=Hq, Hkv=Hkv, Sq=Sq, Sk=Sk, D=D, causal=causal, out=out,
                split=split)


def _mla(B, H, Hkv, Skv):
    return dict(kind="mla", B=B, H=H, Hkv=Hkv, Skv=Skv)


def _gemm(M, N, K, out, split=False):
    return dict(kind="gemm", M=M, N=N, K=K, out=out, split=split)


def _ssd(B, L, H, G, skip):
    return dict(kind="ssd", B=B, L=L, H=H, G=G, skip=skip)


def listed():
    cases = {
        # one short sequence, two heads: the smallest call there is, all launch
        "attn_tiny_d64_s128": _attn(1, 2, 2, 128, 128, 64, False, "fp32"),
        # a batch of prompts of odd length through a model of head dim 64
        "attn_causal_d64_s1001": _attn(4, 16, 16, 1001, 1001, 64, True, "fp32"),
        # the benchmark's dense forward (an encoder, or a training forward)
        "attn_dense_d128_s2k": _attn(8, 32, 32, 2048, 2048, 128, False, "fp32"),
        # prefill of two 4k prompts in a grouped-query decoder, bf16 activations
        "attn_gqa4_causal_d128_s4k": _attn(2, 32, 8, 4096, 4096, 128, True, "bf16"),
        # one decode step of eight sequences of the same decoder against an 8k cache
        "attn_decode_gqa4_b8_s8191": _attn(8, 32, 8, 1, 8191, 128, False, "bf16", split=True),
        # MLA decode step of a large serving batch (DeepSeek-V3's dimensions)
        "mla_b64_s8k": _mla(64, 128, 1, 8192),
        # the same at low batch and a cache of odd length, where latency counts
        "mla_b4_s1999": _mla(4, 128, 1, 1999),
        # the paper's shape M1: a projection over 4096 tokens
        "gemm_m1": _gemm(4096, 8192, 8192, "bf16"),
        # a projection over a short chunk of tokens, odd tile counts
        "gemm_m384_n4224_k8256": _gemm(384, 4224, 8256, "bf16"),
        # the paper's shape V5: one token's projection
        "gemv_v5": _gemm(1, 9216, 9216, "bf16", split=True),
        # Mamba-2 forward of one short prompt of odd length
        "ssd_b1_s1000": _ssd(1, 1000, 64, 1, True),
        # Mamba-2 forward of a full batch (the paper's 64 x 2048)
        "ssd_b64_s2k": _ssd(64, 2048, 64, 1, True),
    }
    return [dict(name=n, **c) for n, c in cases.items()]


def _log(rng, lo, hi):
    """An integer in [lo, hi], even over the logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_any(rng):
    kind = rng.choice(["prefill", "chunk", "decode", "mla", "gemm", "gemv", "ssd"])
    out = rng.choice(["fp32", "bf16"])
    if kind in ("prefill", "chunk", "decode"):
        D = rng.choice([64, 128])
        Hkv = rng.choice([2, 4, 8, 16, 32])
        Hq = Hkv * rng.choice([g for g in (1, 2, 4, 8) if Hkv * g <= 64])
        if kind == "prefill":      # whole prompts
            S = _log(rng, 100, 4096)
            return _attn(_log(rng, 1, 8), Hq, Hkv, S, S, D, rng.random() < 0.6, out)
        if kind == "chunk":        # a chunk of queries against a longer cache
            return _attn(_log(rng, 1, 4), Hq, Hkv, _log(rng, 64, 1024), _log(rng, 1024, 8192), D,
                         rng.random() < 0.6, out, split=rng.random() < 0.5)
        return _attn(_log(rng, 1, 16), Hq, Hkv, 1, _log(rng, 512, 16384), D, False, out,
                     split=True)
    if kind == "mla":
        return _mla(_log(rng, 1, 64), *rng.choice([(128, 1), (128, 1), (64, 2), (16, 1)]),
                    _log(rng, 200, 8192))
    if kind == "gemm":             # M, N in tiles of 128, K in steps of 64
        return _gemm(128 * _log(rng, 1, 64), 128 * _log(rng, 3, 224), 64 * _log(rng, 3, 448), out)
    if kind == "gemv":             # N in 64s, K in 8s
        return _gemm(1, 64 * _log(rng, 16, 600), 8 * _log(rng, 128, 4600), out,
                     split=rng.random() < 0.7)
    G = rng.choice([1, 1, 2, 8])
    return _ssd(_log(rng, 1, 64), _log(rng, 200, 8192), rng.choice([24, 32, 64]), G,
                rng.random() < 0.8)


def draw(rng):
    top = [work(c) for c in listed()]
    flops = max(w["flops"] for w in top)
    while True:
        c = _draw_any(rng)
        w = work(c)
        limit = max(t["bytes"] for t, l in zip(top, listed()) if l["kind"] == c["kind"])
        if w["flops"] <= flops and w["bytes"] <= limit and (
                not c.get("causal") or c["Sq"] <= c["Sk"]):
            return c


# ---------------------------------------------------------------------------
# Inputs and the timed pass

def _normal(g, shape, std=1.0, dtype=torch.bfloat16):
    # drawn in slices of 2^27 elements, so that no fp32 copy of a large tensor is made
    t = torch.empty(shape, dtype=dtype, device=g.device)
    flat = t.view(-1)
    for i in range(0, flat.numel(), 1 << 27):
        s = flat[i:i + (1 << 27)]
        s.copy_(torch.randn(s.numel(), generator=g, device=g.device).mul_(std))
    return t


def _uniform(g, shape, lo, hi):
    return torch.rand(shape, generator=g, device=g.device).mul_(hi - lo).add_(lo)


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    c = case
    if c["kind"] == "attn":
        return dict(case=c, q=_normal(g, (c["B"], c["Hq"], c["Sq"], c["D"])),
                    k=_normal(g, (c["B"], c["Hkv"], c["Sk"], c["D"])),
                    v=_normal(g, (c["B"], c["Hkv"], c["Sk"], c["D"])))
    if c["kind"] == "mla":
        return dict(case=c, q=_normal(g, (c["B"], c["H"], 512)),
                    q_pe=_normal(g, (c["B"], c["H"], 64)),
                    kv=_normal(g, (c["B"], c["Skv"], c["Hkv"], 512)),
                    k_pe=_normal(g, (c["B"], c["Skv"], c["Hkv"], 64)))
    if c["kind"] == "gemm":
        return dict(case=c, a=_normal(g, (c["M"], c["K"])),
                    b=_normal(g, (c["K"], c["N"]), std=c["K"] ** -0.5))
    B, L, H, G = c["B"], c["L"], c["H"], c["G"]
    return dict(case=c, x=_normal(g, (B, L, H, 64)), Bm=_normal(g, (B, L, G, 128)),
                Cm=_normal(g, (B, L, G, 128)),
                dt=_uniform(g, (B, L, H), math.log(1e-3), math.log(1e-1)).exp_(),
                A=-_uniform(g, (H,), 0.0, math.log(16.0)).exp_(),
                D=_uniform(g, (H,), 0.5, 1.5) if c["skip"] else None)


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "attn":
        if c["split"]:
            dt = torch.bfloat16 if c["out"] == "bf16" else torch.float32
            return tileattn.attn_fwd_split(s["q"], s["k"], s["v"], causal=c["causal"],
                                           out_dtype=dt)
        f = tileattn.attn_fwd_bf16out if c["out"] == "bf16" else tileattn.attn_fwd
        return f(s["q"], s["k"], s["v"], causal=c["causal"])
    if c["kind"] == "mla":
        return tileattn.mla_decode(s["q"], s["q_pe"], s["kv"], s["k_pe"])
    if c["kind"] == "gemm":
        f = tileattn.gemv_bf16_split if c["split"] else tileattn.gemm_bf16
        return f(s["a"], s["b"], out_dtype=torch.bfloat16 if c["out"] == "bf16" else None)
    return tileattn.ssd_forward(s["x"], s["dt"], s["A"], s["Bm"], s["Cm"], s["D"])


# ---------------------------------------------------------------------------
# What a pass cannot do without, and how close two correct passes are

def work(case):
    c = case
    if c["kind"] == "attn":
        w = gen.Workload("", 0, c["B"], c["Hq"], c["Hkv"], c["Sq"], c["Sk"], c["D"], c["causal"])
        return {"bytes": w.bytes(2 if c["out"] == "bf16" else 4), "flops": w.flops()}
    if c["kind"] == "mla":
        w = gen.MlaWorkload("", 0, c["B"], c["H"], c["Hkv"], c["Skv"])
        return {"bytes": w.bytes(), "flops": w.flops()}
    if c["kind"] == "gemm":
        w = gen.GemmWorkload("", 0, c["M"], c["N"], c["K"])
        return {"bytes": w.bytes(2 if c["out"] == "bf16" else 4), "flops": w.flops()}
    # x, Bm, Cm, dt, A, D read once; y and the final states written once.  The
    # matrix products of the chunked form at its chunk length: C B^T over the
    # visible pairs of each chunk and group, and the state and scan terms.
    B, L, H, G = c["B"], c["L"], c["H"], c["G"]
    w = gen.SsdWorkload("", 0, B, L, H, G)
    full, tail = divmod(L, CHUNK)
    pairs = full * CHUNK * (CHUNK + 1) // 2 + tail * (tail + 1) // 2
    n_bytes = (2 * B * L * (H * 64 + 2 * G * 128) + 4 * B * L * H + 8 * H
               + 4 * B * L * H * 64 + 4 * B * H * 64 * 128)
    return {"bytes": n_bytes,
            "flops": w.flops_state() + w.flops_scan() + 2 * 128 * B * G * pairs}


def tolerance(case):
    kind = case["kind"]
    if kind == "gemm":
        # exact products, fp32 sums; a bf16 result is rounded once (1.7e-3 from exact())
        return {"rel": 7e-3} if case["out"] == "bf16" else {"rel": 1e-5}
    if kind == "ssd":
        # the bf16 decay-weighted operands of the contractions: 1.7e-3 from exact()
        return {"rel": 7e-3}
    # bf16 softmax weights, fp32 sums: 0.7e-3 (MLA) to 2.3e-3 (bf16 O) from exact()
    return {"rel": 4e-3} if kind == "mla" else {"rel": 9e-3}


# ---------------------------------------------------------------------------
# The same results in 64 bits

def _attn_exact(s, c):
    q, k, v = (s[n].double() for n in "qkv")
    B, Hq, Sq, D = q.shape
    Sk, grp = k.shape[2], Hq // k.shape[1]
    o = torch.empty_like(q)
    lse = torch.empty(q.shape[:3], dtype=torch.float64, device=q.device)
    hide = None
    if c["causal"]:
        i = torch.arange(Sq, device=q.device)[:, None]
        hide = torch.arange(Sk, device=q.device)[None, :] > i + (Sk - Sq)
    for b in range(B):
        for h in range(Hq):
            sc = (q[b, h] @ k[b, h // grp].t().contiguous()) / math.sqrt(D)
            if hide is not None:
                sc.masked_fill_(hide, -math.inf)
            lse[b, h] = torch.logsumexp(sc, 1)
            o[b, h] = torch.exp(sc - lse[b, h][:, None]) @ v[b, h // grp]
    return o, lse


def _mla_exact(s, c):
    q = torch.cat([s["q"], s["q_pe"]], 2).double()
    B, H, _ = q.shape
    Hkv = c["Hkv"]
    grp = H // Hkv
    o = torch.empty(B, H, 512, dtype=torch.float64, device=q.device)
    lse = torch.empty(B, H, dtype=torch.float64, device=q.device)
    for b in range(B):
        for hk in range(Hkv):
            hs = slice(hk * grp, (hk + 1) * grp)
            kv = s["kv"][b, :, hk].double()
            key = torch.cat([kv, s["k_pe"][b, :, hk].double()], 1)
            sc = (q[b, hs] @ key.t().contiguous()) / math.sqrt(576)
            lse[b, hs] = torch.logsumexp(sc, 1)
            o[b, hs] = torch.exp(sc - lse[b, hs][:, None]) @ kv
    return o, lse


def _ssd_exact(s, c):
    """The recurrence h_t = exp(dt_t A) h_{t-1} + dt_t x_t Bm_t^T,
    y_t = h_t Cm_t + D x_t, in blocks of 128 positions: inside a block the
    masked decay matrix, between blocks the carried state."""
    B, L, H, G = c["B"], c["L"], c["H"], c["G"]
    Q, grp, dev = 128, H // G, s["x"].device
    A = s["A"].double()
    y = torch.empty(B, L, H, 64, dtype=torch.float64, device=dev)
    fin = torch.empty(B, H, 64, 128, dtype=torch.float64, device=dev)
    for b in range(B):
        st = torch.zeros(H, 64, 128, dtype=torch.float64, device=dev)
        for t in range(0, L, Q):
            u = slice(t, min(t + Q, L))
            x = s["x"][b, u].double().transpose(0, 1).contiguous()               # [H, n, 64]
            bm = s["Bm"][b, u].double().transpose(0, 1)                          # [G, n, 128]
            cm = s["Cm"][b, u].double().transpose(0, 1)
            bm = bm.repeat_interleave(grp, 0).contiguous()
            cm = cm.repeat_interleave(grp, 0).contiguous()
            dt = s["dt"][b, u].double().t().contiguous()                         # [H, n]
            a = torch.cumsum(dt * A[:, None], 1)
            n = x.shape[1]
            low = torch.ones(n, n, dtype=torch.bool, device=dev).tril()
            dec = (a[:, :, None] - a[:, None, :]).masked_fill(~low, -math.inf).exp()
            wx = x * dt[:, :, None]
            yb = ((cm @ bm.transpose(1, 2).contiguous()) * dec) @ wx
            yb += a.exp()[:, :, None] * (cm @ st.transpose(1, 2).contiguous())
            if s["D"] is not None:
                yb += s["D"].double()[:, None, None] * x
            y[b, u] = yb.transpose(0, 1)
            wx = wx * (a[:, -1:] - a).exp()[:, :, None]
            st = a[:, -1].exp()[:, None, None] * st + wx.transpose(1, 2).contiguous() @ bm
        fin[b] = st
    return y, fin


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] == "attn":
        return _attn_exact(s, case)
    if case["kind"] == "mla":
        return _mla_exact(s, case)
    if case["kind"] == "gemm":
        return s["a"].double() @ s["b"].double()
    return _ssd_exact(s, case)
