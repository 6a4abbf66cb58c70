"""Performance cases: the calls a user of this library makes, over the range of sizes it is used at.

A case is a dict of plain values.  ``listed()`` gives the fixed ones, ``draw(rng)`` one more
of the same ranges, ``prepare(case, seed)`` the tensors a program holds before the call,
``run(state)`` one pass through the public entry points, ``work(case)`` the bytes and
operations the pass cannot do without, ``tolerance(case)`` how far another correct
implementation at the same precision may be off, and ``exact(case, seed)`` the same outputs
in float64 from plain torch.

Kinds:
  attn    ring attention over the whole ring, forward or forward + backward
  host    one host's share of the ring, forward + backward
  decode  a few new tokens against a key/value cache
  ffn     blockwise feed-forward network, forward + backward
  layer   one Algorithm 1 transformer layer, forward + backward
  stack   training step of a stack of LLaMA-style layers
"""
import math

import torch

import paper_2310_01889_amd as ra


# ---------------------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------------------
def _attn(name, dtype, B, S, H, D, N, causal, train):
    c = dict(kind="attn", dtype=dtype, B=B, S=S, H=H, D=D, N=N, causal=causal, train=train)
    return dict(c, name=name) if name else c


def _host(name, c, H, D, N, host):
    d = dict(kind="host", c=c, H=H, D=D, N=N, host=host)
    return dict(d, name=name) if name else d


def _decode(name, B, S, H, D, Tq, N):
    d = dict(kind="decode", B=B, S=S, H=H, D=D, Tq=Tq, N=N)
    return dict(d, name=name) if name else d


def _ffn(name, T, dm, dff, block, act):
    d = dict(kind="ffn", T=T, dm=dm, dff=dff, block=block, act=act)
    return dict(d, name=name) if name else d


def _layer(name, S, dm, H, dff, N, act):
    d = dict(kind="layer", S=S, dm=dm, H=H, dff=dff, N=N, act=act)
    return dict(d, name=name) if name else d


def _stack(name, L, S, dm, H, dff, N):
    d = dict(kind="stack", L=L, S=S, dm=dm, H=H, dff=dff, N=N)
    return dict(d, name=name) if name else d


def listed():
    return [
        # the smallest: the float32 configuration (one head of 1024 tokens, 4 hosts of 256), as
        # a numerical reference or a small float32 model trains with it
        _attn("f32_tiny_train", "f32", 1, 1024, 1, 64, 4, True, True),
        # an ordinary float32 training call: several heads of 4096 tokens
        _attn("f32_train", "f32", 1, 4096, 8, 128, 8, True, True),
        # prefill of a 32768-token prompt at LLaMA-7B attention width (the headline workload)
        _attn("prefill_32k", "bf16", 1, 32768, 32, 128, 8, True, False),
        # training at the 16384-token, 16-head configuration
        _attn("train_16k", "bf16", 1, 16384, 16, 128, 8, True, True),
        # training on a batch whose length does not fill the hosts' blocks
        _attn("train_ragged", "bf16", 2, 3001, 8, 128, 8, True, True),
        # bidirectional attention with 64-wide heads (an encoder), a batch of short sequences
        _attn("train_bidir_d64", "bf16", 4, 2048, 12, 64, 4, False, True),
        # the last host's share of a long ring, 16384 queries against 131072 keys
        _host("host_share", 16384, 16, 128, 8, 7),
        # one new token against a full 262144-token cache
        _decode("decode_262k", 1, 262144, 32, 128, 1, 8),
        # a few new tokens (speculative decoding) for two short sequences: latency
        _decode("decode_short", 2, 4096, 16, 64, 4, 4),
        # the feed-forward network of the 4096-wide layer, 8192 tokens in blocks of 1024
        _ffn("ffn_4096", 8192, 4096, 16384, 1024, 0),
        # one layer of a small model on a short sequence
        _layer("layer_small", 2048, 1024, 8, 4096, 4, 0),
        # the largest: training step of two LLaMA-7B-width layers on 16384 tokens
        _stack("llama_train_16k", 2, 16384, 4096, 32, 11008, 8),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["attn", "attn", "attn", "f32", "host", "decode", "decode", "ffn", "layer", "stack"])
    cap = 0.8 * work(listed()[-1])["flops"]
    while True:
        if kind == "f32":
            N, D = rng.choice([1, 2, 4, 8]), rng.choice([64, 128])
            S = 64 * N * max(1, round(_log(rng, 256, 4096) / (64 * N)))
            c = _attn(None, "f32", rng.choice([1, 2]), S, rng.randint(1, 8), D, N, rng.random() < 0.75,
                      rng.random() < 0.6)
            if work(c)["flops"] <= 1.25 * work(listed()[1])["flops"]:
                return c
        elif kind == "attn":
            N, D = rng.choice([1, 2, 3, 4, 8]), rng.choice([64, 128, 128])
            causal = rng.random() < 0.8
            S = round(_log(rng, 512, 32768))
            if not causal or rng.random() < 0.4:
                S = 128 * N * max(1, round(S / (128 * N)))
            c = _attn(None, "bf16", rng.choice([1, 1, 2, 4]), S, round(_log(rng, 1, 32)), D, N, causal,
                      rng.random() < 0.7)
            if c["B"] * c["S"] * c["H"] * D < 2 ** 29 and work(c)["flops"] <= 0.25 * cap:
                return c
        elif kind == "host":
            N = rng.choice([2, 4, 8])
            c = _host(None, 128 * round(_log(rng, 1024, 16384) / 128), round(_log(rng, 2, 32)), rng.choice([64, 128]),
                      N, rng.randrange(N))
            if work(c)["flops"] <= work(listed()[6])["flops"]:
                return c
        elif kind == "decode":
            N = rng.choice([1, 2, 4, 8])
            S = 32 * N * round(_log(rng, 1024, 262144) / (32 * N))
            c = _decode(None, rng.choice([1, 2, 4]), S, rng.choice([4, 8, 16, 32]), rng.choice([64, 128]),
                        rng.choice([1, 1, 2, 4, 8]), N)
            if work(c)["bytes"] <= work(listed()[7])["bytes"]:
                return c
        elif kind == "ffn":
            block = rng.choice([256, 512, 1024, 2048])
            T = block * max(1, round(_log(rng, 1024, 16384) / block))
            dm = 256 * rng.randint(2, 16)
            c = _ffn(None, T, dm, 256 * max(1, round(dm * rng.uniform(2, 4) / 256)), block, rng.randrange(3))
            if work(c)["flops"] <= 1.5 * work(listed()[9])["flops"]:
                return c
        else:
            N, D = rng.choice([1, 2, 4, 8]), rng.choice([64, 128])
            H = rng.choice([4, 8, 12, 16, 20, 32])
            dm = H * D
            S = 256 * N * max(1, round(_log(rng, 1024, 16384) / (256 * N)))
            dff = 256 * round(dm * rng.uniform(2.5, 4) / 256)
            c = (_layer(None, S, dm, H, dff, N, rng.randrange(3)) if kind == "layer" else
                 _stack(None, rng.choice([1, 2]), S, dm, H, dff, N))
            if dm % 256 == 0 and work(c)["flops"] <= 0.6 * cap:
                return c


# ---------------------------------------------------------------------------------------
# Inputs: i.i.d. N(0, 1) activations, N(0, 0.02) weights, gains around 1
# ---------------------------------------------------------------------------------------
def _dtype(case):
    return torch.float32 if case.get("dtype") == "f32" else torch.bfloat16


class _Draw:
    def __init__(self, seed, dtype=torch.bfloat16):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))
        self.dtype = dtype

    def __call__(self, *shape, std=1.0, mean=0.0):
        x = torch.randn(*shape, generator=self.g, device="cuda", dtype=torch.float32)
        if std != 1.0:
            x.mul_(std)
        if mean != 0.0:
            x.add_(mean)
        return x.to(self.dtype)


def _f32(*shape):
    return torch.empty(*shape, dtype=torch.float32, device="cuda")


def prepare(case, seed):
    k = case["kind"]
    r = _Draw(seed, _dtype(case))
    if k == "attn":
        sh = (case["B"], case["S"], case["H"], case["D"])
        q, kk, v = r(*sh), r(*sh), r(*sh)
        return dict(case=case, q=q, k=kk, v=v, do=r(*sh) if case["train"] else None)
    if k == "host":
        c, H, D, N = case["c"], case["H"], case["D"], case["N"]
        q, kk, v, do = r(1, c, H, D), r(1, N * c, H, D), r(1, N * c, H, D), r(1, c, H, D)
        return dict(case=case, q=q, k=kk, v=v, do=do, o=torch.empty_like(q), lse=_f32(1, H, c),
                    dq=torch.empty_like(q), dk=_f32(1, N * c, H, D), dv=_f32(1, N * c, H, D))
    if k == "decode":
        B, S, H, D = case["B"], case["S"], case["H"], case["D"]
        return dict(case=case, q=r(B, case["Tq"], H, D), k=r(B, S, H, D), v=r(B, S, H, D))
    if k == "ffn":
        T, dm, dff = case["T"], case["dm"], case["dff"]
        x, w1, b1 = r(T, dm), r(dm, dff, std=0.02), r(dff, std=0.02)
        w2, b2, dy = r(dff, dm, std=0.02), r(dm, std=0.02), r(T, dm)
        return dict(case=case, x=x, w1=w1, b1=b1, w2=w2, b2=b2, dy=dy, y=torch.empty_like(x), dx=torch.empty_like(x),
                    dw1=_f32(dm, dff), db1=_f32(dff), dw2=_f32(dff, dm), db2=_f32(dm))
    if k == "layer":
        S, dm, dff = case["S"], case["dm"], case["dff"]
        x = r(S, dm)
        w = [r(dm, dm, std=0.02) for _ in range(4)] + [r(dm, dff, std=0.02), r(dff, dm, std=0.02)]
        return dict(case=case, x=x, w=w, dz=r(S, dm), z=torch.empty_like(x), dx=torch.empty_like(x),
                    dw=[_f32(*t.shape) for t in w])
    S, dm, dff = case["S"], case["dm"], case["dff"]
    x = r(S, dm)
    params = []
    for _ in range(case["L"]):
        g1 = r(dm, std=0.1, mean=1.0)
        wq, wk, wv, wo = (r(dm, dm, std=0.02) for _ in range(4))
        g2 = r(dm, std=0.1, mean=1.0)
        params.append([g1, wq, wk, wv, wo, g2, r(dm, dff, std=0.02), r(dm, dff, std=0.02), r(dff, dm, std=0.02)])
    return dict(case=case, x=x, params=params, dz=r(S, dm), z=torch.empty_like(x), dx=torch.empty_like(x),
                grads=[[_f32(*t.shape) for t in p] for p in params])


# ---------------------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------------------
def run(s):
    c = s["case"]
    k = c["kind"]
    if k == "attn":
        o, lse = ra.attention_fwd(s["q"], s["k"], s["v"], c["N"], c["causal"])
        if not c["train"]:
            return dict(o=o, lse=lse)
        dq, dk, dv = ra.attention_bwd(s["q"], s["k"], s["v"], o, lse, s["do"], c["N"], c["causal"])
        return dict(o=o, lse=lse, dq=dq, dk=dk, dv=dv)
    if k == "host":
        # the gradients the blocks carry when they reach this host: none yet
        s["dk"].zero_()
        s["dv"].zero_()
        ra.ring_attn_fwd_host(s["q"], s["k"], s["v"], s["o"], s["lse"], c["N"], c["host"], True)
        ra.ring_attn_bwd_host(s["q"], s["k"], s["v"], s["o"], s["lse"], s["do"], s["dq"], s["dk"], s["dv"], c["N"],
                              c["host"], True)
        return {n: s[n] for n in ("o", "lse", "dq", "dk", "dv")}
    if k == "decode":
        o, lse = ra.attention_decode(s["q"], s["k"], s["v"], c["N"], True)
        return dict(o=o, lse=lse)
    if k == "ffn":
        ra.blockwise_ffn(s["x"], s["w1"], s["b1"], s["w2"], s["b2"], s["y"], c["block"], c["act"])
        ra.blockwise_ffn_bwd(s["x"], s["w1"], s["b1"], s["w2"], s["dy"], s["dx"], s["dw1"], s["db1"], s["dw2"],
                             s["db2"], c["block"], c["act"])
        return {n: s[n] for n in ("y", "dx", "dw1", "db1", "dw2", "db2")}
    if k == "layer":
        ra.ring_layer_fwd(s["x"], *s["w"], s["z"], c["H"], c["N"], True, c["act"])
        ra.ring_layer_bwd(s["x"], *s["w"], s["dz"], s["dx"], *s["dw"], c["H"], c["N"], True, c["act"])
        return dict(z=s["z"], dx=s["dx"], dw=s["dw"])
    ra.llama_stack_train_step(s["x"], s["params"], s["dz"], s["z"], s["dx"], s["grads"], c["H"], c["N"], True)
    return dict(z=s["z"], dx=s["dx"], grads=s["grads"])


# ---------------------------------------------------------------------------------------
# Work the pass cannot do without: attention forward 4 D flops per visible pair, backward
# 10 D (five contractions); a matrix product 2 flops per multiply-add, its backward twice
# that; inputs read once, outputs written once.
# ---------------------------------------------------------------------------------------
def _pairs(S, causal):
    return S * (S + 1) / 2 if causal else S * S


def work(case):
    k = case["kind"]
    if k == "attn":
        e = 4 if case["dtype"] == "f32" else 2
        n = case["B"] * case["S"] * case["H"]
        p = case["B"] * case["H"] * _pairs(case["S"], case["causal"])
        fl, by = 4.0 * case["D"] * p, 4 * n * case["D"] * e + 4 * n
        if case["train"]:
            fl += 10.0 * case["D"] * p
            by += 4 * n * case["D"] * e
        return dict(bytes=by, flops=fl)
    if k == "host":
        c, H, D, i = case["c"], case["H"], case["D"], case["host"]
        p = H * (i * c * c + _pairs(c, True))
        seen = (i + 1) * c * H * D  # elements of the keys this host sees
        return dict(bytes=4 * c * H * D * 2 + 4 * H * c + 2 * seen * 2 + 2 * seen * 8, flops=14.0 * D * p)
    if k == "decode":
        B, S, H, D, Tq = case["B"], case["S"], case["H"], case["D"], case["Tq"]
        return dict(bytes=2 * B * S * H * D * 2 + 2 * B * Tq * H * D * 2 + 4 * B * H * Tq,
                    flops=4.0 * D * B * H * (Tq * S - Tq * (Tq - 1) / 2))
    if k == "ffn":
        T, dm, dff = case["T"], case["dm"], case["dff"]
        return dict(bytes=2 * (4 * T * dm + 2 * dm * dff + dff + dm) + 4 * (2 * dm * dff + dff + dm),
                    flops=3 * 4.0 * T * dm * dff)
    S, dm, dff, H = case["S"], case["dm"], case["dff"], case["H"]
    L = case.get("L", 1)
    w = 4 * dm * dm + (2 if k == "layer" else 3) * dm * dff
    att = 14.0 * dm * _pairs(S, True)
    return dict(bytes=2 * 4 * S * dm + 6 * L * w, flops=L * (6.0 * S * w + att))


def tolerance(case):
    """Relative 2-norm error between two correct implementations: float32 sums in another
    order, or bf16 probabilities, activations and outputs rounded from them (a layer's
    gradients pass through several such roundings).  Measured against exact(): float32
    attention up to 8e-7; bf16 attention 2.5e-3; feed-forward network 2.4e-3; one layer
    5e-3, with ReLU up to 3e-2 in dW1 (its derivative jumps where a rounded activation changes
    sign); two LLaMA-style layers 1.1e-2."""
    k = case["kind"]
    if case.get("dtype") == "f32":
        return dict(rel=4e-6, max=1e-3)
    if k in ("attn", "host", "decode", "ffn"):
        return dict(rel=1e-2)
    return dict(rel=3e-2 if case.get("act") == 1 else 2e-2)


# ---------------------------------------------------------------------------------------
# The same outputs in float64, plain torch
# ---------------------------------------------------------------------------------------
def _attn64(q, k, v, do, causal, q_pos0=0, chunk=2048):
    """float64 [B, Sq, H, D] attention, lse [B, H, Sq] and, with do, dq, dk, dv."""
    B, Sq, H, D = q.shape
    S = k.shape[1]
    o = torch.zeros_like(q)
    lse = torch.zeros((B, H, Sq), dtype=torch.float64, device=q.device)
    grads = None if do is None else (torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v))
    pos_k = torch.arange(S, device=q.device)
    for b in range(B):
        for h in range(H):
            kh, vh = k[b, :, h].contiguous(), v[b, :, h].contiguous()
            for r in range(0, Sq, chunk):
                e = min(Sq, r + chunk)
                n = min(S, q_pos0 + e) if causal else S
                s = (q[b, r:e, h] @ kh[:n].t()) / math.sqrt(D)
                if causal:
                    pos_q = torch.arange(q_pos0 + r, q_pos0 + e, device=q.device)
                    lo = q_pos0 + r  # keys up to here are visible to every row of the chunk
                    s[:, lo:].masked_fill_(pos_k[None, lo:n] > pos_q[:, None], -math.inf)
                m = s.max(dim=1, keepdim=True).values
                s.sub_(m).exp_()
                l = s.sum(dim=1, keepdim=True)
                s.div_(l)
                lse[b, h, r:e] = (m + l.log())[:, 0]
                oh = s @ vh[:n]
                o[b, r:e, h] = oh
                if do is not None:
                    g = do[b, r:e, h].contiguous()
                    grads[2][b, :n, h] += s.t() @ g
                    ds = g @ vh[:n].t()
                    ds.sub_((g * oh).sum(dim=1, keepdim=True)).mul_(s).mul_(1.0 / math.sqrt(D))
                    grads[0][b, r:e, h] = ds @ kh[:n]
                    grads[1][b, :n, h] += ds.t() @ q[b, r:e, h]
                    del ds
                del s
    return (o, lse) if do is None else (o, lse) + grads


def _act64(h, act):
    """act(h), act'(h)"""
    if act == 1:
        return h.clamp(min=0), (h > 0).to(h.dtype)
    if act == 2:
        a = math.sqrt(2 / math.pi)
        t = torch.tanh(a * (h + 0.044715 * h ** 3))
        return 0.5 * h * (1 + t), 0.5 * (1 + t) + 0.5 * h * (1 - t * t) * a * (1 + 3 * 0.044715 * h * h)
    cdf = 0.5 * (1 + torch.erf(h / math.sqrt(2)))
    return h * cdf, cdf + h * torch.exp(-0.5 * h * h) / math.sqrt(2 * math.pi)


def _ffn64(x, w1, b1, w2, b2, dy, act, chunk=4096):
    """y, dx, dw1, db1, dw2, db2 of the feed-forward network."""
    y, dx = torch.zeros_like(x), torch.zeros_like(x)
    dw1, dw2 = torch.zeros_like(w1), torch.zeros_like(w2)
    db1 = torch.zeros(w1.shape[1], dtype=x.dtype, device=x.device)
    for r in range(0, x.shape[0], chunk):
        xs, g = x[r:r + chunk], dy[r:r + chunk]
        h = xs @ w1
        if b1 is not None:
            h += b1
        a, da = _act64(h, act)
        y[r:r + chunk] = a @ w2 + (0 if b2 is None else b2)
        dh = (g @ w2.t()) * da
        dx[r:r + chunk] = dh @ w1.t()
        dw1 += xs.t() @ dh
        dw2 += a.t() @ g
        db1 += dh.sum(0)
    return y, dx, dw1, db1, dw2, dy.sum(0)


def _layer64(x, w, dz, H, act):
    wq, wk, wv, wo, w1, w2 = w
    S, dm = x.shape
    sh = (1, S, H, dm // H)
    q, k, v = (x @ m for m in (wq, wk, wv))
    o, _ = _attn64(q.view(sh), k.view(sh), v.view(sh), None, True)
    o = o.view(S, dm)
    y = x + o @ wo
    f, dyf, dw1, _, dw2, _ = _ffn64(y, w1, None, w2, None, dz, act)
    dy = dz + dyf
    dwo = o.t() @ dy
    do = dy @ wo.t()
    _, _, dq, dk, dv = _attn64(q.view(sh), k.view(sh), v.view(sh), do.view(sh), True)
    dq, dk, dv = (t.view(S, dm) for t in (dq, dk, dv))
    dx = dy + dq @ wq.t() + dk @ wk.t() + dv @ wv.t()
    return y + f, dx, [x.t() @ dq, x.t() @ dk, x.t() @ dv, dwo, dw1, dw2]


def _norm64(x, g):
    r = torch.rsqrt((x * x).mean(dim=1, keepdim=True) + 1e-6)
    return x * r * g, r


def _norm64_bwd(x, g, r, dy):
    """dx, dg"""
    gd = g * dy
    return r * gd - x * r ** 3 * (gd * x).mean(dim=1, keepdim=True), (dy * x * r).sum(0)


def _rope64(x, H, sign):
    S, dm = x.shape
    D = dm // H
    p = torch.arange(S, device=x.device, dtype=torch.float64)
    f = 10000.0 ** (-2.0 * torch.arange(D // 2, device=x.device, dtype=torch.float64) / D)
    a = p[:, None] * f[None, :]
    c, s = a.cos()[:, None, :], sign * a.sin()[:, None, :]
    v = x.view(S, H, D // 2, 2)
    return torch.stack((v[..., 0] * c - v[..., 1] * s, v[..., 0] * s + v[..., 1] * c), dim=-1).reshape(S, dm)


def _llama64_fwd(x, p, H, chunk=4096):
    g1, wq, wk, wv, wo, g2, w1, w3, w2 = p
    S, dm = x.shape
    sh = (1, S, H, dm // H)
    n1, r1 = _norm64(x, g1)
    q, k, v = _rope64(n1 @ wq, H, 1.0), _rope64(n1 @ wk, H, 1.0), n1 @ wv
    o, _ = _attn64(q.view(sh), k.view(sh), v.view(sh), None, True)
    o = o.view(S, dm)
    h = x + o @ wo
    n2, r2 = _norm64(h, g2)
    z = torch.empty_like(h)
    for r in range(0, S, chunk):
        u = n2[r:r + chunk] @ w1
        z[r:r + chunk] = h[r:r + chunk] + (u * torch.sigmoid(u) * (n2[r:r + chunk] @ w3)) @ w2
    return z, (n1, r1, q, k, v, o, h, n2, r2)


def _llama64_bwd(x, p, dz, H, chunk=4096):
    g1, wq, wk, wv, wo, g2, w1, w3, w2 = p
    S, dm = x.shape
    sh = (1, S, H, dm // H)
    _, (n1, r1, q, k, v, o, h, n2, r2) = _llama64_fwd(x, p, H)
    dn2 = torch.empty_like(x)
    dw1, dw3, dw2 = torch.zeros_like(w1), torch.zeros_like(w3), torch.zeros_like(w2)
    for r in range(0, S, chunk):
        ns, g = n2[r:r + chunk], dz[r:r + chunk]
        u, w = ns @ w1, ns @ w3
        sg = torch.sigmoid(u)
        dw2 += (u * sg * w).t() @ g
        dg = g @ w2.t()
        dw, du = dg * u * sg, dg * w * sg * (1 + u * (1 - sg))
        dw1 += ns.t() @ du
        dw3 += ns.t() @ dw
        dn2[r:r + chunk] = du @ w1.t() + dw @ w3.t()
    dh, dg2 = _norm64_bwd(h, g2, r2, dn2)
    dh = dh + dz
    dwo = o.t() @ dh
    do = dh @ wo.t()
    _, _, dq, dk, dv = _attn64(q.view(sh), k.view(sh), v.view(sh), do.view(sh), True)
    dq, dk, dv = _rope64(dq.view(S, dm), H, -1.0), _rope64(dk.view(S, dm), H, -1.0), dv.view(S, dm)
    dx, dg1 = _norm64_bwd(x, g1, r1, dq @ wq.t() + dk @ wk.t() + dv @ wv.t())
    return dx + dh, [dg1, n1.t() @ dq, n1.t() @ dk, n1.t() @ dv, dwo, dg2, dw1, dw3, dw2]


def exact(case, seed):
    k = case["kind"]
    s = prepare(case, seed)
    d = lambda t: t if t is None else t.double()
    if k == "attn":
        r = _attn64(d(s["q"]), d(s["k"]), d(s["v"]), d(s["do"]), case["causal"])
        return dict(zip(("o", "lse", "dq", "dk", "dv"), r))
    if k == "host":
        r = _attn64(d(s["q"]), d(s["k"]), d(s["v"]), d(s["do"]), True, q_pos0=case["host"] * case["c"])
        return dict(zip(("o", "lse", "dq", "dk", "dv"), r))
    if k == "decode":
        B, Tq, H, D = s["q"].shape
        S = case["S"]
        o = torch.empty((B, Tq, H, D), dtype=torch.float64, device="cuda")
        lse = torch.empty((B, H, Tq), dtype=torch.float64, device="cuda")
        for h in range(H):  # one head at a time: the cache in float64 is large
            oh, lh = _attn64(d(s["q"][:, :, h:h + 1]), d(s["k"][:, :, h:h + 1]), d(s["v"][:, :, h:h + 1]), None, True,
                             q_pos0=S - Tq)
            o[:, :, h:h + 1], lse[:, h:h + 1] = oh, lh
        return dict(o=o, lse=lse)
    if k == "ffn":
        r = _ffn64(d(s["x"]), d(s["w1"]), d(s["b1"]), d(s["w2"]), d(s["b2"]), d(s["dy"]), case["act"])
        return dict(zip(("y", "dx", "dw1", "db1", "dw2", "db2"), r))
    if k == "layer":
        z, dx, dw = _layer64(d(s["x"]), [d(t) for t in s["w"]], d(s["dz"]), case["H"], case["act"])
        return dict(z=z, dx=dx, dw=dw)
    params = [[d(t) for t in p] for p in s["params"]]
    acts = [d(s["x"])]
    for p in params:
        acts.append(_llama64_fwd(acts[-1], p, case["H"])[0])
    g, grads = d(s["dz"]), [None] * len(params)
    for l in reversed(range(len(params))):
        g, grads[l] = _llama64_bwd(acts[l], params[l], g, case["H"])
    return dict(z=acts[-1], dx=g, grads=grads)
