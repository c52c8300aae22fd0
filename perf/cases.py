"""Workloads of the Mixture Compressor expert path, for timing and checking.

Each case is one call (or one short sequence of calls) that a serving or a
compression program makes through the package's public entry points, at the
sizes of the layers the repository is written for (the Mixtral-8x7B-shaped and
OLMoE-shaped MoE layers and the tiny layer of the tests) and, for drawn cases,
at generic sizes of the same ranges:

* ``layer``       route + prune + expert forward of one MoE layer: the call of
                  every serving step, decode (few tokens) to prefill (many);
* ``stack``       the expert half of a whole decoder: one call, n layers;
* ``importance``  the protected set of a prompt, from its attention maps;
* ``router``      the router's linear layer ahead of routing;
* ``pack``        quantizing and packing a whole layer of fp32 experts;
* ``gptq``        GPTQ of one expert matrix: Hessian, factor, quantization.

``listed()`` gives the named cases, ``draw(rng)`` one more of the same ranges;
``prepare`` / ``run`` / ``work`` / ``tolerance`` / ``exact`` take a case.
"""
from __future__ import annotations

import math

import torch

import paper_2410_06270_amd as mc

# Expert widths: the 2.5-bit Mixtral allocation, and an allocation drawn with
# probabilities 0.2 / 0.5 / 0.3 for 1 / 2 / 3 bits over 64 experts.
_MIXTRAL = dict(d=4096, ffn=14336, E=8, k=2, G=128, bits="33322223", skew="bias")
_OLMOE = dict(d=2048, ffn=1024, E=64, k=8, G=64, skew="zipf",
              bits="3322232212311233111222222331332323222232222312221222232233131231")
_TINY = dict(d=256, ffn=512, E=4, k=2, G=32, bits="1232", skew="none")


def _layer(name, shape, T, tau):
    return dict(name=name, kind="layer", T=T, tau=tau, **shape)


def listed():
    return [
        # the smallest call: a toy layer, all launch latency
        _layer("layer_tiny_64", _TINY, 64, 0.3),
        # interactive decoding of one sequence
        _layer("decode_mixtral_1", _MIXTRAL, 1, 0.3),
        # batched decoding, the headline workload
        _layer("decode_mixtral_32", _MIXTRAL, 32, 0.3),
        # batched decoding over many small experts
        _layer("decode_olmoe_16", _OLMOE, 16, 0.05),
        # a short prompt (or a prompt chunk beside running decodes), ragged
        _layer("prefill_mixtral_333", _MIXTRAL, 333, 0.3),
        # a long prompt
        _layer("prefill_mixtral_4096", _MIXTRAL, 4096, 0.2),
        # a long prompt over many small experts, skewed routing
        _layer("prefill_olmoe_2048", _OLMOE, 2048, 0.05),
        # the expert half of a whole 32-layer decoder, one decode step of 64 sequences
        dict(name="stack_mixtral_64", kind="stack", layers=32, T=64, tau=0.3, **_MIXTRAL),
        # protecting the important tokens of a long prompt
        dict(name="importance_4096", kind="importance", H=32, L=4096, d=4096, rho=0.02),
        # the router ahead of a long prompt's routing
        dict(name="router_mixtral_4096", kind="router", T=4096, d=4096, E=8),
        # compressing a layer by rounding to nearest
        dict(name="pack_mixtral", kind="pack", **_MIXTRAL),
        # compressing one expert matrix (gate) with GPTQ, 8192 calibration rows
        dict(name="gptq_mixtral_gate", kind="gptq", R=14336, K=4096, N=8192, G=128, b=3),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _log_mult(rng, lo, hi, m):
    return m * max(1, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / m)))


def _draw_shape(rng):
    """A layer's shape: one of the three above, or a generic one (d and ffn any
    multiples of 128) with no more weights than the largest of them."""
    pick = rng.randrange(5)
    if pick < 3:
        return dict([_MIXTRAL, _OLMOE, _TINY][pick])
    while True:
        d, ffn = _log_mult(rng, 256, 4096, 128), _log_mult(rng, 512, 14336, 128)
        E = rng.choice([4, 8, 16, 24, 60, 64])
        if E * d * ffn <= 8 * 4096 * 14336:
            break
    k = min(rng.choice([1, 2, 2, 4, 8]), E)
    bits = "".join(rng.choice("1222233") for _ in range(E))
    return dict(d=d, ffn=ffn, E=E, k=k, G=rng.choice([32, 64, 128]), bits=bits,
                skew=rng.choice(["none", "bias", "zipf"]))


def draw(rng):
    kind = rng.choice(["layer"] * 6 + ["stack", "importance", "router", "pack", "gptq"])
    if kind == "layer":
        s = _draw_shape(rng)
        top = min(4096.0, 4096 * 2 * 4096 * 14336 / (s["k"] * s["d"] * s["ffn"]))
        T = _log_int(rng, 1, top) if rng.random() < 0.5 else _log_int(rng, 1, 128)
        tau = rng.choice([0.0, 0.2, 0.3]) if s["k"] <= 2 else rng.choice([0.0, 0.05, 0.1])
        return dict(kind=kind, T=T, tau=tau, **s)
    if kind == "stack":
        n = rng.randint(2, 32)
        s = _draw_shape(rng)
        T = _log_int(rng, 1, 64)
        return dict(kind=kind, layers=n, T=T, tau=0.3 if s["k"] <= 2 else 0.05, **s)
    if kind == "importance":
        return dict(kind=kind, H=rng.randint(4, 32), L=_log_int(rng, 100, 4096), d=_log_mult(rng, 256, 4096, 128),
                    rho=rng.choice([0.02, 0.1]))
    if kind == "router":
        return dict(kind=kind, T=_log_int(rng, 1, 4096), d=_log_mult(rng, 256, 4096, 128), E=rng.choice([4, 8, 8, 16]))
    if kind == "pack":
        return dict(kind=kind, **_draw_shape(rng))
    return dict(kind="gptq", R=_log_mult(rng, 512, 14336, 128), K=_log_mult(rng, 256, 4096, 128),
                N=_log_int(rng, 256, 8192), G=rng.choice([32, 64, 128]), b=rng.choice([1, 2, 3]))


# ------------------------------------------------------------------ inputs --
def _gen(seed, stream):
    return torch.Generator(device="cuda").manual_seed((1000003 * (seed + 1) + 7919 * stream) % (2 ** 62))


def _randn(shape, seed, stream, dtype=torch.float32):
    return torch.randn(shape, generator=_gen(seed, stream), device="cuda", dtype=dtype)


def _widths(case):
    return [int(c) for c in case["bits"]]


def _weights(case, seed, layer=0):
    """fp32 N(0, 0.02^2): gate and up [E][ffn][d], down [E][d][ffn]."""
    E, d, ffn = case["E"], case["d"], case["ffn"]
    return [_randn(s, seed, 1000 * (layer + 1) + m).mul_(0.02)
            for m, s in enumerate([(E, ffn, d), (E, ffn, d), (E, d, ffn)])]


def _logits(case, seed, layer=0):
    """N(0, 1) scores, plus a per-expert offset: N(0, 0.5^2), the logarithm of
    a Zipf(1.1) popularity over a random order of the experts, or none."""
    E, T, st = case["E"], case["T"], 1000 * (layer + 1)
    lg = _randn((T, E), seed, st + 10)
    if case["skew"] == "bias":
        lg += 0.5 * _randn((E,), seed, st + 11)
    elif case["skew"] == "zipf":
        perm = torch.randperm(E, generator=_gen(seed, st + 12), device="cuda")
        p = torch.arange(1, E + 1, device="cuda", dtype=torch.float64) ** -1.1
        lg += (p / p.sum())[perm].log().float()
    return lg


def _protected(case, seed, layer=0):
    """A tenth of the tokens (none below 5 tokens) are marked important."""
    T = case["T"]
    m = torch.zeros(T, dtype=torch.uint8, device="cuda")
    perm = torch.randperm(T, generator=_gen(seed, 1000 * (layer + 1) + 13), device="cuda")
    m[perm[:int(0.1 * T + 0.5)]] = 1
    return m


def _tokens(case, seed, n="T"):
    return _randn((case[n], case["d"]), seed, 1).to(torch.bfloat16)


def _packed(case, seed, layer=0):
    L = mc.PackedLayer(case["E"], case["d"], case["ffn"], _widths(case), case["G"])
    w = _weights(case, seed, layer)
    mc.pack(*w, L)
    return L


def _attention(case, seed):
    """Causal softmaxes of N(0, 1.5^2) scores with +4 on the first key (the
    attention sink real maps show), bf16 [H][L][L]."""
    H, L = case["H"], case["L"]
    out = torch.empty((H, L, L), dtype=torch.bfloat16, device="cuda")
    above = torch.ones((L, L), dtype=torch.bool, device="cuda").triu_(1)
    for h in range(H):
        s = _randn((L, L), seed, 50 + h).mul_(1.5)
        s[:, 0] += 4.0
        s.masked_fill_(above, float("-inf"))
        out[h] = torch.softmax(s, dim=1).to(torch.bfloat16)
    return out


def _router_weight(case, seed):
    return (_randn((case["E"], case["d"]), seed, 2) / math.sqrt(case["d"])).to(torch.bfloat16)


def _calibration(case, seed):
    """Correlated, outlier-heavy layer inputs: rank-8 factors plus noise, channel
    scales exp(N(0, 0.5^2)), 1 % of the channels times 8; bf16 [N][K]."""
    N, K = case["N"], case["K"]
    x = _randn((N, 8), seed, 3) @ _randn((8, K), seed, 4) / math.sqrt(8) + 0.5 * _randn((N, K), seed, 5)
    scale = torch.exp(0.5 * _randn((K,), seed, 6))
    scale[torch.randperm(K, generator=_gen(seed, 7), device="cuda")[:max(1, K // 100)]] *= 8.0
    return (x * scale).to(torch.bfloat16)


def _matrix(case, seed):
    return _randn((case["R"], case["K"]), seed, 8).mul_(0.02)


# ----------------------------------------------------------------- prepare --
def prepare(case, seed):
    kind = case["kind"]
    u8 = dict(dtype=torch.uint8, device="cuda")
    st = dict(case=case)
    if kind == "layer":
        T, E, k, d, ffn = (case[n] for n in ("T", "E", "k", "d", "ffn"))
        st.update(x=_tokens(case, seed), logits=_logits(case, seed), important=_protected(case, seed),
                  routing=mc.Routing(T, E, k), layer=_packed(case, seed),
                  y=torch.zeros((T, d), dtype=torch.bfloat16, device="cuda"),
                  ws=torch.empty(mc.forward_workspace(T, E, k, d, ffn), **u8))
    elif kind == "stack":
        T, E, k, d, ffn, n = (case[m] for m in ("T", "E", "k", "d", "ffn", "layers"))
        st.update(x=_tokens(case, seed), layers=[_packed(case, seed, l) for l in range(n)],
                  logits=torch.stack([_logits(case, seed, l) for l in range(n)]),
                  important=torch.stack([_protected(case, seed, l) for l in range(n)]),
                  routing=mc.Routing(T, E, k), y=torch.zeros((T, d), dtype=torch.bfloat16, device="cuda"),
                  tmp=torch.zeros((T, d), dtype=torch.bfloat16, device="cuda"),
                  ws=torch.empty(mc.stack_workspace(T, E, k, d, ffn), **u8))
    elif kind == "importance":
        H, L = case["H"], case["L"]
        st.update(attn=_attention(case, seed), x=_tokens(case, seed, "L"), important=torch.zeros(L, **u8),
                  importance=torch.zeros(L, dtype=torch.float32, device="cuda"),
                  ws=torch.empty(mc.importance_workspace(H, L), **u8))
    elif kind == "router":
        st.update(x=_tokens(case, seed), w=_router_weight(case, seed),
                  logits=torch.zeros((case["T"], case["E"]), dtype=torch.float32, device="cuda"))
    elif kind == "pack":
        st.update(w=_weights(case, seed),
                  layer=mc.PackedLayer(case["E"], case["d"], case["ffn"], _widths(case), case["G"]))
    else:
        R, K = case["R"], case["K"]
        L = mc.PackedLayer(1, K, R, [case["b"]], case["G"])
        L.words.zero_()
        L.sz.zero_()
        f64 = dict(dtype=torch.float64, device="cuda")
        st.update(x=_calibration(case, seed), w=_matrix(case, seed), layer=L, H=torch.empty((K, K), **f64),
                  U=torch.empty((K, K), **f64), dead=torch.empty(K, **u8), loss=torch.empty(R, **f64),
                  ws=torch.empty(mc.gptq_workspace(R, K), **u8))
    return st


# --------------------------------------------------------------------- run --
def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "layer":
        r = st["routing"]
        mc.route_forward(st["x"], st["logits"], st["important"], case["tau"], r, st["layer"], st["y"], st["ws"])
        return dict(y=st["y"], topk_idx=r.topk_idx, topk_w=r.topk_w, kept=r.kept)
    if kind == "stack":
        mc.stack_forward(st["x"], st["layers"], st["logits"], st["important"], case["tau"], st["routing"],
                         st["y"], st["tmp"], st["ws"])
        return st["y"]
    if kind == "importance":
        mc.token_importance(st["attn"], st["x"], case["rho"], st["important"], st["ws"], st["importance"])
        return dict(importance=st["importance"], important=st["important"])
    if kind == "router":
        mc.router_logits(st["x"], st["w"], st["logits"])
        return st["logits"]
    if kind == "pack":
        mc.pack(*st["w"], st["layer"])
        return dict(words=st["layer"].words, sz=st["layer"].sz)
    mc.gptq_hessian(st["x"], st["H"])
    mc.gptq_factor(st["H"], st["U"], st["dead"], st["ws"])
    mc.gptq_quantize(st["layer"], 0, 0, st["w"], st["U"], st["dead"], st["ws"], st["loss"])
    n = case["R"] * case["K"]
    return dict(H=st["H"], U=st["U"], words=st["layer"].words[:n * case["b"] // 32],
                sz=st["layer"].sz[:n // case["G"]], loss=st["loss"])


# -------------------------------------------------------------------- work --
def _layer_work(case):
    T, E, k, d, ffn, G = (case[n] for n in ("T", "E", "k", "d", "ffn", "G"))
    bits = _widths(case)
    touched = E * (1.0 - (1.0 - k / E) ** T)        # experts some token selects (even routing)
    weights = touched * 3 * d * ffn * (sum(bits) / E / 8 + 4.0 / G)
    return weights, 6.0 * T * k * d * ffn


def work(case):
    kind = case["kind"]
    if kind in ("layer", "stack"):
        w, f = _layer_work(case)
        n = case.get("layers", 1)
        io = 4.0 * case["T"] * case["d"] + n * 4.0 * case["T"] * case["E"]
        return {"bytes": n * w + io, "flops": n * f}
    if kind == "importance":
        H, L, d = case["H"], case["L"], case["d"]
        return {"bytes": H * L * (L + 1.0) + 2.0 * L * d + 5.0 * L, "flops": H * L * (L + 1.0) / 2 + L * d}
    if kind == "router":
        T, d, E = case["T"], case["d"], case["E"]
        return {"bytes": 2.0 * T * d + 2.0 * E * d + 4.0 * T * E, "flops": 2.0 * T * d * E}
    if kind == "pack":
        n = 3.0 * case["d"] * case["ffn"]
        return {"bytes": n * (case["E"] * (4 + 4.0 / case["G"]) + sum(_widths(case)) / 8),
                "flops": n * case["E"] * 8}
    R, K, N = case["R"], case["K"], case["N"]
    # H, the Cholesky factor of its inverse, one multiply-subtract per (row, column pair)
    return {"bytes": 2.0 * N * K + 16.0 * K * K + 4.0 * R * K + R * K * (case["b"] / 8 + 4.0 / case["G"]) + 8.0 * R,
            "flops": 1.0 * N * K * K + 2.0 * K ** 3 / 3 + 1.0 * R * K * K}


# --------------------------------------------------------------- tolerance --
def tolerance(case):
    """About four times what the path shows against exact()."""
    kind = case["kind"]
    if kind == "layer":                 # one bf16 rounding of y: rel 1.7e-3, max 5e-3
        return {"rel": 7e-3, "max": 2e-2, "differ": 1e-3}
    if kind == "stack":                 # a bf16 rounding of h and of its norm per layer: 2.2e-2, 0.11
        return {"rel": 8e-2, "max": 4e-1}
    if kind == "importance":            # fp32 sums: 1.2e-7, 1.7e-7
        return {"rel": 5e-7, "max": 1e-6, "differ": 1e-3}
    if kind == "router":                # fp64 sums, one fp32 rounding: 2.5e-8, 6e-8
        return {"rel": 1e-7, "max": 2.5e-7}
    if kind == "pack":
        return "exact"
    # fp64 throughout; U 6e-14, 1.4e-12.  A code flips only where its weight
    # sits within that of a midpoint, and then changes the rest of its row.
    return {"rel": 1e-11, "max": 1e-8, "differ": 1e-4}


# ------------------------------------------------------------------- exact --
def _group_params(w, b, G):
    """Scale and zero of every group of G columns (fp16 values, as fp64 [R][K/G][1])."""
    g = w.view(w.shape[0], -1, G)
    mn, mx = g.amin(2, keepdim=True), g.amax(2, keepdim=True)
    # in fp64 and rounded to fp32: the same as one fp32 division (53 >= 2 * 24 + 2 bits)
    s = ((mx - mn).double() / ((1 << b) - 1)).float().clamp(max=65504.0).half()
    s = torch.where(s == 0, torch.ones_like(s), s)
    z = (-mn.double() / s.double()).float().clamp(-65504.0, 65504.0).half() + 0.0
    return s, z


def _codes(w, s, z, b, G):
    """The level s (q - z) nearest to each weight, ties to the even q."""
    g = w.view(w.shape[0], -1, G).double()
    sd, zd = s.double(), z.double()
    below = torch.zeros_like(g)
    for j in range((1 << b) - 1):
        below += (sd * (j + 0.5 - zd) < g)
    tie = (sd * (below + 0.5 - zd) == g) & (below % 2 == 1) & (below < (1 << b) - 1)
    return below + tie


def _dequantized(w, b, G):
    s, z = _group_params(w, b, G)
    return (s.double() * (_codes(w, s, z, b, G) - z.double())).view(w.shape)


def _exact_routing(case, seed, layer=0):
    """(topk_idx, weights fp64, kept) of every token."""
    lg = _logits(case, seed, layer)
    k, tau = case["k"], torch.tensor(case["tau"], dtype=torch.float32).double().item()
    val, idx = torch.sort(lg, dim=1, descending=True, stable=True)
    val, idx = val[:, :k].double(), idx[:, :k]
    ex = torch.exp(val - val[:, :1])
    keep = ~(ex < tau * ex.sum(1, keepdim=True)) | _protected(case, seed, layer).bool()[:, None]
    keep[:, 0] = True
    w = torch.where(keep, ex, torch.zeros_like(ex))
    return idx, w / w.sum(1, keepdim=True), keep


def _exact_layer(case, seed, x, layer=0):
    idx, w, keep = _exact_routing(case, seed, layer)
    mats = _weights(case, seed, layer)
    y = torch.zeros_like(x)
    for e, b in enumerate(_widths(case)):
        t, r = torch.nonzero((idx == e) & keep, as_tuple=True)
        if t.numel() == 0:
            continue
        gate, up, down = (_dequantized(m[e], b, case["G"]) for m in mats)
        xe = x[t]
        a = xe @ gate.t().contiguous()
        h = a * torch.sigmoid(a) * (xe @ up.t().contiguous())
        y.index_add_(0, t, w[t, r][:, None] * (h @ down.t().contiguous()))
    return y, idx, w, keep


def _packed_words(codes, b):
    """Codes [R][K] -> the packed 32-bit words: 16 x 128 tiles, lane
    l = n % 16 + 16 ((k % 32) / 8), code pairs at the same bit of both halves."""
    R, K = codes.shape
    c = codes.long().view(R // 16, 16, K // 128, 4, 4, 4, 2)      # [nt][n][kt][u][kq][j/2][half]
    c = c.permute(0, 2, 4, 1, 3, 5, 6).reshape(R // 16, K // 128, 64, 16, 2)   # [..][lane][pair][half]
    w = torch.zeros((R // 16, K // 128, 64, b), dtype=torch.int64, device=codes.device)
    for i in range(16):
        for h in range(2):
            q = c[..., i, h]
            if b == 1:
                w[..., 0] |= q << (16 * h + i)
            elif b == 2:
                w[..., i // 8] |= q << (16 * h + 2 * (i % 8))
            elif i < 15:
                w[..., i // 5] |= q << (16 * h + 3 * (i % 5))
            else:
                for p in range(3):
                    w[..., p] |= ((q >> p) & 1) << (16 * h + 15)
    return torch.where(w >= 2 ** 31, w - 2 ** 32, w).to(torch.int32).reshape(-1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "layer":
        y, idx, w, keep = _exact_layer(case, seed, _tokens(case, seed).double())
        return dict(y=y, topk_idx=idx.to(torch.int32), topk_w=w, kept=keep.to(torch.uint8))
    if kind == "stack":
        h = _tokens(case, seed).double()
        for l in range(case["layers"]):
            xn = h / torch.sqrt((h * h).mean(1, keepdim=True) + 1e-5)
            h = h + _exact_layer(case, seed, xn, l)[0]
        return h
    if kind == "importance":
        H, L = case["H"], case["L"]
        attn, x = _attention(case, seed), _tokens(case, seed, "L").double()
        cs = torch.zeros(L, dtype=torch.float64, device="cuda")
        for h in range(H):
            cs += attn[h].double().sum(0)
        seen = torch.arange(L, 0, -1, dtype=torch.float64, device="cuda")
        imp = x.abs().sum(1) * (cs / H) / seen
        n = int(math.floor(torch.tensor(case["rho"], dtype=torch.float32).double().item() * L + 0.5))
        mask = torch.zeros(L, dtype=torch.uint8, device="cuda")
        mask[torch.sort(imp, descending=True, stable=True)[1][:n]] = 1
        return dict(importance=imp, important=mask)
    if kind == "router":
        return _tokens(case, seed).double() @ _router_weight(case, seed).double().t().contiguous()
    if kind == "pack":
        words, szs = [], []
        mats = _weights(case, seed)
        for e, b in enumerate(_widths(case)):
            for m in mats:
                s, z = _group_params(m[e], b, case["G"])
                words.append(_packed_words(_codes(m[e], s, z, b, case["G"]).view(m[e].shape), b))
                word = (s.view(torch.int16).int() & 0xffff) | (z.view(torch.int16).int() << 16)
                szs.append(word.view(m.shape[1] // 16, 16, -1).permute(0, 2, 1).reshape(-1))
        return dict(words=torch.cat(words), sz=torch.cat(szs))
    K = case["K"]
    x = _calibration(case, seed).double()
    H = 2.0 * (x.t().contiguous() @ x)
    d = torch.diagonal(H)
    Hd = H + torch.diag((d == 0).double())
    Hd = Hd + torch.diag(torch.full((K,), 0.01 * float(torch.diagonal(Hd).mean()), dtype=torch.float64, device="cuda"))
    # H^-1 = U^T U with U upper: U = J L^-1 J for the lower factor L of J H J
    Lc = torch.linalg.cholesky(torch.flip(Hd, (0, 1)).cpu())
    U = torch.flip(torch.linalg.solve_triangular(Lc, torch.eye(K, dtype=torch.float64), upper=False), (0, 1))
    return dict(H=H, U=U.cuda(), words=None, sz=None, loss=None)
