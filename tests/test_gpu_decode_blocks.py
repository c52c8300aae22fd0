"""The decode GEMVs on experts with more pairs than a work item holds (17 to 47:
two and three items, the last one full or a single pair), at every group size,
by ordinary and by non-temporal loads, on 8- and 16-wave workgroups, with a
split gate/up reduction, and on routing buffers that hold garbage.  The layers
are large enough that their batches keep the GEMVs (checked: the GEMMs'
preparation must not have run).  The reference is fp64 torch on the packed
layer's own codes and scale/zero words."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BITS = [3, 3, 2, 1, 3, 2, 2, 3]
# (E, d, ffn): weights read by ordinary loads (under 384 MB) and by non-temporal
# ones (Mixtral-sized: 463 MB at G = 128 and more for smaller groups), and a d
# whose 36 chunks need two splits of the gate/up reduction
ORDINARY = (8, 2048, 7168)
STREAMED = (8, 4096, 14336)
SPLIT = (4, 4608, 8192)


@pytest.fixture(scope="module")
def layer():
    """layer(shape, G) -> the packed layer, made once in a row."""
    import paper_2410_06270_amd as mc
    made = {}

    def get(shape, G):
        if (shape, G) not in made:
            made.clear()
            torch.cuda.empty_cache()
            E, d, ffn = shape
            g = torch.Generator(device="cuda").manual_seed(d + G)
            L = mc.PackedLayer(E, d, ffn, [BITS[e % len(BITS)] for e in range(E)], G)
            mc.pack(*(torch.randn(s, generator=g, device="cuda").mul_(0.02)
                      for s in ((E, ffn, d), (E, ffn, d), (E, d, ffn))), L)
            torch.cuda.synchronize()
            made[(shape, G)] = L
        return made[(shape, G)]
    return get


def dense(L, e, m, G):
    """Matrix m of expert e as fp64 [R][K], s (q - z) exactly."""
    import paper_2410_06270_amd as mc
    R, K = (L.ffn, L.d) if m < 2 else (L.d, L.ffn)
    codes = torch.empty((R, K), dtype=torch.uint8, device="cuda")
    mc.codes_export(L, e, m, codes)
    n = L.d * L.ffn // G
    sz = L.sz.view(torch.int32)[(3 * e + m) * n:(3 * e + m + 1) * n].view(R // 16, K // G, 16).permute(0, 2, 1)
    half = sz.contiguous().view(torch.float16).view(R, K // G, 1, 2).double()
    return (half[..., 0] * (codes.view(R, K // G, G).double() - half[..., 1])).view(R, K)


def reference(L, G, x, top, w):
    """Eq. 1 in fp64: x [T][d], top and w [T][k]."""
    y = torch.zeros_like(x)
    for e in range(L.E):
        t, r = torch.nonzero(top == e, as_tuple=True)
        if t.numel() == 0:
            continue
        a = x[t] @ dense(L, e, 0, G).t().contiguous()
        h = a * torch.sigmoid(a) * (x[t] @ dense(L, e, 1, G).t().contiguous())
        y.index_add_(0, t, w[t, r][:, None] * (h @ dense(L, e, 2, G).t().contiguous()))
    return y


def skewed_logits(T, E, k, second, g):
    """Every token selects expert 0 first, the first `second` of them expert 1
    next, the others one of the rest; noise decides further ranks."""
    lg = torch.randn((T, E), generator=g, device="cuda")
    t = torch.arange(T, device="cuda")
    lg[:, 0] += 40.0
    lg[t, torch.where(t < second, 1, 2 + t % (E - 2))] += 39.0
    return lg


def forward(mc, L, r, x, T, k, gemvs=True):
    """mc_moe_forward on a batch that must take the GEMVs (or the GEMMs); NaN
    where not written."""
    y = torch.full((T, L.d), 0x7FC1, dtype=torch.int16, device="cuda")
    ws = torch.empty(mc.forward_workspace(T, L.E, k, L.d, L.ffn), dtype=torch.uint8, device="cuda")
    mc.timing_enable(True)
    try:
        mc.moe_forward(x.view(torch.int16), r, L, y, ws)
        torch.cuda.synchronize()
        assert mc.timing_read("gateup")[1] == 1
        assert mc.timing_read("prefill_prep")[1] == (0 if gemvs else 1)
    finally:
        mc.timing_enable(False)
    return y


@pytest.mark.parametrize("shape,T,k,second,counts", [
    (ORDINARY, 17, 2, 17, (17, 17)),      # a full item and one of a single pair
    (ORDINARY, 32, 2, 16, (32, 16)),      # two full items; one
    (ORDINARY, 47, 2, 33, (47, 33)),      # three items, the last of 15 pairs and of one
    (STREAMED, 4, 4, 4, None),            # 8-wave workgroups for gate/up and down
    (STREAMED, 8, 4, 4, None),            # 16-wave ones for down
    (STREAMED, 17, 2, 17, (17, 17)),
    (STREAMED, 47, 2, 33, (47, 33)),
    (STREAMED, 52, 2, 20, (52, 20)),      # streamed layers keep the GEMVs up to 14 pairs an expert
    (SPLIT, 17, 2, 17, (17, 17)),
])
@pytest.mark.parametrize("G", [32, 64, 128])
def test_gemv_blocks(layer, G, shape, T, k, second, counts):
    import paper_2410_06270_amd as mc
    L = layer(shape, G)
    g = torch.Generator(device="cuda").manual_seed(T + G)
    x = torch.randn((T, L.d), generator=g, device="cuda").to(torch.bfloat16)
    lg = skewed_logits(T, L.E, k, second, g)
    r = mc.Routing(T, L.E, k)
    mc.route_and_prune(lg, None, 0.0, r)
    y = forward(mc, L, r, x, T, k)
    if counts:
        assert tuple(r.counts[:2].tolist()) == counts
    val, top = torch.sort(lg.double(), dim=1, descending=True)
    want = reference(L, G, x.double(), top[:, :k], torch.softmax(val[:, :k], dim=1))
    got = y.view(torch.bfloat16).double()
    # one bf16 rounding of y (at most 2^-8 of the value) and the fp16 rounding of
    # h: relative 2^-11 at most and independent over the ffn terms of a sum, so
    # its standard deviation is below 2^-12 of the token's rms (a 1-bit expert's
    # outputs are several times a 3-bit one's) and eight of them stay below 2^-9
    rms = want.square().mean(dim=1, keepdim=True).sqrt()
    assert ((got - want).abs() <= 2.0 ** -8 * want.abs() + 2.0 ** -9 * rms).all()


@pytest.mark.parametrize("shape,T", [
    (ORDINARY, 47),                # 12 pairs an expert
    (STREAMED, 55),                # 14
    ((8, 1024, 3584), 11),         # up to 110 M weights: 12 tokens
    ((16, 2048, 2048), 15),        # up to 250 M: 16 tokens
    ((20, 512, 1024), 11),         # more than 16 experts, up to 60 M: 12 tokens
])
def test_last_gemv_batch(layer, shape, T):
    """Where the GEMVs hand over to the GEMMs: T tokens take the former, T + 1
    the latter, and both agree on the tokens they share."""
    import paper_2410_06270_amd as mc
    L = layer(shape, 128)
    x = torch.randn((T + 1, L.d), generator=torch.Generator(device="cuda").manual_seed(T), device="cuda").to(torch.bfloat16)
    lg = torch.randn((T + 1, L.E), generator=torch.Generator(device="cuda").manual_seed(T + 1), device="cuda")
    y = []
    for n in (T, T + 1):
        r = mc.Routing(n, L.E, 2)
        mc.route_and_prune(lg[:n], None, 0.3, r)
        y.append(forward(mc, L, r, x[:n], n, 2, gemvs=n == T).view(torch.bfloat16)[:T].double())
    # one bf16 rounding and the rounding of h on each side (see test_gemv_blocks)
    rms = y[1].square().mean(dim=1, keepdim=True).sqrt()
    assert ((y[0] - y[1]).abs() <= 2.0 ** -7 * y[1].abs() + 2.0 ** -8 * rms).all()


@pytest.mark.parametrize("shape", [ORDINARY, STREAMED])
def test_gemv_garbage_routing(layer, shape):
    """Routing buffers that no routing call filled: every index is range-checked
    on the device, so y is written (wrong values) and nothing else."""
    import paper_2410_06270_amd as mc
    T, k = 32, 2
    P = T * k
    L = layer(shape, 128)
    n = np.random.default_rng(T)
    r = mc.Routing(T, L.E, k)
    for buf in (r.counts, r.offsets, r.pair_token, r.pair_pos):
        m = buf.numel()
        a = np.where(n.random(m) < 0.5, n.integers(-(1 << 30), 1 << 30, m), n.integers(-2 * P, 2 * P, m))
        buf.copy_(torch.from_numpy(a.astype(np.int32)).view_as(buf))
    r.counts[:2] = P                          # two experts claim every pair slot
    r.offsets[:2] = 0
    r.topk_w.copy_(torch.from_numpy(n.random(r.topk_w.numel()).astype(np.float32)).view_as(r.topk_w))
    x = torch.randn((T, L.d), generator=torch.Generator(device="cuda").manual_seed(T), device="cuda").to(torch.bfloat16)
    print("garbage routing on %s" % (shape,), flush=True)
    y = forward(mc, L, r, x, T, k)
    assert not (y == 0x7FC1).any()
