"""The grouped GEMMs on every m-tile size, at the edges of their tiles: the
pairs of each expert set exactly (around one, two, three and four fragment
rows of 32, one pair, none), every group size, 3- and 5-chunk reductions (the
staging ring is two chunks deep), widths 1, 2 and 3; against the oracle, and
bit-identical between the workspace and the scratch entry points."""
import numpy as np
import pytest

import oracle
import synthetic

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BITS = [1, 2, 3, 2]


def counted_logits(counts, seed):
    """Logits [T][E] (top-1) that route counts[e] tokens, in random order, to e."""
    g = np.random.default_rng(seed)
    lg = g.standard_normal((sum(counts), len(counts))).astype(np.float32)
    e = g.permutation(np.repeat(np.arange(len(counts)), counts))
    lg[np.arange(len(e)), e] += 20.0
    return lg


@pytest.fixture(scope="module")
def layer():
    """layer(d, ffn, G) -> (packed layer, the oracle's), made once."""
    import paper_2410_06270_amd as mc
    made = {}

    def get(d, ffn, G):
        if (d, ffn, G) not in made:
            made.clear()
            mats = synthetic.layer_weights(1, E=4, d=d, ffn=ffn)
            L = mc.PackedLayer(4, d, ffn, BITS, G)
            mc.pack(*(torch.from_numpy(np.stack([m[i] for m in mats])).cuda() for i in range(3)), L)
            torch.cuda.synchronize()
            made[(d, ffn, G)] = (L, oracle.pack_layer(mats, BITS, G)[2])
        return made[(d, ffn, G)]
    return get


SMALL = (384, 640)      # 32-token m-tiles whatever the batch; 3- and 5-chunk reductions
WIDE = (384, 4224)      # 64-token ones from 450 pairs an expert on
LONG = (2176, 4224)     # 128-token ones from 3400 pairs an expert on


@pytest.mark.parametrize("shape,counts", [
    (SMALL, [12, 0, 0, 0]),             # the fewest tokens that take the GEMMs
    (SMALL, [1, 31, 32, 0]),            # T = 64, one fragment row
    (SMALL, [33, 31, 64, 1]),
    (SMALL, [65, 0, 1, 94]),
    (WIDE, [1722, 63, 65, 1]),          # one and two fragment rows of 64-token m-tiles
    (WIDE, [640, 672, 33, 500]),
    (LONG, [13216, 33, 96, 129]),       # one to four fragment rows of 128-token m-tiles
])
@pytest.mark.parametrize("G", [32, 64, 128])
def test_gemm_tile_edges(layer, G, shape, counts):
    import paper_2410_06270_amd as mc
    d, ffn = shape
    L, logical = layer(d, ffn, G)
    T = sum(counts)
    x = synthetic.activations(1, T, d=d)
    lg = counted_logits(counts, T)
    r = mc.Routing(T, 4, 1)
    xd = torch.from_numpy(x.view(np.int16)).cuda()
    mc.route_and_prune(torch.from_numpy(lg).cuda(), None, 0.0, r)
    y = torch.empty((T, d), dtype=torch.int16, device="cuda")
    need = mc.forward_workspace(T, 4, 1, d, ffn)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    mc.moe_forward(xd, r, L, y, ws)
    if need <= 32 << 20:
        y2 = torch.empty_like(y)
        mc.moe_forward_noalloc(xd, r, L, y2)
        assert torch.equal(y, y2)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(r.counts.cpu().numpy(), counts)
    ref = oracle.route(lg, None, 1, 0.0)
    toks = None
    if T > 200:          # the first and last pairs of every expert's list and a spread
        lists = [ref["pair_token"][ref["offsets"][e]:ref["offsets"][e + 1]] for e in range(4)]
        toks = {int(t) for p in lists for t in (*p[:2], *p[-2:])}
        toks |= set(np.random.default_rng(T).choice(T, 24, replace=False).tolist())
        toks = sorted(toks)
    y_ref = oracle.moe_forward(x, ref, logical, G, tokens=toks)
    got = oracle.bf16_to_float64(y.cpu().numpy().view(np.uint16))
    if toks is not None:
        got = got[toks]
        assert y_ref.shape == got.shape
    # one bf16 rounding of y (8 significant bits: at most 2^-8 of the value),
    # and the fp16 rounding of h: relative 2^-11 at most and independent over
    # the ffn terms of a sum, so its standard deviation is below 2^-12 of the
    # token's rms (a 1-bit expert's outputs are several times a 3-bit one's)
    # and eight of them stay below 2^-9 of it
    rms = np.sqrt((y_ref ** 2).mean(axis=1, keepdims=True))
    assert (np.abs(got - y_ref) <= 2.0 ** -8 * np.abs(y_ref) + 2.0 ** -9 * rms).all()
