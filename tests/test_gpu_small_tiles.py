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

D, FFN, BITS = 384, 640, [1, 2, 3, 2]


def counted_logits(counts, seed):
    """Logits [T][E] (top-1) that route counts[e] tokens, in random order, to e."""
    g = np.random.default_rng(seed)
    lg = g.standard_normal((sum(counts), len(counts))).astype(np.float32)
    e = g.permutation(np.repeat(np.arange(len(counts)), counts))
    lg[np.arange(len(e)), e] += 20.0
    return lg


@pytest.fixture(scope="module")
def layers():
    import paper_2410_06270_amd as mc
    mats = synthetic.layer_weights(1, E=4, d=D, ffn=FFN)
    out = {}
    for G in (32, 64, 128):
        L = mc.PackedLayer(4, D, FFN, BITS, G)
        mc.pack(*(torch.from_numpy(np.stack([m[i] for m in mats])).cuda() for i in range(3)), L)
        out[G] = (L, oracle.pack_layer(mats, BITS, G)[2])
    torch.cuda.synchronize()
    return out


# per-expert pairs; the average decides the m-tile: 32 tokens up to 40 pairs
# an expert, 64 above, 128 from 512 on
@pytest.mark.parametrize("counts", [
    [12, 0, 0, 0],             # the fewest tokens that take the GEMMs
    [1, 31, 32, 0],            # T = 64, one fragment row
    [33, 31, 64, 1],
    [65, 0, 1, 94],            # an average of 40: the last of the 32-token tiles
    [63, 64, 65, 1],           # two fragment rows
    [128, 129, 96, 33],
    [1969, 33, 97, 1],         # an average of 525
])
@pytest.mark.parametrize("G", [32, 64, 128])
def test_gemm_tile_edges(layers, G, counts):
    import paper_2410_06270_amd as mc
    L, logical = layers[G]
    T = sum(counts)
    x = synthetic.activations(1, T, d=D)
    lg = counted_logits(counts, T)
    r = mc.Routing(T, 4, 1)
    xd = torch.from_numpy(x.view(np.int16)).cuda()
    mc.route_and_prune(torch.from_numpy(lg).cuda(), None, 0.0, r)
    y = torch.empty((T, D), dtype=torch.int16, device="cuda")
    ws = torch.empty(mc.forward_workspace(T, 4, 1, D, FFN), dtype=torch.uint8, device="cuda")
    mc.moe_forward(xd, r, L, y, ws)
    y2 = torch.empty_like(y)
    mc.moe_forward_noalloc(xd, r, L, y2)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(r.counts.cpu().numpy(), counts)
    assert torch.equal(y, y2)
    y_ref = oracle.moe_forward(x, oracle.route(lg, None, 1, 0.0), logical, G)
    got = oracle.bf16_to_float64(y.cpu().numpy().view(np.uint16))
    # one bf16 rounding of y (8 significant bits: at most 2^-8 of the value),
    # and the fp16 rounding of h: relative 2^-11 at most and independent over
    # the 640 terms of a sum, so its standard deviation is below 2^-12 of the
    # token's rms (a 1-bit expert's outputs are several times a 3-bit one's)
    # and eight of them stay below 2^-9 of it
    rms = np.sqrt((y_ref ** 2).mean(axis=1, keepdims=True))
    assert (np.abs(got - y_ref) <= 2.0 ** -8 * np.abs(y_ref) + 2.0 ** -9 * rms).all()
