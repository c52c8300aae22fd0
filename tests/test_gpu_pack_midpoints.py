"""The packing kernel decides codes by fp32 thresholds instead of the exact
midpoints: at every width and group size, weights placed on the midpoints
(rounded to fp32) and on their fp32 neighbours get the oracle's exact codes,
as do groups whose range spans signed zeros, subnormals and the fp16 limits."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def midpoint_groups(R, K, G, bits, seed):
    """fp32 [R][K]: each group has a random range (scales from subnormal to
    saturating), its other weights at or next to the midpoints s (j + 1/2 - z)."""
    g = np.random.default_rng(seed)
    W = np.empty((R, K), np.float32)
    L = (1 << bits) - 1
    for r in range(R):
        for k in range(0, K, G):
            scale = np.float32(10.0 ** g.uniform(-9, 5))
            lo, hi = sorted(g.standard_normal(2) * scale)
            if (r + k // G) % 4 == 0:
                lo = np.float32(0.0)                       # z = 0: a midpoint below every weight
                hi = abs(hi)
            w = np.full(G, lo, np.float32)
            w[1] = hi
            s, z, _ = oracle.quantize_group(w, bits)
            s, z = (float(np.array(v, np.uint16).view(np.float16)) for v in (s, z))
            for i in range(2, G):
                m = np.float32(np.clip(s * (g.integers(0, L) + 0.5 - z), lo, hi))
                step = g.integers(-1, 2)
                w[i] = m if step == 0 else np.nextafter(m, np.float32(np.inf * step), dtype=np.float32)
            w[2:] = np.clip(w[2:], w[0], w[1])
            w[3] = 0.0 if lo <= 0 <= hi else w[3]
            w[4] = -0.0 if lo <= 0 <= hi else w[4]
            W[r, k:k + G] = g.permutation(w)
    return W


@pytest.mark.parametrize("G", [32, 64, 128])
@pytest.mark.parametrize("bits", [1, 2, 3])
def test_pack_midpoints_bit_exact(bits, G):
    import paper_2410_06270_amd as mc
    d, ffn = 256, 128
    mats = [tuple(midpoint_groups(*shape, G, bits, 10 * bits + m)
                  for m, shape in enumerate([(ffn, d), (ffn, d), (d, ffn)]))]
    words, sz, _ = oracle.pack_layer(mats, [bits], G)
    L = mc.PackedLayer(1, d, ffn, [bits], G)
    mc.pack(*(torch.from_numpy(m[None].copy()).cuda() for m in mats[0]), L)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(L.sz.cpu().numpy().view(np.uint32), sz)
    np.testing.assert_array_equal(L.words.cpu().numpy().view(np.uint32), words)
