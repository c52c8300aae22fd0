"""One-call routing + forward on the batches whose routing runs inside the
GEMMs' preparation launch: every routing output and y equal the two-call path
bit for bit (the routing kernel, then the preparation that reads its lists),
for the expert counts and token counts at the edges of that path."""
import numpy as np
import pytest

import synthetic

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("G", [32, 64, 128])
@pytest.mark.parametrize("E,k,d,ffn,T,tau", [
    (1, 1, 128, 128, 64, 0.0),        # one expert: its list fills two fragment rows
    (3, 2, 640, 128, 12, 0.3),        # d past one 512-column block, the fewest tokens
    (4, 2, 256, 512, 64, 0.3),
    (16, 8, 1152, 256, 64, 0.05),     # 16 experts, four lanes a token's selection shares with three others
    (16, 1, 256, 128, 33, 0.0),
    (17, 2, 256, 128, 32, 0.3),       # past the path: two launches
])
def test_route_prep_equals_two_calls(G, E, k, d, ffn, T, tau):
    import paper_2410_06270_amd as mc
    g = np.random.default_rng(E * 1000 + T)
    w = [torch.from_numpy(g.standard_normal(s).astype(np.float32) * np.float32(0.05)).cuda()
         for s in ((E, ffn, d), (E, ffn, d), (E, d, ffn))]
    L = mc.PackedLayer(E, d, ffn, [1 + e % 3 for e in range(E)], G)
    mc.pack(*w, L)
    x = torch.from_numpy(synthetic.to_bf16_bits(g.standard_normal((T, d)).astype(np.float32)).view(np.int16)).cuda()
    lg = g.standard_normal((T, E)).astype(np.float32)
    lg[::5] = lg[::5, :1]                                  # ties
    lg = torch.from_numpy(lg).cuda()
    imp = torch.from_numpy((g.random(T) < 0.2).astype(np.uint8)).cuda()
    ws = torch.full((mc.forward_workspace(T, E, k, d, ffn),), 0xff, dtype=torch.uint8, device="cuda")   # NaN patterns
    out = []
    for one_call in (False, True):
        r = mc.Routing(T, E, k)
        y = torch.zeros((T, d), dtype=torch.int16, device="cuda")
        ws.fill_(0xff)
        if one_call:
            mc.route_forward(x, lg, imp, tau, r, L, y, ws)
        else:
            mc.route_and_prune(lg, imp, tau, r)
            mc.moe_forward(x, r, L, y, ws)
        torch.cuda.synchronize()
        n = int(r.offsets[E])
        out.append([y] + [r.topk_idx, r.topk_w, r.kept, r.counts, r.offsets, r.pair_token[:n], r.pair_rank[:n],
                          r.pair_w[:n], r.pair_pos, r.n_pruned])
    for a, b in zip(*out):
        assert torch.equal(a, b)
    assert torch.isfinite(out[0][0].view(torch.bfloat16).float()).all()
