"""Token importance of maps on both sides of the size from which they are read
by non-temporal loads (384 MB of the triangle), whole and ragged in 128-token
tiles, against 64-bit sums of the same bf16 map."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("H,L", [
    (24, 4000),      # 384.1 MB: streamed; 4000 = 31 * 128 + 32, a ragged last tile
    (24, 3992),      # 382.6 MB: not
    (96, 2048),      # 402.8 MB, whole tiles
])
def test_importance_stream(H, L):
    import paper_2410_06270_amd as mc
    d = 128
    g = torch.Generator(device="cuda").manual_seed(H + L)
    attn = torch.empty((H, L, L), dtype=torch.bfloat16, device="cuda")
    for h in range(H):
        attn[h] = torch.rand((L, L), generator=g, device="cuda").div_(L).to(torch.bfloat16)   # not zero above the diagonal
    x = torch.randn((L, d), generator=g, device="cuda").to(torch.bfloat16)
    imp = torch.empty(L, dtype=torch.float32, device="cuda")
    mask = torch.empty(L, dtype=torch.uint8, device="cuda")
    ws = torch.empty(mc.importance_workspace(H, L), dtype=torch.uint8, device="cuda")
    mc.token_importance(attn, x, 0.02, mask, ws, imp)
    cs = torch.zeros(L, dtype=torch.float64, device="cuda")
    for h in range(H):
        cs += attn[h].double().tril_().sum(0)
    want = x.double().abs().sum(1) * (cs / H) / torch.arange(L, 0, -1, dtype=torch.float64, device="cuda")
    # fp32 sums of positive terms, at most 2^-24 of the sum for each of the
    # longest chain's additions (8 rows of a head slice's heads, 16 phases, 64
    # lanes, the tiles): well under 256 of them
    torch.testing.assert_close(imp.double(), want, rtol=256 * 2.0 ** -24, atol=0)
    assert int(mask.sum()) == int(0.02 * L + 0.5)
