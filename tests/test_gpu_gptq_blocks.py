"""GPTQ at the edges of its blocks: one 128-column block, panels of 512 columns
full, partial and one block over, 64- and 128-wide update tiles, every width
and group size (codes and scale/zero words equal the oracle's on the oracle's
U); the factor where its merges are uneven; the Hessian of an unaligned x."""
import numpy as np
import pytest

import oracle
import synthetic

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def to_dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("R,K,bits,G", [
    (128, 128, 1, 32),        # a single block, no update
    (256, 512, 2, 64),        # one full panel
    (128, 640, 3, 128),       # a panel and one block
    (384, 1152, 3, 32),       # two panels and one block
    (128, 384, 1, 128),       # a partial panel
    (8192, 640, 2, 128),      # 64 row tiles: the 128-wide update tiles for four column tiles
])
def test_quantize_blocks_bit_exact(R, K, bits, G):
    import paper_2410_06270_amd as mc
    W = np.random.default_rng(R + K).standard_normal((R, K)).astype(np.float32) * np.float32(0.02)
    X = synthetic.calibration(1, 2 * K, K, tag=K + bits)
    U, dead = oracle.gptq_factor(oracle.gptq_hessian(X))
    rows = np.arange(R) if R <= 512 else np.array([0, 63, 64, 127, 128, R - 1])
    q, s, z, loss, margin = oracle.gptq_quantize_u(W[rows], U, dead, bits, G)
    L = mc.PackedLayer(1, K, R, [bits], G)
    ws = torch.empty(mc.gptq_workspace(R, K), dtype=torch.uint8, device="cuda")
    got_loss = torch.empty(R, dtype=torch.float64, device="cuda")
    mc.gptq_quantize(L, 0, 0, to_dev(W), to_dev(U), to_dev(dead), ws, loss=got_loss)
    codes = torch.empty((R, K), dtype=torch.uint8, device="cuda")
    mc.codes_export(L, 0, 0, codes)
    torch.cuda.synchronize()
    # rows whose decisions sit within 1e-12 of a midpoint may differ (none do)
    same = (codes.cpu().numpy()[rows] == q).all(axis=1)
    assert (same | (margin < 1e-12)).all() and same.mean() > 0.99
    np.testing.assert_allclose(got_loss.cpu().numpy()[rows][same], loss[same], rtol=1e-12)
    sz = L.sz.cpu().numpy().view(np.uint32)[:R * K // G].reshape(R // 16, K // G, 16)
    want = (s.astype(np.uint32) | (z.astype(np.uint32) << 16))
    got = sz.transpose(0, 2, 1).reshape(R, K // G)[rows]
    np.testing.assert_array_equal(got[same], want[same])


def test_quantize_most_rows():
    """The most rows the entry point takes (R K = 2^31): the first and last rows
    as in a call of their own (rows are independent)."""
    import paper_2410_06270_amd as mc
    R, K, G = 1 << 24, 128, 128
    U, dead = oracle.gptq_factor(oracle.gptq_hessian(synthetic.calibration(1, 2 * K, K, tag=K)))
    U, dead = to_dev(U), to_dev(dead)
    W = torch.randn((R, K), generator=torch.Generator(device="cuda").manual_seed(R), device="cuda").mul_(0.02)

    def quantize(w):
        n = w.shape[0]
        L = mc.PackedLayer(1, K, n, [1], G)
        ws = torch.empty(mc.gptq_workspace(n, K), dtype=torch.uint8, device="cuda")
        loss = torch.empty(n, dtype=torch.float64, device="cuda")
        mc.gptq_quantize(L, 0, 0, w, U, dead, ws, loss=loss)
        torch.cuda.synchronize()
        return L.words.view(torch.int32)[:n * K // 32], L.sz.view(torch.int32)[:n], loss

    every = quantize(W)
    for rows in (slice(0, 128), slice(R - 128, R)):
        for big, small, per in zip(every, quantize(W[rows].contiguous()), (K // 32, 1, 1)):
            assert torch.equal(big[rows.start * per:rows.stop * per], small)


def test_quantize_infinite_weight():
    """An infinite weight of either sign in the last column: its error, and so
    the row's loss, is infinite (a division's, not a NaN); the other rows are
    untouched."""
    import paper_2410_06270_amd as mc
    R, K, G = 128, 128, 32
    W = np.random.default_rng(3).standard_normal((R, K)).astype(np.float32) * np.float32(0.02)
    W[5, K - 1] = np.inf
    W[9, K - 1] = -np.inf
    U, dead = oracle.gptq_factor(oracle.gptq_hessian(synthetic.calibration(1, 2 * K, K, tag=K)))
    L = mc.PackedLayer(1, K, R, [2], G)
    ws = torch.empty(mc.gptq_workspace(R, K), dtype=torch.uint8, device="cuda")
    loss = torch.empty(R, dtype=torch.float64, device="cuda")
    mc.gptq_quantize(L, 0, 0, to_dev(W), to_dev(U), to_dev(dead), ws, loss=loss)
    torch.cuda.synchronize()
    loss = loss.cpu().numpy()
    assert loss[5] == np.inf and loss[9] == np.inf
    rows = [r for r in range(R) if r not in (5, 9)]
    want = oracle.gptq_quantize_u(W[rows], U, dead, 2, G)[3]
    np.testing.assert_allclose(loss[rows], want, rtol=1e-12)


@pytest.mark.parametrize("K", [128, 384, 640, 896])
def test_factor_uneven_merges(K):
    import paper_2410_06270_amd as mc
    H = oracle.gptq_hessian(synthetic.calibration(1, 2 * K, K, tag=K))
    U = torch.empty((K, K), dtype=torch.float64, device="cuda")
    dead = torch.empty(K, dtype=torch.uint8, device="cuda")
    mc.gptq_factor(to_dev(H), U, dead, torch.empty(mc.gptq_workspace(16, K), dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    Ur, _ = oracle.gptq_factor(H)
    U = U.cpu().numpy()
    np.testing.assert_array_equal(U, np.triu(U))
    # fp64 factorisations of a damped Gram matrix (condition below 1e4): errors
    # grow at most like K * cond * 2^-53 < 1e-9; 1e-11 leaves a hundredfold
    assert np.abs(U - Ur).max() <= 1e-11 * np.abs(Ur).max()


@pytest.mark.parametrize("N,off", [(1, 0), (33, 0), (70, 1), (64, 3)])
def test_hessian_alignment_and_rows(N, off):
    """x at any 2-byte offset; calibration rows that do not fill a step."""
    import paper_2410_06270_amd as mc
    K = 128
    X = synthetic.calibration(1, N, K, tag=N)
    buf = torch.zeros(N * K + off, dtype=torch.int16, device="cuda")
    buf[off:] = to_dev(X.view(np.int16)).reshape(-1)
    H = torch.empty((K, K), dtype=torch.float64, device="cuda")
    mc.gptq_hessian(buf[off:].view(N, K), H)
    torch.cuda.synchronize()
    Xa = np.abs(oracle.bf16_to_float64(X))
    H = H.cpu().numpy()
    assert (np.abs(H - oracle.gptq_hessian(X)) <= N * 2.0 ** -52 * 2.0 * (Xa.T @ Xa)).all()
    np.testing.assert_array_equal(H, H.T)
