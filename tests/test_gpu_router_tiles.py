"""Router logits on every token and expert tile of the vector kernel (1, 2, 4
and 8 tokens, 4 and 8 experts a workgroup), with ragged last tiles and rows
shorter and longer than one pass of the workgroup: within one fp32 ulp of the
correctly rounded logits, and equal to them almost everywhere."""
import numpy as np
import pytest

import oracle
import synthetic

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("T", [3, 512, 513, 1024, 1027, 2048, 2051])
@pytest.mark.parametrize("d,E", [(8, 3), (264, 4), (2056, 5), (24, 8), (2176, 9), (128, 15)])
def test_router_tiles(T, d, E):
    import paper_2410_06270_amd as mc
    g = np.random.default_rng(T * 31 + d + E)
    x = synthetic.to_bf16_bits(g.standard_normal((T, d)).astype(np.float32))
    w = synthetic.to_bf16_bits(g.standard_normal((E, d)).astype(np.float32))
    logits = torch.empty((T, E), dtype=torch.float32, device="cuda")
    mc.router_logits(torch.from_numpy(x.view(np.int16)).cuda(), torch.from_numpy(w.view(np.int16)).cuda(), logits)
    torch.cuda.synchronize()
    got = logits.cpu().numpy()
    toks = sorted({0, 1, 2, T // 2, T - 2, T - 1})
    ref = oracle.router_logits(x, w, tokens=toks)[toks]
    assert (np.abs(got[toks] - ref) <= np.spacing(np.abs(ref))).all()
    # every token against fp64 (whose own error is far below an fp32 ulp)
    full = oracle.bf16_to_float64(x) @ oracle.bf16_to_float64(w).T
    assert (np.abs(got - full) <= 0.501 * np.spacing(np.abs(full).astype(np.float32)) + 1e-12).all()
