"""GPU test of the gate network's training step at the sizes where its split can
go wrong: one row, the edges of a wave's 16 samples and of a 64-sample chunk,
and batches where the 64 blocks take one or two chunks, the last one ragged."""
import numpy as np
import pytest

from oracle import mlp as omlp
from paper_2609_07387_amd import gate, ucns

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 17, 64, 65, 4096, 4097, 6223])
def test_train_step_chunk_edges(n):
    """Loss, gradient and first moments against the oracle's backward with the
    same bf16 rounding points.  Tolerances: the two differ by FP32 summation
    order (1e-6 of a sum) and by bf16 roundings of dH that fall on the other
    side (2^-9 of one term); 2e-2 of a block's largest entry covers the latter
    where a gradient is a single sample's."""
    import torch

    rng = np.random.default_rng(100 + n)
    p = gate.init_params(rng.normal(size=12) * 0.5 - 3.0, rng.uniform(0.5, 2.0, 12), 5)
    F = (rng.normal(size=(n, 12)) - 3.0).astype(np.float32)
    Y = (rng.random(n) < 0.3).astype(np.float32)
    P = torch.tensor(p, device="cuda")
    G = torch.full_like(P, float("nan"))
    A = torch.zeros(2 * ucns.MLP_NPARAM, dtype=torch.float32, device="cuda")
    L = torch.zeros(1, dtype=torch.float32, device="cuda")
    ucns.mlp_train_step(P, G, A, torch.tensor(F, device="cuda"), torch.tensor(Y, device="cuda"), 2.5, 1e-3, 1, L)
    torch.cuda.synchronize()
    loss_ref, g_ref = omlp.loss_and_grad(p.astype(np.float64), F.astype(np.float64), Y, 2.5, emulate_bf16=True)
    g = G.cpu().numpy().astype(np.float64)
    assert abs(L.item() - loss_ref) < 1e-5 * max(1, loss_ref)
    for name, a, b in (("W1", 32, 32 + 12 * 64), ("b1", 1056, 1120), ("W2", 1120, 5216), ("b2", 5216, 5280),
                       ("w3", 5280, 5344), ("b3", 5344, 5345)):
        err = np.abs(g[a:b] - g_ref[a:b]).max() / max(np.abs(g_ref[a:b]).max(), 1e-12)
        assert err < 2e-2, (name, err)
    assert np.all(g[:32] == 0) and np.all(g[32 + 12 * 64:1056] == 0) and np.all(g[5345:] == 0)
    m = A.cpu().numpy().astype(np.float64)[:ucns.MLP_NPARAM]
    assert np.abs(m - 0.1 * g).max() <= 1e-6 * max(np.abs(g).max(), 1e-30)
