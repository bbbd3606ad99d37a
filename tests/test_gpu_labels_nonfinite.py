"""GPU test of the gate's training labels where the state holds an infinity: a
cell whose stencils reach it is labelled as the oracle labels it (its
indicators are NaN, taken as 0, and its weights leave the linear ones), so that
it is not collected as a smooth sample."""
import math

import numpy as np
import pytest

import oracle
from paper_2609_07387_amd import inputs, ucns

from parity_helpers import as_oracle_phys

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("precision", [ucns.F64, ucns.F32])
@pytest.mark.parametrize("mesh,order", [("tet", 2), ("hex", 2), ("tet", 3)])
def test_labels_beside_a_nonfinite_value_match_oracle(mesh, order, precision, value):
    """|omega - lambda| is in [0, 1]; FP32 labels of the rough field carry the
    weights' FP32 rounding (1e-3 covers it; what the test looks for is 0.999
    against less than 0.02)."""
    import torch

    if mesh == "tet":
        m = inputs.kuhn_tet_mesh((5, 5, 5), (2 * math.pi * 5 / 8,) * 3, (True,) * 3)
    else:
        m = inputs.hex_box_mesh((9, 8, 7), tuple(2 * math.pi * a / 8 for a in (9, 8, 7)), (True,) * 3)
    rng = np.random.default_rng(5)
    rho = rng.uniform(0.9, 1.1, m.n_cell)
    U = np.stack([rho, 0.3 * rho, -0.2 * rho, 0.1 * rho, 2.57 * rho])
    for v, c in enumerate(rng.permutation(m.n_cell)[:2]):
        U[v, c] = value
    ph = ucns.phys(flux="hllc")
    _, oflags, olabel = oracle.OracleMesh(m, order=order).reconstruct(U, as_oracle_phys(ph), None, with_flags=True)
    lm = ucns.Mesh(m, order=order)
    lm.upload(precision)
    ws = ucns.Workspace(lm, precision, False)
    label = torch.full((m.n_cell,), float("nan"), dtype=torch.float32, device="cuda")
    ucns.reconstruct(lm, ph, torch.from_numpy(U).cuda(), precision, ws.face_state, None, ws.flags, label)
    torch.cuda.synchronize()
    assert np.array_equal(ws.flags.cpu().numpy(), oflags)
    assert np.abs(label.cpu().numpy() - olabel).max() < 1e-3
