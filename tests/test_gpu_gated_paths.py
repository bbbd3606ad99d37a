"""GPU tests of the ways a gated reconstruction takes its troubled cells: the
whole wave per cell (one or two of them in a wave), a lane per stencil, a lane
per cell.  Each has to give a troubled cell the values the ungated call gives
it."""
import math

import numpy as np
import pytest

from paper_2609_07387_amd import inputs, ucns

pytestmark = pytest.mark.gpu

MESH = {
    # 1,008 and 1,512 cells: the last wave holds 48 and 40
    "hex": lambda: inputs.hex_box_mesh((14, 9, 8), tuple(2 * math.pi * a / 8 for a in (14, 9, 8)), (True,) * 3),
    "tet": lambda: inputs.kuhn_tet_mesh((7, 6, 6), tuple(2 * math.pi * a / 8 for a in (7, 6, 6)), (True,) * 3),
    # four element types, 960 cells: cells with fewer faces than slots and stencils of several sizes
    "mixed": lambda: inputs.mixed_bl_mesh((9, 5, 6), (2.25, 1.0, 0.75), (2, 2), 2, 1.2, 0.15, 0.05),
}


def _setup(mesh, order, precision):
    """Mesh, state (5 % noise: the weights move) and a function mask -> point
    states [NF * Q, n_cell, 5], flags."""
    import torch

    lm = ucns.Mesh(MESH[mesh](), order=order)
    cen = lm.cell_geometry()[1]
    rng = np.random.default_rng(3)
    U = np.ascontiguousarray(inputs.tgv_conserved(cen).T)
    U *= 1 + 0.05 * rng.standard_normal(U.shape) * np.array([1, 1, 1, 1, 0.02])[:, None]
    U[0] += 0.05 * np.sin(cen[:, 0])
    U[3] = 0.1 * U[0] * np.cos(cen[:, 2])
    lm.upload(precision)
    Ud = torch.from_numpy(U).cuda()

    def run(mask):
        ws = ucns.Workspace(lm, precision, False)
        ws.face_state.zero_()
        m = None if mask is None else torch.from_numpy(mask).cuda()
        ucns.reconstruct(lm, ucns.phys(mach=0.5), Ud, precision, ws.face_state, m, ws.flags)
        torch.cuda.synchronize()
        pad = -(-lm.n_cell // 64) * 64
        fs = ws.face_state.reshape(lm.nfmax * lm.qmax, pad, 5)[:, :lm.n_cell].double().cpu().numpy()
        return fs, ws.flags.cpu().numpy()

    return lm, U, run


@pytest.mark.parametrize("precision", [ucns.F64, ucns.F32])
@pytest.mark.parametrize("mesh,order", [("hex", 2), ("hex", 3), ("tet", 2), ("tet", 3), ("mixed", 2)])
def test_few_troubled_cells_take_the_ungated_values(mesh, order, precision):
    """One troubled cell per wave, at every lane of a wave once, then two: the
    lanes past the cell's stencil members (54 on hexahedra, 32 or 36 on
    tetrahedra) as well as those that load one.  Tolerance: the sums of at most
    54 products are formed in another order, 54 roundings of 1.1e-16 (FP64) or
    6e-8 (FP32) of the largest value, times ten for the nonlinear weights."""
    lm, U, run = _setup(mesh, order, precision)
    ref, rflags = run(None)
    scale = np.array([np.abs(U[0]).max()] + [np.abs(U[1:4]).max()] * 3 + [np.abs(U[4]).max()])
    tol = 10 * 54 * (1.1e-16 if precision == ucns.F64 else 6e-8)
    worst = 0.0
    waves = -(-lm.n_cell // 64)
    for first in range(0, 64, waves):
        for second in (None, 21):
            mask = np.ones(lm.n_cell, np.uint8)
            for w in range(waves):
                for lane in [(first + w) % 64] + ([] if second is None else [(first + w + second) % 64]):
                    if 64 * w + lane < lm.n_cell:
                        mask[64 * w + lane] = 0
            fs, flags = run(mask)
            t = mask == 0
            assert np.array_equal(flags[t], rflags[t])
            worst = max(worst, (np.abs(fs - ref)[:, t] / scale).max())
    assert worst <= tol, worst


@pytest.mark.parametrize("precision", [ucns.F64, ucns.F32])
@pytest.mark.parametrize("mesh", ["hex", "tet", "mixed"])
def test_all_troubled_is_the_ungated_call_bitwise(mesh, precision):
    """A mask without a smooth cell has every wave take the lane-per-cell path
    (no wave of these meshes holds fewer than 40 cells), the ungated call's own:
    the same operations in the same order, so the same bits."""
    lm, U, run = _setup(mesh, 2, precision)
    ref, rflags = run(None)
    fs, flags = run(np.zeros(lm.n_cell, np.uint8))
    assert np.array_equal(flags, rflags)
    assert np.array_equal(fs, ref), np.abs(fs - ref).max()
