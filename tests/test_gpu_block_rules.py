"""GPU test of the reconstruction's launch rules: the same field on meshes either
side of each rule (waves per block, non-temporal streams, partial last waves)
takes the same values, since a cell's point states depend on its stencil only.

A periodic box of n copies of a small box along z holds the small box's cells n
times, with the same stencils up to the cell ids; the field repeats likewise.
Stencil members are listed in ascending id, so the copies differ by summation
order only: 1e-13 of the largest value in FP64 (26 + 54 terms of 1e-16 each), a
few 1e-7 in FP32.  A face's points are numbered by its owner, the lower id,
which differs at the box's seam: values are compared sorted over a face's
points."""
import math

import numpy as np
import pytest

from paper_2609_07387_amd import inputs, ucns

pytestmark = pytest.mark.gpu

BASE = (9, 9, 9)


def _point_states(copies, order, precision, gated):
    import torch

    n = (BASE[0], BASE[1], BASE[2] * copies)
    h = 2 * math.pi / BASE[0]
    m = inputs.hex_box_mesh(n, tuple(h * a for a in n), (True,) * 3)
    lm = ucns.Mesh(m, order=order)
    cen = lm.cell_geometry()[1]
    U = np.ascontiguousarray(inputs.tgv_conserved(cen).T)
    U[0] += 0.05 * np.sin(cen[:, 0] + 2 * cen[:, 2])
    lm.upload(precision)
    ws = ucns.Workspace(lm, precision, False)
    mask = torch.from_numpy(np.tile((np.arange(9 ** 3) % 5 != 0).astype(np.uint8), copies)).cuda() if gated else None
    ucns.reconstruct(lm, ucns.phys(), torch.from_numpy(U).cuda(), precision, ws.face_state, mask, ws.flags)
    torch.cuda.synchronize()
    pad = -(-lm.n_cell // 64) * 64
    fs = ws.face_state.reshape(lm.nfmax * lm.qmax, pad, 5)[:, :lm.n_cell].double().cpu().numpy()
    return np.sort(fs.reshape(lm.nfmax, lm.qmax, copies, 9 ** 3, 5), axis=1)


# copies: waves per block one below 2,048 waves (P2 FP64: 179 copies are 2,039
# waves, 181 are 2,062), streams beyond 250 MB from about 74 (P2 FP64), 137
# (P2 FP32), 38 (P3 FP64) and 8 (P4 FP64) copies
@pytest.mark.parametrize("order,precision,gated,copies", [
    (2, ucns.F64, False, 70), (2, ucns.F64, False, 80), (2, ucns.F64, False, 181), (2, ucns.F64, True, 181),
    (2, ucns.F32, False, 130), (2, ucns.F32, False, 181), (2, ucns.F32, True, 181),
    (3, ucns.F64, False, 36), (3, ucns.F64, False, 42), (3, ucns.F32, False, 60),
    (4, ucns.F64, False, 2), (4, ucns.F64, False, 9), (4, ucns.F32, False, 17)])
def test_copies_agree_across_launch_rules(order, precision, gated, copies):
    ref = _point_states(1, order, precision, gated)
    got = _point_states(copies, order, precision, gated)
    tol = (1e-13 if precision == ucns.F64 else 1e-6) * np.abs(ref).max()
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() <= tol, np.abs(got - ref).max() / np.abs(ref).max()


def _fallback(copies, order, precision, gated):
    """Flags and point states of a field with near-vacuum cells, whose
    polynomials go negative at some face points."""
    import torch

    n = (BASE[0], BASE[1], BASE[2] * copies)
    h = 2 * math.pi / BASE[0]
    lm = ucns.Mesh(inputs.hex_box_mesh(n, tuple(h * a for a in n), (True,) * 3), order=order)
    rng = np.random.default_rng(5)
    rho = np.where(rng.random(9 ** 3) < 0.1, 1e-3, 1.0) * rng.uniform(0.9, 1.1, 9 ** 3)
    U = np.stack([rho, 0.3 * rho, -0.2 * rho, 0.1 * rho, rho * 2.5 + 0.07 * rho])
    U = np.ascontiguousarray(np.tile(U, (1, copies)))
    lm.upload(precision)
    ws = ucns.Workspace(lm, precision, False)
    mask = torch.from_numpy(np.tile((np.arange(9 ** 3) % 3 != 0).astype(np.uint8), copies)).cuda() if gated else None
    ucns.reconstruct(lm, ucns.phys(mach=1.0), torch.from_numpy(U).cuda(), precision, ws.face_state, mask, ws.flags)
    torch.cuda.synchronize()
    pad = -(-lm.n_cell // 64) * 64
    fs = ws.face_state.reshape(lm.nfmax, lm.qmax, pad, 5)[:, :, :lm.n_cell].double().cpu().numpy()
    return (ws.flags.cpu().numpy().reshape(copies, 9 ** 3),
            np.sort(fs.reshape(lm.nfmax, lm.qmax, copies, 9 ** 3, 5), axis=1))


# without a gate the kernel finishes its marked cells itself, with one a pass does
@pytest.mark.parametrize("order,precision,gated,copies", [
    (2, ucns.F64, True, 80), (2, ucns.F32, True, 150), (2, ucns.F64, False, 80), (3, ucns.F64, True, 40),
    (3, ucns.F32, True, 80), (4, ucns.F64, False, 9)])
def test_positivity_fallback_across_launch_rules(order, precision, gated, copies):
    flags, fs = _fallback(1, order, precision, gated)
    flags_n, fs_n = _fallback(copies, order, precision, gated)
    assert (flags & 4).any() and not (flags & 0x80).any()
    if gated:
        assert (flags & 2).any()
    assert np.array_equal(flags_n, np.repeat(flags, copies, 0))
    assert (fs_n[..., 0] > 1e-10).all()  # density positive at every point
    # (the weights amplify the summation-order difference near vacuum: ten times
    # the tolerance of the smooth field)
    tol = (1e-12 if precision == ucns.F64 else 1e-5) * np.abs(fs).max()
    assert np.abs(fs_n - fs).max() <= tol
