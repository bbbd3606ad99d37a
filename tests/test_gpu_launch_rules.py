"""GPU tests of the reconstruction on both sides of each launch rule: plain or
non-temporal operator streams, one or four waves per block, plain or
non-temporal stores of the point states.  Each case states its side, worked out
from the mesh's own sizes, so a case that no longer crosses its rule fails.

The box is n copies of a 9 x 9 x 9 periodic box along z, with the field
repeated: each copy holds the small box's cells with the same stencils, listed
in another order where ids wrap at the seam."""
import math

import numpy as np
import pytest

import oracle
from paper_2609_07387_amd import inputs, ucns

from parity_helpers import as_oracle_phys, face_maps, face_major

pytestmark = pytest.mark.gpu

N = 9
CACHE = 256 << 20  # the memory-side cache the rules are about


def _box(copies, order):
    h = 2 * math.pi / N
    n = (N, N, N * copies)
    return ucns.Mesh(inputs.hex_box_mesh(n, tuple(h * a for a in n), (True,) * 3), order=order)


def _sides(lm, precision, gated):
    """(non-temporal streams, waves per block, non-temporal point-state stores)
    of an ungated or masked call without gradients on a mesh of even stencils."""
    t = 8 if precision == ucns.F64 else 4
    padded = -(-lm.n_cell // 64) * 64
    if lm.K == 34:
        nt = padded * t * (34 * lm.mc_pad + 9 * lm.nd_max * lm.md_pad) > CACHE - (6 << 20)
        return nt, 4 if nt else 1, False
    stream = t * lm.K * lm.mc_pad + 4 * lm.mc_pad + t * 3 * lm.nfmax * lm.qmax
    stream += 4 * lm.nfmax if gated else lm.nd_max * lm.md_pad * (3 * t + 4)
    nt = padded * stream > CACHE - (6 << 20)
    waves = -(-lm.n_cell // 64)
    return nt, 1 if not nt or gated or waves <= 2048 else 4, t * 5 * lm.nfmax * lm.qmax * padded > CACHE // 16 * 11


def _call(lm, U, precision, mask, copies):
    """Point states [NF, Q, copies, 729, 5] and flags [copies, 729]."""
    import torch

    lm.upload(precision)
    ws = ucns.Workspace(lm, precision, False)
    m = None if mask is None else torch.from_numpy(np.tile(mask, copies)).cuda()
    Ud = torch.from_numpy(np.ascontiguousarray(np.tile(U, (1, copies)))).cuda()
    ucns.reconstruct(lm, ucns.phys(mach=1.0), Ud, precision, ws.face_state, m, ws.flags)
    torch.cuda.synchronize()
    pad = -(-lm.n_cell // 64) * 64
    fs = ws.face_state.reshape(lm.nfmax, lm.qmax, pad, 5)[:, :, :lm.n_cell].double().cpu().numpy()
    return fs.reshape(lm.nfmax, lm.qmax, copies, N ** 3, 5), ws.flags.cpu().numpy().reshape(copies, N ** 3)


SIDES = [  # order, precision, mask, copies, (streams marked, waves per block, stores marked)
    (2, ucns.F64, False, 86, (False, 1, False)), (2, ucns.F64, False, 92, (True, 1, False)),
    (2, ucns.F64, False, 181, (True, 4, False)), (2, ucns.F64, False, 262, (True, 4, False)),
    (2, ucns.F64, False, 266, (True, 4, True)),
    (2, ucns.F64, True, 136, (False, 1, False)), (2, ucns.F64, True, 143, (True, 1, False)),
    (2, ucns.F64, True, 266, (True, 1, True)),
    (2, ucns.F32, False, 160, (False, 1, False)), (2, ucns.F32, False, 168, (True, 1, False)),
    (2, ucns.F32, False, 181, (True, 4, False)),
    (2, ucns.F32, True, 264, (False, 1, False)), (2, ucns.F32, True, 270, (True, 1, False)),
    (3, ucns.F64, False, 30, (False, 1, False)), (3, ucns.F64, False, 33, (True, 1, False)),
    (3, ucns.F64, False, 120, (True, 1, True)), (3, ucns.F64, False, 182, (True, 4, True)),
    (3, ucns.F32, False, 58, (False, 1, False)), (3, ucns.F32, False, 62, (True, 1, False)),
    # (four-wave blocks whose last one reaches past the last tile: 593 and 1,094 waves)
    (4, ucns.F64, False, 11, (False, 1, False)), (4, ucns.F64, False, 13, (True, 4, False)),
    (4, ucns.F32, False, 22, (False, 1, False)), (4, ucns.F32, False, 24, (True, 4, False)),
]


@pytest.mark.parametrize("order,precision,gated,copies,sides", SIDES)
def test_both_sides_of_each_rule(order, precision, gated, copies, sides):
    """A smooth field and one with near-vacuum cells, whose polynomials go
    negative at some face points, on the large box against the small one.

    A face's points are numbered by its owner, which differs at the seam: values
    are compared sorted over a face's points.  Smooth field: the sums' order,
    1e-13 of the largest value in FP64 (at most 130 terms of 1e-16) and 1e-6 in
    FP32.  Near vacuum the weights amplify that: ten times as much, and equal
    flags.  A cell that fell back to first order (without a gate inside the main
    kernel, over the points it has just stored) holds its average, exactly."""
    import torch  # noqa: F401  (its HIP runtime is loaded before the library)

    one, lm = _box(1, order), _box(copies, order)
    assert _sides(lm, precision, gated) == sides
    rng = np.random.default_rng(5)
    cen = one.cell_geometry()[1]
    smooth = np.ascontiguousarray(inputs.tgv_conserved(cen).T)
    smooth[0] += 0.05 * np.sin(cen[:, 0] + 2 * cen[:, 2])
    rho = np.where(rng.random(N ** 3) < 0.1, 1e-3, 1.0) * rng.uniform(0.9, 1.1, N ** 3)
    vacuum = np.stack([rho, 0.3 * rho, -0.2 * rho, 0.1 * rho, 2.57 * rho])
    mask = (np.arange(N ** 3) % 3 != 0).astype(np.uint8) if gated else None
    eps = 1e-13 if precision == ucns.F64 else 1e-6
    for U, tol in ((smooth, eps), (vacuum, 10 * eps)):
        ref, rflags = _call(one, U, precision, mask, 1)
        fs, flags = _call(lm, U, precision, mask, copies)
        assert np.array_equal(flags, np.repeat(rflags, copies, 0))
        worst = 0.0
        for lf in range(lm.nfmax):
            worst = max(worst, np.abs(np.sort(fs[lf], axis=0) - np.sort(ref[lf], axis=0)).max())
        assert worst <= tol * np.abs(ref).max(), worst / np.abs(ref).max()
        first = (flags & 4) != 0
        avg = (U if precision == ucns.F64 else U.astype(np.float32)).T.astype(np.float64)
        for k in np.nonzero(first.any(axis=1))[0]:
            assert np.array_equal(fs[:, :, k, first[k]], np.broadcast_to(avg[first[k]], fs[:, :, k, first[k]].shape))
    assert first.any() and not (flags & 0x80).any()


@pytest.mark.parametrize("precision", [ucns.F64, ucns.F32])
@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("mesh,order", [("tet", 2), ("tet", 3), ("mixed", 2)])
def test_positivity_fallback_on_tets_and_mixed_cells(mesh, order, gated, precision):
    """The fallback on triangles (three points a face, staged three at a time at
    P3), on cells with fewer faces than slots and, with a gate on the mixed mesh,
    in waves whose cells have stencils of several sizes (the fallback pass walks
    the largest of its marked cells' own).  FP64: flags and point states as the
    oracle's (1e-9 of the largest value: condition numbers up to 2e4 times 1e-14,
    amplified near vacuum).  Both precisions: a first-order cell holds its average
    at its own points exactly, any other is positive there."""
    import torch

    if mesh == "tet":
        m = inputs.kuhn_tet_mesh((5, 5, 4), tuple(2 * math.pi * a / 8 for a in (5, 5, 4)), (True,) * 3)
    else:
        m = inputs.mixed_bl_mesh((9, 5, 6), (2.25, 1.0, 0.75), (2, 2), 2, 1.2, 0.15, 0.05)
    lm, om = ucns.Mesh(m, order=order), oracle.OracleMesh(m, order=order)
    if mesh == "mixed":
        assert om.mc_min < om.mc_max and lm.nfmax == 6
    n = m.n_cell
    rng = np.random.default_rng(7)
    rho = np.where(rng.random(n) < 0.1, 1e-3, 1.0) * rng.uniform(0.9, 1.1, n)
    U = np.stack([rho, 0.3 * rho, -0.2 * rho, 0.1 * rho, 2.57 * rho])
    mask = (rng.random(n) < 0.7).astype(np.uint8) if gated else None
    ph = ucns.phys(flux="hllc", mach=1.0)
    lm.upload(precision)
    ws = ucns.Workspace(lm, precision, False)
    ucns.reconstruct(lm, ph, torch.from_numpy(U).cuda(), precision, ws.face_state,
                     None if mask is None else torch.from_numpy(mask).cuda(), ws.flags)
    torch.cuda.synchronize()
    flags = ws.flags.cpu().numpy()
    ofs, oflags, _ = om.reconstruct(U, as_oracle_phys(ph), mask, with_flags=True)
    fl, fo, sl = face_maps(lm, om)
    a, b = face_major(lm, ws.face_state.double().cpu().numpy())[fl, sl, :lm.qmax], ofs[fo, sl, :lm.qmax]
    own = np.nonzero(om.cell_faces()[0] >= 0)[0]  # the cell of each (face, side) pair
    valid = ~np.isnan(b[..., 0])
    assert (flags & 4).any() and (not gated or (flags & 2).any()) and not (flags & 0x80).any()
    if precision == ucns.F64:
        assert np.array_equal(flags, oflags)
        assert np.abs(a - b)[valid].max() <= 1e-9 * np.abs(U).max()
    avg = (U if precision == ucns.F64 else U.astype(np.float32)).T.astype(np.float64)[own][:, None, :]
    first = ((flags & 4) != 0)[own][:, None] & valid
    assert np.array_equal(a[first], np.broadcast_to(avg, a.shape)[first])
    rest = valid & ~first
    rho_q, p_q = a[..., 0], 0.4 * (a[..., 4] - 0.5 * (a[..., 1:4] ** 2).sum(-1) / a[..., 0])
    assert (rho_q[rest] > 0).all() and (p_q[rest] > 0).all()
