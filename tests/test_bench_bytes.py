"""CPU check of the bytes the benchmark's rates count: what the kernels read, not
the scheme's indicator matrix where they read less (or, at P4, padding too)."""
import math
import os

import pytest

import bench
from paper_2609_07387_amd import inputs, ucns

pytestmark = pytest.mark.skipif(not os.path.exists(ucns.LIB_PATH), reason="libucns.so not built")


def test_bytes_read_per_cell():
    """Against the scheme's accounting: FP64 P2 one value for 45, FP32 P2 one
    more, P3 16 for 190, P4 720 for 595 and ids in groups of four (80 and 22
    members: 80 and 24 ids)."""
    hex2 = ucns.Mesh(inputs.periodic_hex_mesh(6), order=2)
    hex3 = ucns.Mesh(inputs.hex_box_mesh((7, 7, 7), (1.0,) * 3, (True,) * 3), order=3)
    hex4 = ucns.Mesh(inputs.hex_box_mesh((9, 9, 9), (1.0,) * 3, (True,) * 3), order=4)

    def extra(lm, precision, **kw):
        return (bench.recon_bytes_per_cell(lm, precision, read=True, **kw)
                - bench.recon_bytes_per_cell(lm, precision, **kw))

    assert extra(hex2, ucns.F64) == 8 * (1 - 45)
    assert extra(hex2, ucns.F64, grad=True) == 8 * (1 - 45)
    assert extra(hex2, ucns.F32) == 4 * (46 - 45)
    assert extra(hex2, ucns.F32, linear=True, gate=True) == 0
    assert extra(hex3, ucns.F64) == 8 * (16 - 190) and extra(hex3, ucns.F32) == 4 * (16 - 190)
    assert (hex4.mc_pad, hex4.md_pad, hex4.nd_max) == (80, 22, 6)
    assert extra(hex4, ucns.F64) == 8 * (720 - 595) + 4 * 6 * (24 - 22)
    # and no cell moves more than its share of the arena it reads from
    for lm in (hex2, hex3, hex4):
        for p, t in ((ucns.F64, 8), (ucns.F32, 4)):
            written = t * 5 * lm.nfmax * lm.qmax + 1
            staged = 40 + 64 if lm.K == 34 else 0
            stored = lm.arena_bytes(p) / lm.n_cell
            assert math.isfinite(stored)
            assert bench.recon_bytes_per_cell(lm, p, read=True) - written - staged - 40 <= stored
