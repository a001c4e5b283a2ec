"""Tiles of the 2D blocked passes where they can go wrong: chunk groups that do not divide a site's
chunks (the last group is smaller), windows barely within the row, the row of a single tile, segments
shorter than a pass is deep, columns of just two halos, and items that do not divide over the XCDs."""
import numpy as np
import pytest

import oracle
import paper_1105_5481_amd as kpm
from paper_1105_5481_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

# (Lx, Ly, R, precision, spin hopping, KPM_LAUNCH_TB_GROUP, KPM_LAUNCH_TBLOCK, march_items)
TILES = [
    (97, 31, 21, kpm.F64, False, -1, -1, 512),    # C = 11
    (97, 31, 21, kpm.F64, False, 4, 5, 512),
    (131, 23, 19, kpm.F32, False, 2, 6, 4),       # C = 5, few and long segments
    (131, 23, 7, kpm.F64, True, 3, 6, 100000),    # C = 7, shortest segments
    (64, 13, 34, kpm.F32, True, -1, 6, 512),      # C = 17, columns of two halos
    (257, 12, 1, kpm.F64, True, -1, 6, 512),      # C = 1: 512-site rule not met, one step per launch
    (513, 12, 1, kpm.F64, True, -1, 6, 512),      # C = 1: three windows of 256 sites
    (700, 40, 3, kpm.F32, False, 1, -1, 64),      # more items than slots
]


@pytest.mark.parametrize("case", TILES, ids=lambda c: f"{c[0]}x{c[1]}-R{c[2]}-{'f64' if c[3] == 0 else 'f32'}-g{c[5]}-d{c[6]}")
def test_blocked_tiles(case):
    Lx, Ly, R, prec, spin, group, depth, items = case
    N, M, vec = Lx * Ly, 45, wl.VEC_PHASE if spin else wl.VEC_RADEMACHER
    op = wl.Lattice(dim=2, L=(Lx, Ly, 1), t=1.0, onsite=wl.anderson_onsite(N, 1.0, 3))
    if spin:
        op.hop, op.spinor = wl.HOP_SPIN, wl.spinor_of(*wl.spins_uniform(N, 4))
    a, b = oracle.scale_from_bounds(*gu.oracle_bounds(op), 0.01)
    with kpm.launch_settings(small=0, tblock=depth, tb_group=group, march_items=items):
        h = kpm.Hamiltonian(op, a, b, prec)
        s = kpm.Solve(h, M, R, vec, 8, 0)
        mode, deepest = kpm.lib().kpm_solve_mode(s._s), kpm.lib().kpm_solve_depth(s._s)
        s.close()
        h.free()
        got = gu.gpu_moments(op, a, b, prec, M, R, vec, seed=8)
    blocked = Lx != 257
    assert (mode == 3) == blocked and (deepest > 1) == blocked
    if depth > 0 and blocked:
        assert deepest == depth
    with kpm.launch_settings(small=0, tblock=0):
        one = gu.gpu_moments(op, a, b, prec, M, R, vec, seed=8)
    ref = gu.oracle_moments(op, a, b, M, R, vec, 8)
    # the vectors are those of one-step launches; only the order of the FP64 partial sums differs
    if prec == kpm.F64:
        gu.assert_fp64(got, ref, "tiles")
        assert np.abs(got - one).max() <= 1e-15
    else:
        gu.assert_fp32(got, ref, "tiles")
        assert np.abs(got - one).max() <= 1e-12
