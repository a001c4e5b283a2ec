"""Site moments with one to 256 columns per solve: from one sum per wave to two per thread of the column
sums, several solves in a row, the last smaller.  Repeated sites agree, and sites match the oracle."""
import numpy as np
import pytest

import oracle
import paper_1105_5481_amd as kpm
from paper_1105_5481_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

CASES = [  # (L, spin hopping, sites, M)
    ((30, 20, 9), False, 300, 21),       # two solves of 150 columns
    ((19, 18, 17), True, 256, 18),       # FP64: 256 chunks per site
    ((19, 18, 17), True, 515, 12),       # three solves, the last of 171
    ((120, 51), False, 2, 40),           # FP64: one chunk, four sums
    ((57, 96), True, 1 + 64, 15),
    ((96, 57), False, 21, 19),           # chunks per site that do not divide a block
]


@pytest.mark.parametrize("prec", [kpm.F64, kpm.F32])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{'x'.join(map(str, c[0]))}-{'spin' if c[1] else 'real'}-n{c[2]}-M{c[3]}")
def test_columns(case, prec):
    L, spin, n, M = case
    N = int(np.prod(L))
    op = wl.Lattice(dim=len(L), L=tuple(L) + (1,) * (3 - len(L)), t=1.0, onsite=wl.anderson_onsite(N, 1.0, 7))
    if spin:
        op.hop, op.spinor = wl.HOP_SPIN, wl.spinor_of(*wl.spins_uniform(N, 8))
    a, b = oracle.scale_from_bounds(*gu.oracle_bounds(op), 0.01)
    h = kpm.Hamiltonian(op, a, b, prec)
    sites = np.random.default_rng(n).integers(0, N, n).tolist()
    sites[-1] = sites[0]
    assert kpm.lib().kpm_site_workspace_bytes(h.handle, n, M) > 0
    mus = [m.cpu().numpy() for m in kpm.site_moments(h, sites, M)]
    h.free()
    assert len(mus) == n and np.array_equal(mus[0], mus[-1])
    assert all(m[0] == 1.0 for m in mus)
    for k in {0, n // 3, n // 2, n - 2}:
        ref = gu.oracle_moments(op, a, b, M, 1, wl.VEC_UNIT, 0, sites[k])
        (gu.assert_fp64 if prec == kpm.F64 else gu.assert_fp32)(mus[k], ref, f"site {sites[k]}")
