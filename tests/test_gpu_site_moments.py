"""Site moments as the columns of one solve: against the oracle and against one solve per site, for
column counts that fill chunks or leave them ragged, repeated sites, several solves in a row, and
moment counts around the ring of partials."""
import numpy as np
import pytest

import oracle
import paper_1105_5481_amd as kpm
from paper_1105_5481_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

CASES = [  # (L, spin hopping, sites, M): more than the 4992 sites of one vector that fit an LDS
    ((19, 18, 17), False, 2, 40),
    ((19, 18, 17), True, 5, 33),
    ((20, 20, 20), True, 64, 66),
    ((30, 20, 9), False, 70, 31),       # two solves of 35 columns
    ((120, 51), False, 7, 34),
    ((80, 67), True, 33, 1),
    ((72, 71), True, 3, 2),
    ((24, 23, 12), True, 131, 35),      # three solves, the last smaller
]


@pytest.mark.parametrize("prec", [kpm.F64, kpm.F32])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{'x'.join(map(str, c[0]))}-{'spin' if c[1] else 'real'}-n{c[2]}-M{c[3]}")
def test_columns_match_oracle_and_single_solves(case, prec):
    L, spin, n, M = case
    N = int(np.prod(L))
    op = wl.Lattice(dim=len(L), L=tuple(L) + (1,) * (3 - len(L)), t=1.0, onsite=wl.anderson_onsite(N, 1.0, 7))
    if spin:
        op.hop, op.spinor = wl.HOP_SPIN, wl.spinor_of(*wl.spins_uniform(N, 8))
    a, b = oracle.scale_from_bounds(*gu.oracle_bounds(op), 0.01)
    h = kpm.Hamiltonian(op, a, b, prec)
    g = np.random.default_rng(n)
    sites = g.integers(0, N, n).tolist()
    sites[-1] = sites[0]
    assert kpm.lib().kpm_site_workspace_bytes(h.handle, n, M) > 0
    mus = [m.cpu().numpy() for m in kpm.site_moments(h, sites, M)]
    one = [m.cpu().numpy() for m in kpm.moments_batched([h] * n, M, 1, wl.VEC_UNIT, [0] * n, sites)]
    h.free()
    assert np.array_equal(mus[0], mus[-1])
    for k in range(n):
        # the vectors are the same; at most the order of the FP64 partial sums (of at most N R = N
        # products of modulus <= 1, normalised by 1) differs
        assert np.abs(mus[k] - one[k]).max() <= (1e-15 if prec == kpm.F64 else 1e-13), k
    for k in {0, n // 2, n - 1}:
        ref = gu.oracle_moments(op, a, b, M, 1, wl.VEC_UNIT, 0, sites[k])
        (gu.assert_fp64 if prec == kpm.F64 else gu.assert_fp32)(mus[k], ref, f"site {sites[k]}")


def test_site_moments_fall_back():
    """CSR operators, few sites and a single site take one solve per site; bad sites are refused."""
    for op in (wl.lattice_to_csr(wl.square_lattice(50, W=1.0, seed=3)), wl.square_lattice(9, W=1.0, seed=3)):
        a, b = oracle.scale_from_bounds(*gu.oracle_bounds(op), 0.01)
        h = kpm.Hamiltonian(op, a, b, kpm.F64)
        assert kpm.lib().kpm_site_workspace_bytes(h.handle, 4, 20) == 0
        mu = kpm.site_moments(h, [3, 60], 20)[1].cpu().numpy()
        gu.assert_fp64(mu, gu.oracle_moments(op, a, b, 20, 1, wl.VEC_UNIT, 0, 60), "fallback")
        with pytest.raises(kpm.KPMError):
            kpm.site_moments(h, [h.N], 20)
        h.free()
