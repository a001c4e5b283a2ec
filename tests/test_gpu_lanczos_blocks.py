"""The Lanczos launches at the edges of their block counts: one block, counts that are and are not a
multiple of the XCDs, the cap of 512 and the larger cap of vectors above 2^21 chunks."""
import numpy as np
import pytest

import paper_1105_5481_amd as kpm
from paper_1105_5481_amd import workloads as wl
from tests import gpu_util as gu
from tests.test_gpu_lanczos import COEF_TOL, _oracle_lanczos

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,k", [((3, 2), 3), ((16, 16), 40), ((17, 151), 30), ((64, 32), 512), ((331, 397), 12),
                                 ((1500, 1400), 3)], ids=str)
def test_lanczos_block_counts(L, k):
    N = L[0] * L[1]
    op = wl.Lattice(dim=2, L=(*L, 1), t=1.0, onsite=wl.anderson_onsite(N, 1.0, 5))
    h = kpm.Hamiltonian(op, 2.0, 0.1, kpm.F64)
    got = kpm.lanczos_bounds(h, k, 3, 0.005, clamp=None)
    h.free()
    al, be = _oracle_lanczos(op, 2.0, 0.1, k, 3)
    m = min(int(got["m"]), 40)   # beyond loss of orthogonality the coefficients follow the rounding
    assert np.abs(got["alpha"][:m] - al[:m]).max() <= COEF_TOL
    assert np.abs(got["beta"][:m - 1] - be[:m - 1]).max(initial=0.0) <= COEF_TOL
    lo, hi = gu.oracle_bounds(op)
    assert lo - 0.1 <= got["e_lo"] < got["e_hi"] <= hi + 0.1


@pytest.mark.parametrize("L", [(16, 12, 20), (61, 43)], ids=str)
def test_lanczos_phase_start_is_normalised_exactly(L):
    """<xi|xi> of phase vectors is no whole number: with it and every later sum rounded once, the
    coefficients are the oracle's bit for bit, also where rounding errors have grown."""
    theta, phi = wl.spins_uniform(int(np.prod(L)), 23)
    op = wl.Lattice(dim=len(L), L=L + (1,) * (3 - len(L)), t=1.0, hop=wl.HOP_SPIN, spinor=wl.spinor_of(theta, phi))
    h = kpm.Hamiltonian(op, 4.0, 0.0, kpm.F64)
    got = kpm.lanczos_bounds(h, 150, 3, 0.005, clamp=None)
    h.free()
    al, be = _oracle_lanczos(op, 4.0, 0.0, 150, 3)
    assert np.array_equal(got["alpha"], al[:len(got["alpha"])])
    assert np.array_equal(got["beta"], be[:len(got["beta"])])
