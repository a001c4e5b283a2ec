"""FP64 dot products keep their error terms whatever the size of the products: moments of operators scaled
far below 1 (products of 1e-14, whose signs cancel) and of scales that do not enclose the spectrum
(vectors that grow without bound) agree with the oracle to the last bit or one beside it, in every kind of
lattice and sparse kernel.  Both sides evaluate the same vectors; a sum of products p in pairs is off by
about 2^-100 of the sum of |p|, so with at most 2^40 of cancellation the two rounded moments differ by one
unit in the last place at most."""
import numpy as np
import pytest

import oracle
import paper_1105_5481_amd as kpm
from paper_1105_5481_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

CASES = {  # (hopping or "csr", L, R, mode of the solve)
    "few sites, one workgroup": ("real", (20, 20), 6, 2),
    "few sites, many launches": ("spin", (12, 13, 13), 24, 2),
    "march": ("spin", (20, 21, 22), 6, 1),
    "march in runs": ("real", (30, 30, 40), 5, 1),
    "blocked 2D": ("real", (301, 77), 8, 3),
    "flat": ("csr", (61, 50), 9, 0),
}


def _ulps(x, y):
    return np.abs(x - y) / np.spacing(np.maximum(np.abs(x), np.abs(y)))


def _op(kind, L):
    N = int(np.prod(L))
    op = wl.Lattice(dim=len(L), L=tuple(L) + (1,) * (3 - len(L)), t=1.0, onsite=wl.anderson_onsite(N, 1.0, 21))
    if kind == "spin":
        op.hop, op.spinor = wl.HOP_SPIN, wl.spinor_of(*wl.spins_uniform(N, 22))
    return wl.lattice_to_csr(op) if kind == "csr" else op


@pytest.mark.parametrize("scale", [1e14, 0.7])
@pytest.mark.parametrize("name", list(CASES))
def test_moments_to_the_last_bit(name, scale):
    kind, L, R, mode = CASES[name]
    op, M = _op(kind, L), 4 if scale > 1 else 50
    vec = wl.VEC_PHASE if kind == "spin" else wl.VEC_RADEMACHER
    h = kpm.Hamiltonian(op, scale, 0.0, kpm.F64)
    s = kpm.Solve(h, M, R, vec, 5, 2)
    assert kpm.lib().kpm_solve_mode(s._s) == mode
    s.close()
    mu = kpm.moments(h, M, R, vec, 5, 2).cpu().numpy()
    h.free()
    ref = gu.oracle_moments(op, scale, 0.0, M, R, vec, 5, 2)
    u = _ulps(mu, ref)
    print(f"  {name} scale {scale}: {u.max():.1f} ulp at most, |mu| {np.abs(ref).min():.2e} .. {np.abs(ref).max():.2e}", flush=True)
    assert u.max() <= 1.0


@pytest.mark.parametrize("scale", [1e14, 0.7])
def test_site_moments_to_the_last_bit(scale):
    op, M = _op("spin", (19, 18, 17)), 4 if scale > 1 else 50
    h = kpm.Hamiltonian(op, scale, 0.0, kpm.F64)
    at = [5, 3000, 77]
    mus = kpm.site_moments(h, at, M)
    for mu, i in zip(mus, at):
        ref = gu.oracle_moments(op, scale, 0.0, M, 1, wl.VEC_UNIT, 0, i)
        assert _ulps(mu.cpu().numpy(), ref).max() <= 1.0, i
    h.free()
