"""March solves cut into segments of one plane and up, walked in runs inside shared launches, and the
even placement of a wave's items over the XCDs: every batched result equals its solo solve bit for
bit, whatever runs and ranges the launch gave it, and the FP64 ones match the oracle."""
import numpy as np
import pytest

import oracle
import paper_1105_5481_amd as kpm
from paper_1105_5481_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def _ops(shapes, spin):
    out = []
    for k, (Lx, Ly, Lz) in enumerate(shapes):
        N = Lx * Ly * max(Lz, 1)
        op = wl.Lattice(dim=3 if Lz else 2, L=(Lx, Ly, max(Lz, 1)), t=1.0, onsite=wl.anderson_onsite(N, 1.0, 50 + k))
        if spin:
            op.hop, op.spinor = wl.HOP_SPIN, wl.spinor_of(*wl.spins_uniform(N, 80 + k))
        out.append(op)
    return out


# extents along the march axis below, at and above the run length; one instance of many XCD shares;
# a handful of launches with fewer blocks than runs need
SHAPES = {
    "many": [(9 + k % 5, 7 + k % 4, 1 + (5 * k) % 23) for k in range(40)],
    "one large": [(40, 41, 42)] + [(6, 5, 17 + k) for k in range(3)],
    "few": [(11, 13, 9), (5, 6, 3)],
    "flat": [(50 + k, 33, 0) for k in range(12)],
}


@pytest.mark.parametrize("prec", [kpm.F64, kpm.F32])
@pytest.mark.parametrize("spin", [False, True])
@pytest.mark.parametrize("kind", list(SHAPES))
def test_runs_and_even_shares_equal_solo(kind, spin, prec):
    ops = _ops(SHAPES[kind], spin)
    M, R, vec = 23, 9, wl.VEC_PHASE
    ab = [oracle.scale_from_bounds(*gu.oracle_bounds(op), 0.01) for op in ops]
    with kpm.launch_settings(small=0, tblock=0):
        hs = [kpm.Hamiltonian(op, a, b, prec) for op, (a, b) in zip(ops, ab)]
        n = len(hs)
        seeds, insts = [3 + k for k in range(n)], list(range(n))
        solo = [kpm.moments(h, M, R, vec, seeds[k], k).cpu().numpy() for k, h in enumerate(hs)]
        for kw in (dict(), dict(wave_mib=1), dict(max_blocks=8)):
            with kpm.launch_settings(**kw):
                got = [m.cpu().numpy() for m in kpm.moments_batched(hs, M, R, vec, seeds, insts)]
            for k in range(n):
                assert np.array_equal(got[k], solo[k]), (kw, k)
        for h in hs:
            h.free()
    for k in (0, n - 1):
        ref = gu.oracle_moments(ops[k], *ab[k], M, R, vec, seeds[k], k)
        (gu.assert_fp64 if prec == kpm.F64 else gu.assert_fp32)(solo[k], ref, f"{kind} {k}")
