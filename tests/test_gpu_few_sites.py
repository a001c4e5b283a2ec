"""Solves of few sites, one workgroup per group of a site's chunks: sizes at the edges of waves, of the
workgroup and of the two-chunk threads, chunk counts that do not divide into groups, solves whose state
lives in the workspace between launches (few and many steps per ring of partials), and shared launches.
Moments match the oracle, and chunked, batched and dynamic solves equal the plain one bit for bit."""
import numpy as np
import pytest

import oracle
import paper_1105_5481_amd as kpm
from paper_1105_5481_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def _op(kind, L, seed):
    N = int(np.prod(L))
    op = wl.Lattice(dim=len(L), L=tuple(L) + (1,) * (3 - len(L)), t=1.0, onsite=wl.anderson_onsite(N, 1.0, seed))
    if kind == "spin":
        theta, phi = wl.spins_uniform(N, seed)
        op.hop, op.spinor, op.theta, op.phi = wl.HOP_SPIN, wl.spinor_of(theta, phi), theta, phi
    return wl.lattice_to_csr(op) if kind == "csr" else op


CASES = [  # (kind, L, R, M): C chunks per site in FP64 / FP32
    ("real", (5, 5, 5), 1, 30),          # two waves, one group
    ("spin", (4, 4, 4), 37, 1),          # one wave, start vectors only
    ("real", (3, 2), 70, 33),            # 6 sites: groups of a wave's worth of chunks
    ("spin", (9, 7), 40, 41),            # 63 sites: 40 / 20 chunks in groups of 3 / 2
    ("real", (32, 32), 8, 64),           # a full workgroup
    ("spin", (32, 33), 5, 35),           # two chunks per thread, the second ragged
    ("spin", (12, 13, 13), 24, 27),      # 2028 sites, state in the workspace
    ("real", (64, 32), 33, 1300),        # 2048 sites; more steps than a ring of partials
    ("real", (45, 45), 2, 20),           # 2025 sites, all steps in one launch
    ("real", (61, 47), 2, 25),           # 2867 sites: chunks from the LDS alone
    ("csr", (11, 9, 8), 13, 26),
    ("csr", (40, 50), 40, 18),
]


@pytest.mark.parametrize("prec", [kpm.F64, kpm.F32])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}{'x'.join(map(str, c[1]))}-R{c[2]}-M{c[3]}")
def test_few_sites(case, prec):
    kind, L, R, M = case
    vec = wl.VEC_PHASE if kind == "spin" else wl.VEC_RADEMACHER
    op = _op(kind, L, 61)
    a, b = oracle.scale_from_bounds(*gu.oracle_bounds(op), 0.01)
    ref = gu.oracle_moments(op, a, b, M, R, vec, 5, 2)
    h = kpm.Hamiltonian(op, a, b, prec)
    s = kpm.Solve(h, M, R, vec, 5, 2)
    assert kpm.lib().kpm_solve_mode(s._s) == 2
    s.close()
    mu = kpm.moments(h, M, R, vec, 5, 2).cpu().numpy()
    (gu.assert_fp64 if prec == kpm.F64 else gu.assert_fp32)(mu, ref, "few sites")
    for chunk in (1, 7, 10 ** 6):
        s = kpm.Solve(h, M, R, vec, 5, 2)
        while s.advance(chunk) > 0:
            pass
        assert np.array_equal(s.finish().cpu().numpy(), mu), chunk
        s.close()
    got = kpm.moments_batched([h, h], [M, M], [R, R], vec, [5, 5], [2, 2])
    assert all(np.array_equal(g.cpu().numpy(), mu) for g in got)
    h.free()


def test_few_sites_share_launches():
    """Solves of different sizes, groups and step counts in one dynamic batch, joining late."""
    specs = [("real", (32, 33), 20, 90), ("real", (5, 6), 3, 41), ("spin", (12, 13, 13), 24, 150),
             ("spin", (6, 6, 6), 9, 33), ("real", (20, 20, 5), 31, 700), ("real", (16, 16, 16), 8, 60)]
    for prec in (kpm.F64, kpm.F32):
        hs, ss, solo = [], [], []
        for k, (kind, L, R, M) in enumerate(specs):
            op = _op(kind, L, 70 + k)
            h = kpm.Hamiltonian(op, *oracle.scale_from_bounds(*gu.oracle_bounds(op), 0.01), prec)
            vec = wl.VEC_PHASE if kind == "spin" else wl.VEC_RADEMACHER
            solo.append(kpm.moments(h, M, R, vec, k, 1).cpu().numpy())
            ss.append(kpm.Solve(h, M, R, vec, k, 1))
            hs.append(h)
        batch = kpm.Batch(capacity=8)
        for s in ss[:3]:
            batch.add(s)
        batch.advance(5)
        for s in ss[3:]:
            batch.add(s)
        q = 0
        while any(s.remaining > 0 for s in ss):
            batch.advance((64, 3, 17)[q % 3])
            q += 1
        for k, s in enumerate(ss):
            batch.remove(s)
            assert np.array_equal(s.finish().cpu().numpy(), solo[k]), k
            s.close()
            hs[k].free()
        batch.free()
