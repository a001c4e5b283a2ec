"""Shared launches of flat solves (CSR, and lattices without the march kernels) with members of 48 to 63
tiles, which the placement splits over the XCDs where they exceed an even share: every member of a static
and of a dynamic batch equals its solo solve bit for bit, and one of them matches the oracle."""
import numpy as np
import pytest

import oracle
import paper_1105_5481_amd as kpm
from paper_1105_5481_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def _csr(n, cplx, seed):
    """A random sparse Hermitian matrix: the diagonal and, for each of three permutations p, entries at
    (i, p(i)) and (p(i), i)."""
    g = np.random.default_rng(seed)
    i = np.arange(n)
    cols, vals = [i], [g.uniform(-0.5, 0.5, n) + 0j]
    for _ in range(3):
        p = g.permutation(n)
        q = np.argsort(p)
        v = g.uniform(-1, 1, n) + (1j * g.uniform(-1, 1, n) if cplx else 0)
        v[p == i] = v[p == i].real
        cols += [p, q]
        vals += [v, v[q].conj()]
    col, val = np.stack(cols, 1), np.stack(vals, 1)
    return wl.CSR(n=n, row_ptr=np.arange(n + 1, dtype=np.int64) * col.shape[1], col=col.reshape(-1).astype(np.int32),
                  val_re=np.ascontiguousarray(val.real.reshape(-1)),
                  val_im=np.ascontiguousarray(val.imag.reshape(-1)) if cplx else None)


def _lattice(L, seed):
    return wl.Lattice(dim=3, L=L, t=1.0, onsite=wl.anderson_onsite(L[0] * L[1] * L[2], 1.0, seed))


# (operators, precision, R, settings); tiles of 256 chunks (lattices: elems_per_thread = 1)
CASES = {
    "nine of 50 tiles": (lambda: [_csr(3200, False, k) for k in range(9)], kpm.F32, 16, {}),
    "eight, one of 63": (lambda: [_csr(2700 + 30 * k, True, k) for k in range(7)] + [_csr(8000, True, 9)], kpm.F64, 2, {}),
    "twelve of 59": (lambda: [_csr(3000, True, k) for k in range(12)], kpm.F32, 10, {}),
    "flat lattices": (lambda: [_lattice((17, 16, 13 - k % 2), k) for k in range(10)], kpm.F64, 7,
                      dict(march=0, elems_per_thread=1)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_flat_members_equal_solo(name):
    make, prec, R, settings = CASES[name]
    ops, M = make(), 21
    vec = wl.VEC_PHASE if getattr(ops[0], "val_im", None) is not None else wl.VEC_RADEMACHER
    ab = [oracle.scale_from_bounds(*gu.oracle_bounds(op), 0.01) for op in ops]
    n = len(ops)
    with kpm.launch_settings(**settings):
        hs = [kpm.Hamiltonian(op, a, b, prec) for op, (a, b) in zip(ops, ab)]
        s = kpm.Solve(hs[0], M, R, vec, 3, 0)
        assert kpm.lib().kpm_solve_mode(s._s) == 0
        s.close()
        solo = [kpm.moments(h, M, R, vec, 3 + k, k).cpu().numpy() for k, h in enumerate(hs)]
        got = kpm.moments_batched(hs, M, R, vec, [3 + k for k in range(n)], list(range(n)))
        for k in range(n):
            assert np.array_equal(got[k].cpu().numpy(), solo[k]), ("static", k)
        ss = [kpm.Solve(h, M, R, vec, 3 + k, k) for k, h in enumerate(hs)]
        batch = kpm.Batch(capacity=n)
        for s in ss:
            batch.add(s)
        while any(s.remaining > 0 for s in ss):
            batch.advance(4)
        for k, s in enumerate(ss):
            batch.remove(s)
            assert np.array_equal(s.finish().cpu().numpy(), solo[k]), ("dynamic", k)
            s.close()
        batch.free()
        for h in hs:
            h.free()
    ref = gu.oracle_moments(ops[-1], *ab[-1], M, R, vec, 3 + n - 1, n - 1)
    (gu.assert_fp64 if prec == kpm.F64 else gu.assert_fp32)(solo[-1], ref, name)


@pytest.mark.parametrize("sites", [9, 12])
def test_csr_site_moments(sites):
    """Local moments of a CSR operator: one solve per site in one batch, 55 tiles each."""
    op, M = _csr(14000, True, 4), 20
    a, b = oracle.scale_from_bounds(*gu.oracle_bounds(op), 0.01)
    h = kpm.Hamiltonian(op, a, b, kpm.F64)
    at = [37 * k * k + 5 for k in range(sites)]
    mus = [m.cpu().numpy() for m in kpm.site_moments(h, at, M)]
    for k, i in enumerate(at):
        assert np.array_equal(mus[k], kpm.moments(h, M, 1, wl.VEC_UNIT, 0, i).cpu().numpy()), k
    gu.assert_fp64(mus[-1], gu.oracle_moments(op, a, b, M, 1, wl.VEC_UNIT, 0, at[-1]), "csr site")
    h.free()
