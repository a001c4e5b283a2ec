"""CSR steps walk a row eight entries at a time: rows of no entry, of one, and at the multiples of eight,
with the stored diagonal first, inside or absent, over tiles of one chunk per thread and of more, with a
ragged last tile.  Moments match the oracle, and chunked and batched solves equal the plain one bit for bit."""
import numpy as np
import pytest

import oracle
import paper_1105_5481_amd as kpm
from paper_1105_5481_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
STATIC = 64 << 20   # bytes of the library's own scratch


def _rows(n, cplx, seed):
    """A Hermitian matrix of 2 x 2 .. 19 x 19 full blocks down the diagonal (rows of 1 .. 18 off-diagonal
    entries), two empty rows before each block, diagonals stored for every other block."""
    rng = np.random.default_rng(seed)
    rp, col, val = [0], [], []
    i, k = 0, 0
    while i < n:
        for _ in range(min(2, n - i)):      # empty rows
            rp.append(len(col))
            i += 1
        b = min(2 + k % 18, n - i)
        h = rng.uniform(-1, 1, (b, b)) + (1j * rng.uniform(-1, 1, (b, b)) if cplx else 0)
        h = h + h.conj().T
        for r in range(b):
            js = [j for j in range(b) if k % 2 or j != r]
            col += [i + j for j in js]
            val += [h[r, j] for j in js]
            rp.append(len(col))
        i, k = i + b, k + 1
    val = np.array(val, dtype=complex)
    return wl.CSR(n=n, row_ptr=np.array(rp, dtype=np.int64), col=np.array(col, dtype=np.int32),
                  val_re=np.ascontiguousarray(val.real), val_im=np.ascontiguousarray(val.imag) if cplx else None)


@pytest.mark.parametrize("prec", [kpm.F64, kpm.F32])
@pytest.mark.parametrize("n,cplx,R,tpt", [(3001, True, 5, 4), (3001, False, 3, 2), (5003, True, 1, 1),
                                          (4997, False, 17, 4), (2600, True, 8, 4)])
def test_csr_rows(n, cplx, R, tpt, prec):
    op, M = _rows(n, cplx, 7), 37
    vec = wl.VEC_PHASE if cplx else wl.VEC_RADEMACHER
    a, b = oracle.scale_from_bounds(*gu.oracle_bounds(op), 0.01)
    ref = gu.oracle_moments(op, a, b, M, R, vec, 5, 2)
    h = kpm.Hamiltonian(op, a, b, prec)
    with kpm.launch_settings(small=0, elems_per_thread=tpt):
        s = kpm.Solve(h, M, R, vec, 5, 2)
        assert kpm.lib().kpm_solve_mode(s._s) == 0
        s.close()
        mu = kpm.moments(h, M, R, vec, 5, 2).cpu().numpy()
        (gu.assert_fp64 if prec == kpm.F64 else gu.assert_fp32)(mu, ref, "csr rows")
        for chunk in (1, 7):
            s = kpm.Solve(h, M, R, vec, 5, 2)
            while s.advance(chunk) > 0:
                pass
            assert np.array_equal(s.finish().cpu().numpy(), mu), chunk
            s.close()
        got = kpm.moments_batched([h, h], [M, M], [R, R], vec, [5, 5], [2, 2])
        assert all(np.array_equal(g.cpu().numpy(), mu) for g in got)
    h.free()


@pytest.mark.parametrize("kind,R,M", [("csr", 71, 75), ("spin", 8, 551), ("real", 2, 62)])
def test_scratch_limit(kind, R, M):
    """Solves that fit the static scratch with coarse tiles only: they take those, and run there."""
    if kind == "csr":
        n = 103733
        op = wl.CSR(n=n, row_ptr=np.arange(n + 1, dtype=np.int64), col=((np.arange(n) ^ 1) % n).astype(np.int32),
                    val_re=np.full(n, 0.5))
        op.col[-1], op.val_re[-1] = n - 1, 0.25
    else:
        L = (353, 731) if kind == "spin" else (890, 1172)
        N = L[0] * L[1]
        op = wl.Lattice(dim=2, L=L + (1,), t=1.0, onsite=wl.anderson_onsite(N, 1.0, 3))
        if kind == "spin":
            theta, phi = wl.spins_uniform(N, 3)
            op.hop, op.spinor, op.theta, op.phi = wl.HOP_SPIN, wl.spinor_of(theta, phi), theta, phi
    vec = wl.VEC_RADEMACHER if kind == "csr" else wl.VEC_PHASE
    a, b = oracle.scale_from_bounds(*gu.oracle_bounds(op), 0.01)
    h = kpm.Hamiltonian(op, a, b, kpm.F32)
    size = h.workspace_bytes(M, R, vec)
    assert 0.9 * STATIC < size <= STATIC
    mu = kpm.moments(h, M, R, vec, 5, 2).cpu().numpy()
    assert np.array_equal(kpm.moments_static(h, M, R, vec, 5, 2).cpu().numpy(), mu)
    with kpm.launch_settings(tblock=0, elems_per_thread=2):   # one step per launch, other tiles
        gu.assert_fp32(kpm.moments(h, M, R, vec, 5, 2).cpu().numpy(), mu, "scratch limit")
    h.free()
