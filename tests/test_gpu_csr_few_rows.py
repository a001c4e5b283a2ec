"""CSR operators of few rows run in one workgroup's LDS up to 10240 entries and 32 per row; with more or
longer rows they take the flat kernels.  Moments match the oracle on either side of both lines."""
import numpy as np
import pytest

import oracle
import paper_1105_5481_amd as kpm
from paper_1105_5481_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def _circulant(n, per, seed):
    """n rows of exactly `per` entries (odd): the diagonal and per // 2 neighbours on either side."""
    g = np.random.default_rng(seed)
    col, val = np.empty((n, per), dtype=np.int32), np.empty((n, per))
    i = np.arange(n)
    col[:, 0], val[:, 0] = i, g.uniform(-0.5, 0.5, n)
    for k in range(1, per // 2 + 1):
        w = g.uniform(-1, 1, n)          # w[i] links i and i + k
        col[:, 2 * k - 1], val[:, 2 * k - 1] = (i + k) % n, w
        col[:, 2 * k], val[:, 2 * k] = (i - k) % n, np.roll(w, k)
    return wl.CSR(n=n, row_ptr=np.arange(n + 1, dtype=np.int64) * per, col=col.reshape(-1), val_re=val.reshape(-1))


@pytest.mark.parametrize("prec", [kpm.F64, kpm.F32])
@pytest.mark.parametrize("n,per,R,mode", [(2048, 5, 40, 2), (930, 11, 3, 2), (931, 11, 3, 0), (300, 31, 9, 2), (300, 33, 9, 0),
                                          (1000, 401, 5, 0), (12, 3, 2, 2)])
def test_few_rows(n, per, R, mode, prec):
    op, M = _circulant(n, per, 3), 26
    a, b = oracle.scale_from_bounds(*gu.oracle_bounds(op), 0.01)
    h = kpm.Hamiltonian(op, a, b, prec)
    s = kpm.Solve(h, M, R, wl.VEC_RADEMACHER, 5, 2)
    assert kpm.lib().kpm_solve_mode(s._s) == mode
    s.close()
    mu = kpm.moments(h, M, R, wl.VEC_RADEMACHER, 5, 2).cpu().numpy()
    h.free()
    ref = gu.oracle_moments(op, a, b, M, R, wl.VEC_RADEMACHER, 5, 2)
    (gu.assert_fp64 if prec == kpm.F64 else gu.assert_fp32)(mu, ref, f"{n} rows of {per}")
