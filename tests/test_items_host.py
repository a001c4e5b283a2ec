"""Host check of the work items of shared launches: whatever split the placement gives a member, the
blocks of the grid run each of its items exactly once, in every kind of kernel."""
import ctypes

import numpy as np
import pytest

import paper_1105_5481_amd as kpm

FLAT, MARCH, BLOCKED, BLOCKED3 = 0, 1, 3, 4


@pytest.fixture(scope="module")
def L():
    return kpm.lib()


def _missed(L, mode, static, units, segs, planes, xcd, cap=2048, run=3):
    u, s, p = (np.array(v, dtype=np.uint32) for v in (units, segs, planes))
    x = np.array(xcd, dtype=np.int32)
    nb = np.minimum((u * s + 7) // 8 * 8, cap).astype(np.uint32)
    P = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    return L.kpm_selftest_items(mode, run, static, len(u), P(u), P(s), P(p), P(nb), P(x)), x


@pytest.mark.parametrize("static", [0, 1])
@pytest.mark.parametrize("mode", [FLAT, BLOCKED, BLOCKED3])
@pytest.mark.parametrize("sizes", [[50] * 9, [48, 20, 20, 20, 20, 20, 20, 20], [63] + [11] * 9, [59] * 12, [200, 50, 50]],
                         ids=["nine50", "one48", "one63", "twelve59", "few"])
def test_members_split_by_the_placement(L, sizes, mode, static):
    """Members of 48 to 63 tiles, which come without a split of their own and get one from the placement."""
    n = len(sizes)
    bad, xcd = _missed(L, mode, static, sizes, [1] * n, [1] * n, [0 if t < 64 else 1 for t in sizes])
    assert bad == 0
    if sizes == [50] * 9:
        assert xcd.max() > 0 and xcd.min() == 0    # the last of them is split


@pytest.mark.parametrize("static", [0, 1])
@pytest.mark.parametrize("mode", [FLAT, MARCH, BLOCKED, BLOCKED3])
@pytest.mark.parametrize("case", range(8))
def test_every_item_once(L, case, mode, static):
    """Random members under every split (0 none, 1 by units, 2 by segments, 3 evenly), block caps below
    the number of items, and march segments short enough to be walked in runs."""
    g = np.random.default_rng(100 + case)
    n = [1, 2, 7, 8, 9, 17, 40, 120][case]
    units = np.maximum(1, np.exp(g.uniform(0, np.log(80), n)).astype(int))
    segs = np.ones(n, int) if mode == FLAT else g.integers(1, 30, n)
    planes = g.integers(1, 5, n) if mode == MARCH else np.ones(n, int)
    xcd = [int(g.choice([0, 3] + ([1] if u >= 8 else []) + ([2] if s >= 8 else []))) if u * s >= 64 else 0
           for u, s in zip(units, segs)]
    for cap in (8, 64, 2048):
        for run in (3, 4):    # planes of a run
            assert _missed(L, mode, static, units, segs, planes, xcd, cap, run)[0] == 0, (cap, run)
