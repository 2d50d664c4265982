"""Softened M2L tiles hold targets of one octant and one level: adaptive trees
whose octants have targets on many levels, fewer than a tile's 64 on each (a tile
that mixed levels would run one level's tables for the other), at the per-offset
and the sign-class orders, against the oracle."""
import numpy as np
import pytest

from gpu_util import gpu_solve, oracle_tree, rel_l2, say
from paper_2508_02626_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [0, 3, 4, 5, 6, 7, 8, 9, 10])
def test_many_levels_per_octant(p):
    eps, kw = 0.003, dict(leaf_size=8)
    x, q = inputs.plummer(1800, 7)
    t = oracle_tree(x, **kw)
    e = t.export()
    tg = np.diff(e["V_off"].astype(np.int64)) > 0
    counts = np.zeros((8, t.depth + 1), int)
    np.add.at(counts, ((e["morton"][tg] & np.uint64(7)).astype(int), e["level"][tg]), 1)
    assert ((counts > 0).sum(1) >= 3).all() and (counts % 64 != 0).sum() > 20
    pl, phi, fld = gpu_solve(x, q, p, kernel="softened", softening=eps, **kw)
    pl.close()
    ophi, ofld = t.fmm_soft(p, q, eps)
    a, b = rel_l2(phi, ophi), rel_l2(fld, ofld)
    say("  p %d, %d groups: phi %.2e field %.2e" % (p, (counts > 0).sum(), a, b))
    assert a <= 1e-12 and b <= 1e-12
