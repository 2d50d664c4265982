"""M2P at the edges of its splits: passes of up to 16, 32 and 64 targets and
leaves of more, W lists from one box to more than 64, orders on both sides of the
four-group line, with and without the gradient, against the oracle."""
import numpy as np
import pytest

from gpu_util import oracle_tree, rel_l2, say, to_dev
from paper_2508_02626_amd import inputs

pytestmark = pytest.mark.gpu


def _core(n, m):
    """n points in a cube, m of them in a cube 0.03 as wide: the leaves around
    it have W lists of 1 to more than 60 boxes and 1 to `leaf` targets."""
    x, q = inputs.uniform(n, 90 + n % 7)
    x[:m] = 0.51 + 0.03 * (x[:m] - 0.5)
    return x, q


@pytest.mark.parametrize("p", [1, 10, 11])
@pytest.mark.parametrize("leaf", [1, 16, 17, 32, 33, 64, 65, 130])
def test_m2p_matches_oracle(leaf, p):
    from paper_2508_02626_amd import fmm
    x, q = _core(40 * leaf + 500, 20 * leaf + 250)
    t = oracle_tree(x, leaf_size=leaf)
    w = np.diff(t.export()["W_off"].astype(np.int64))
    ophi, ofld = t.fmm(p, q)
    pl = fmm.Plan(to_dev(x), p, leaf_size=leaf)
    phi, fld = (a.cpu().numpy() for a in pl.evaluate(to_dev(q)))
    only = pl.evaluate(to_dev(q), want_field=False)[0].cpu().numpy()
    pl.close()
    e, f = rel_l2(phi, ophi), rel_l2(fld, ofld)
    say("  leaf %d p %d W lists up to %d: phi %.2e field %.2e" % (leaf, p, w.max(), e, f))
    assert w.max() > 0 and e <= 1e-12 and f <= 1e-12 and rel_l2(only, ophi) <= 1e-12
