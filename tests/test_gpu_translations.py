"""M2M and L2L by parity classes: orders at the ends of the row-tile counts, trees
with few and with many parents of a level (on both sides of the lines that split
a row tile's products over wavefronts), two levels only, and lone chains of
children, against the oracle."""
import numpy as np
import pytest

from gpu_util import oracle_tree, rel_l2, say, to_dev
from paper_2508_02626_amd import fmm, inputs

pytestmark = pytest.mark.gpu


def _chain():
    """Pairs of nearly coincident points: chains of boxes with one child each."""
    x, q = inputs.uniform(240, 31)
    x[120:] = x[:120] + 1e-4
    return x, q


TREES = {
    "depth2": (lambda: inputs.uniform(700, 21), dict(uniform_depth=2, root=[0, 0, 0, 1])),
    "depth3": (lambda: inputs.uniform(3000, 22), dict(uniform_depth=3, root=[0, 0, 0, 1])),
    "depth4_sparse": (lambda: inputs.uniform(300, 23), dict(uniform_depth=4, root=[0, 0, 0, 1])),
    "plummer": (lambda: inputs.plummer(2500, 24), dict(leaf_size=20)),
    "chain": (_chain, dict(leaf_size=1)),
}


@pytest.mark.parametrize("p", [5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16])
@pytest.mark.parametrize("tree", list(TREES))
def test_translations_match_oracle(tree, p):
    if p > 8 and tree == "depth4_sparse":
        pytest.skip("the oracle's time; its levels are those of depth3 and one more")
    gen, kw = TREES[tree]
    x, q = gen()
    pl = fmm.Plan(to_dev(x), p, **kw)
    phi, fld = (a.cpu().numpy() for a in pl.evaluate(to_dev(q)))
    pl.close()
    ophi, ofld = oracle_tree(x, **kw).fmm(p, q)
    e, f = rel_l2(phi, ophi), rel_l2(fld, ofld)
    say("  %s p %d: phi %.2e field %.2e" % (tree, p, e, f))
    assert e <= 1e-12 and f <= 1e-12


@pytest.mark.parametrize("n,leaf", [(60000, 8), (200000, 6)])
def test_many_parents_agree_between_orders(n, leaf):
    """Thousands of parents per level (one wavefront per row tile, unsplit column
    classes): the distance of order 8 from order 11 is that of the truncation."""
    x, q = inputs.uniform(n, 25)
    q = np.abs(q)
    out = []
    for p in (8, 11):
        pl = fmm.Plan(to_dev(x), p, leaf_size=leaf)
        out.append(pl.evaluate(to_dev(q), want_field=False)[0].cpu().numpy())
        pl.close()
    e = rel_l2(out[0], out[1])
    say("  n %d: order 8 against 11 %.2e" % (n, e))
    assert 1e-12 < e <= 1e-5
