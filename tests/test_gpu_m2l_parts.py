"""M2L tiles split into parts: from the most parts (a few tiles) through the
fewer of middling trees to the fixed split of large ones, at orders on both
sides of the slot / sign-class and the add / store lines, against the oracle."""
import pytest

from gpu_util import gpu_solve, oracle_tree, rel_l2, say
from paper_2508_02626_amd import inputs

pytestmark = pytest.mark.gpu

# (points, leaf size): about 9, 30, 100 and 250 tiles of 64 targets
TREES = [(1500, 16), (6000, 8), (17000, 6), (45000, 6)]


@pytest.mark.parametrize("p", [0, 4, 5, 6, 11, 12])
@pytest.mark.parametrize("n,leaf", TREES)
def test_parts_match_oracle(n, leaf, p):
    if p > 6 and n > 20000:
        pytest.skip("the large tree is run at orders up to 6 (the oracle's time)")
    x, q = inputs.uniform(n, 60 + p)
    pl, phi, fld = gpu_solve(x, q, p, leaf_size=leaf)
    ophi, ofld = oracle_tree(x, leaf_size=leaf).fmm(p, q)
    e, f = rel_l2(phi, ophi), rel_l2(fld, ofld)
    say("  n %d leaf %d p %d boxes %d: phi %.2e field %.2e" % (n, leaf, p, pl.sizes()["boxes"], e, f))
    assert e <= 1e-12 and f <= 1e-12


@pytest.mark.parametrize("p", [3, 5, 7, 13])
@pytest.mark.parametrize("n,leaf", TREES[:3])
def test_parts_mixed_within_the_mixed_bound(n, leaf, p):
    x, q = inputs.plummer(n, 70 + p)
    _, phi, fld = gpu_solve(x, q, p, leaf_size=leaf, precision="mixed")
    _, rphi, rfld = gpu_solve(x, q, p, leaf_size=leaf)
    assert rel_l2(phi, rphi) <= 3e-7 and rel_l2(fld, rfld) <= 1e-6
