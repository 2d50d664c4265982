"""Sizes at which the plan's sort and scans change their way (one block, 512- or
1024-element tiles, scanned histograms; one, two or three scan launches), with
odd and even numbers of digit passes and many equal keys, bit for bit."""
import numpy as np
import pytest

from gpu_util import TREE_KEYS, oracle_tree, say, to_dev
from paper_2508_02626_amd import inputs

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 63, 65, 1024, 1025, 2048, 2049, 4097, 8192, 8193, 16384, 16385, 32768, 32769, 131072, 131073]


def _same_tree(x, **kw):
    from paper_2508_02626_amd import fmm
    pl = fmm.Plan(to_dev(x), 2, **kw)
    g, t = pl.export_tree(), oracle_tree(x, **kw)
    o = t.export()
    for k in TREE_KEYS:
        assert np.array_equal(g[k].astype(np.int64), o[k].astype(np.int64)), k
    pl.close()


@pytest.mark.parametrize("depth", [2, 5, 6, 21])  # 1, 2, 3 and 8 digit passes
@pytest.mark.parametrize("n", SIZES)
def test_adaptive_tree(n, depth):
    x, _ = inputs.plummer(n, 3)
    x[n // 2:] = x[:n - n // 2]  # every key twice: ties in the original order
    say("plan sizes n", n, "depth", depth)
    _same_tree(x, leaf_size=40, max_depth=depth)


@pytest.mark.parametrize("n,depth", [(3000, 4), (20000, 2), (9000, 5)])  # 4681, 73 and 37449 boxes
def test_uniform_tree(n, depth):
    _same_tree(inputs.uniform(n, 4)[0], uniform_depth=depth, root=[0, 0, 0, 1])


@pytest.mark.parametrize("n", [4194304, 4194305])
def test_scan_over_all_particles(n):
    """The two sides of the largest scan: the boxes tile the sorted particles."""
    from paper_2508_02626_amd import fmm
    x, _ = inputs.uniform(n, 5)
    pl = fmm.Plan(to_dev(x), 1, leaf_size=64)
    g = pl.export_tree()
    assert np.array_equal(np.sort(g["perm"]), np.arange(n))
    leaf = g["nchild"] == 0
    o = np.argsort(g["first"][leaf])
    first, count = g["first"][leaf][o].astype(np.int64), g["count"][leaf][o].astype(np.int64)
    assert first[0] == 0 and np.array_equal(first[1:], np.cumsum(count)[:-1]) and first[-1] + count[-1] == n
    assert count.max() <= 64
    pl.close()
