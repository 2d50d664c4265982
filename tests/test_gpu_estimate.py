"""Plans of small and middling trees, whose M2L parts keep slices of partial sums,
hold no more device memory than their admission estimate; uniform trees of no or
one level of targets too."""
import pytest

from gpu_util import say, to_dev
from paper_2508_02626_amd import fmm, inputs
from test_gpu_boundary import TorchAllocator

pytestmark = pytest.mark.gpu

SETS = {"uniform": inputs.uniform, "plummer": inputs.plummer, "clusters": inputs.clusters}


@pytest.mark.parametrize("p", [0, 4, 6, 8, 12, 16])
@pytest.mark.parametrize("n,leaf", [(1000, 64), (1000, 128), (3000, 8), (10000, 64), (10000, 128), (17389, 64)])
def test_adaptive_footprint_below_estimate(n, leaf, p):
    for name, gen in SETS.items():
        al = TorchAllocator()  # (the library's own cache counts whole chunks)
        pl = fmm.Plan(to_dev(gen(n, 3)[0]), p, leaf_size=leaf, allocator=al.c)
        f, e = pl.footprint(), fmm.estimate(n, p, leaf)
        pl.close()
        say("  %s n %d leaf %d p %d: %d of %d bytes" % (name, n, leaf, p, f, e))
        assert f <= e


@pytest.mark.parametrize("p", [0, 4, 6, 8, 12, 16])
@pytest.mark.parametrize("depth", [0, 1, 2, 3, 4])
def test_uniform_footprint_below_estimate(depth, p):
    n = 2000
    al = TorchAllocator()
    pl = fmm.Plan(to_dev(inputs.uniform(n, 3)[0]), p, uniform_depth=depth, root=[0, 0, 0, 1], allocator=al.c)
    f, e = pl.footprint(), fmm.estimate(n, p, uniform_depth=depth)
    pl.close()
    say("  depth %d p %d: %d of %d bytes" % (depth, p, f, e))
    assert f <= e
