"""M2P runs four wavefronts per leaf: a batch of more leaves than one launch may
have threads for (2^32 / 256) takes several launches."""
import numpy as np
import pytest

from gpu_util import say, to_dev
from paper_2508_02626_amd import fmm, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("want_field", [True, False])
def test_batch_of_more_leaves_than_one_launch(want_field):
    n, plans = 65700, 256
    x, q = inputs.uniform(n, 77)
    xd, qd = to_dev(x), to_dev(q)
    pl = [fmm.Plan(xd, 1, leaf_size=1) for _ in range(plans)]
    g = pl[0].export_tree()
    leaves, w = int((g["nchild"] == 0).sum()), np.diff(g["W_off"].astype(np.int64))
    say("  %d leaves in all, %d of a plan's with a W list" % (leaves * plans, (w > 0).sum()))
    assert leaves * plans * 256 >= 2 ** 32 and (w > 0).sum() > leaves // 4
    one = pl[0].evaluate(qd, want_field=want_field)
    for got in fmm.evaluate_batch(pl, [qd] * plans, want_field=want_field):
        for a, b in zip(got, one):
            assert (a is None and b is None) or bool((a == b).all())
    for p in pl:
        p.close()
