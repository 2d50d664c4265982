"""P2P over U lists of several batches of 64 boxes, whose partial chunks the next
batch completes: one to 130 targets (every number of lane groups, several passes),
potential and field of the leaf with the long list alone, against the oracle's
FMM of the same order.  And what the kernel's flush of the last chunk rests on:
no list's last batch is empty."""
import numpy as np
import pytest

from gpu_util import oracle_tree, rel_l2, say, to_dev
from paper_2508_02626_amd import fmm, inputs

pytestmark = pytest.mark.gpu


def _face(targets, leaf, seed):
    """`targets` points alone in one octant of the unit cube, beside a sheet whose
    256 (1/16)^2 columns hold one to four points more than a leaf."""
    rng = np.random.default_rng(seed)
    lone = rng.uniform(0.1, 0.4, (targets, 3))
    cols = [(i, j) for i in range(16) for j in range(16)]
    m = leaf + rng.integers(1, 5, len(cols))
    sheet = [np.stack([0.5 + 0.02 * rng.uniform(0, 1, k), (i + rng.uniform(0, 1, k)) / 16,
                       (j + rng.uniform(0, 1, k)) / 16], 1) for (i, j), k in zip(cols, m)]
    x = np.concatenate([lone] + sheet)
    return x, rng.uniform(0.5, 1.5, len(x))


@pytest.mark.parametrize("targets", [1, 2, 3, 17, 40, 64, 65, 130])
def test_long_list_targets_match_oracle(targets):
    leaf, p = max(targets, 8), 2
    kw = dict(leaf_size=leaf, root=[0, 0, 0, 1])
    x, q = _face(targets, leaf, 100 + targets)
    pl = fmm.Plan(to_dev(x), p, **kw)
    g = pl.export_tree()
    box = next(b for b in range(len(g["level"])) if g["nchild"][b] == 0 and 0 in g["perm"][g["first"][b]:g["first"][b] + g["count"][b]])
    u = int(g["U_off"][box + 1] - g["U_off"][box])
    assert g["count"][box] == targets and u > 192
    phi, fld = (a.cpu().numpy()[:targets] for a in pl.evaluate(to_dev(q)))
    only = pl.evaluate(to_dev(q), want_field=False)[0].cpu().numpy()[:targets]
    pl.close()
    ophi, ofld = (a[:targets] for a in oracle_tree(x, **kw).fmm(p, q))
    pl = fmm.Plan(to_dev(x), p, precision="mixed", **kw)
    mphi, mfld = (a.cpu().numpy()[:targets] for a in pl.evaluate(to_dev(q)))
    pl.close()
    e = rel_l2(phi, ophi), rel_l2(fld, ofld), rel_l2(mphi, ophi), rel_l2(mfld, ofld)
    say("  %d targets, %d boxes: phi %.2e field %.2e mixed %.2e %.2e" % ((targets, u) + e))
    assert e[0] <= 1e-12 and e[1] <= 1e-12 and e[2] <= 3e-7 and e[3] <= 1e-6
    assert np.array_equal(phi, only)


@pytest.mark.parametrize("name,gen,kw", [
    ("plummer", lambda: inputs.plummer(20000, 3), dict(leaf_size=1)),
    ("clusters", lambda: inputs.clusters(20000, 3), dict(leaf_size=3)),
    ("uniform_sparse", lambda: inputs.uniform(200, 3), dict(uniform_depth=5, root=[0, 0, 0, 1])),
])
def test_no_list_ends_in_an_empty_batch(name, gen, kw):
    pl = fmm.Plan(to_dev(gen()[0]), 1, **kw)
    g = pl.export_tree()
    pl.close()
    u = np.diff(g["U_off"].astype(np.int64))
    say("  %s: U lists up to %d, %d boxes empty" % (name, u.max(), (g["count"] == 0).sum()))
    assert (g["count"] > 0).all() or u.max() <= 27
