"""M2P of plans with 8192 and more W-list leaves, which take one wavefront each
instead of four: sampled targets put together from the exported expansions by the
oracle's single operators (near field, the W boxes' multipoles, the leaf's local
expansion).  A batch of such plans with more leaves than a launch of four
wavefronts each may have threads for (2^32 / 256) equals its plans alone."""
import numpy as np
import pytest

import oracle
from gpu_util import say, to_dev
from paper_2508_02626_amd import fmm, inputs

pytestmark = pytest.mark.gpu


def _centres(g, root, axes):
    lev, m = g["level"].astype(np.int64), g["morton"].astype(np.uint64)
    c = np.zeros((len(lev), 3))
    for k in range(3):
        v = np.zeros(len(lev), np.int64)
        for b in range(21):
            v |= ((m >> np.uint64(3 * b + axes[k])) & np.uint64(1)).astype(np.int64) << b
        c[:, k] = (v + 0.5) / 2.0 ** lev
    return root[:3] + root[3] * c


# (points, leaf size, order): passes of up to 16, 32 and 64 targets and leaves of more
CASES = [(20000, 1, p) for p in (1, 5, 6, 9, 10, 11, 12, 14, 16)] + [(300000, 16, 8), (1000000, 32, 6),
                                                                   (1000000, 32, 10), (1600000, 70, 4)]


@pytest.mark.parametrize("n,leaf,p", CASES)
def test_one_wave_targets_from_single_operators(n, leaf, p):
    x, q = inputs.plummer(n, 3)
    root = np.array([-1.0, -1.0, -1.0, 2.0])
    pl = fmm.Plan(to_dev(x), p, leaf_size=leaf, root=list(root))
    qd = to_dev(q)
    phi, fld = (a.cpu().numpy() for a in pl.evaluate(qd))
    only = pl.evaluate(qd, want_field=False)[0].cpu().numpy()
    g = pl.export_tree()
    M, L = pl.export_expansions()
    pl.close()
    w = np.diff(g["W_off"].astype(np.int64))
    boxes = np.flatnonzero(w > 0)
    assert len(boxes) >= 8192
    # a bit of the code per axis: x is the highest of three
    cen = _centres(g, root, (2, 1, 0))
    inside = np.abs(x[g["perm"][g["first"][boxes]]] - cen[boxes]) / (root[3] / 2.0 ** g["level"][boxes])[:, None]
    assert inside.max() <= 0.5 + 1e-9
    part = lambda b: g["perm"][g["first"][b]:g["first"][b] + g["count"][b]]
    cnt = g["count"][boxes]
    pick = {int(boxes[0]), int(boxes[-1]), int(boxes[np.argmax(w[boxes])]), int(boxes[np.argmax(cnt)]), int(boxes[np.argmin(cnt)])}
    pick |= set(np.random.default_rng(p).choice(boxes, 8, replace=False).tolist())
    got, ref, gf, rf, po = [], [], [], [], []
    for b in sorted(pick):
        t = part(b)
        u = np.concatenate([part(s) for s in g["U_src"][g["U_off"][b]:g["U_off"][b + 1]]])
        d = x[t][:, None, :] - x[u][None, :, :]
        r2 = (d * d).sum(-1)
        inv = np.where(r2 > 0, 1 / np.sqrt(np.where(r2 > 0, r2, 1)), 0)
        a, f = inv @ q[u], (d * (q[u][None, :] * inv ** 3)[:, :, None]).sum(1)
        for s in g["W_src"][g["W_off"][b]:g["W_off"][b + 1]]:
            da, df = oracle.m2p(p, cen[s], M[s], x[t])
            a, f = a + da, f + df
        da, df = oracle.l2p(p, cen[b], L[b], x[t])
        got.append(phi[t]); ref.append(a + da); gf.append(fld[t]); rf.append(f + df); po.append(only[t])
    got, ref, gf, rf, po = (np.concatenate(v) for v in (got, ref, gf, rf, po))
    e = np.abs(got - ref).max() / np.abs(ref).max()
    ef = np.abs(gf - rf).max() / np.abs(rf).max()
    say("  n %d leaf %d p %d: %d leaves with W lists up to %d, %d targets: phi %.2e field %.2e"
        % (n, leaf, p, len(boxes), w.max(), len(ref), e, ef))
    assert e <= 1e-12 and ef <= 1e-12 and np.abs(po - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("want_field", [True, False])
def test_batch_of_more_leaves_than_one_launch_of_four(want_field):
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
