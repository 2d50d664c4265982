"""P2P at the edges of its passes and chunks: leaves of 1, 2, 63 to 65 and more
targets, source streams around whole chunks (64 and 128), U lists of more than
64 boxes, FP64 and FP32, with and without the field, against the direct sum."""
import numpy as np
import pytest

from gpu_util import rel_l2, say, to_dev
from paper_2508_02626_amd import fmm, inputs

pytestmark = pytest.mark.gpu


def _direct(x, q):
    d = x[:, None, :] - x[None, :, :]
    r2 = (d * d).sum(-1)
    inv = np.where(r2 > 0, 1.0 / np.sqrt(np.where(r2 > 0, r2, 1.0)), 0.0)
    return inv @ q, (d * (q[None, :] * inv ** 3)[:, :, None]).sum(1)


def _check(x, q, precision, **kw):
    pl = fmm.Plan(to_dev(x), 1, precision=precision, **kw)
    phi, fld = (a.cpu().numpy() for a in pl.evaluate(to_dev(q)))
    only = pl.evaluate(to_dev(q), want_field=False)[0].cpu().numpy()
    pl.close()
    rphi, rfld = _direct(x, q)
    e, f = rel_l2(phi, rphi), rel_l2(fld, rfld)
    say("  n %d %s %s: phi %.2e field %.2e" % (len(q), precision, kw, e, f))
    b = (1e-13, 1e-13) if precision == "fp64" else (3e-7, 1e-6)
    assert e <= b[0] and f <= b[1] and np.array_equal(phi, only)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [1, 2, 3, 31, 33, 63, 64, 65, 127, 128, 129, 191, 193, 256, 257, 700])
def test_one_leaf(n, precision):
    x, _ = inputs.uniform(n, 40)
    q = np.linspace(0.5, 1.5, n)  # (no cancellation)
    _check(x, q, precision, uniform_depth=0, root=[0, 0, 0, 1])


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("per", [1, 2, 9, 16, 17])
def test_two_levels_of_near_boxes(per, precision):
    """Eight leaves, each the neighbour of all: streams of 8 * per sources."""
    rng = np.random.default_rng(41)
    c = np.array([[i, j, k] for i in (0, 1) for j in (0, 1) for k in (0, 1)]) / 2.0
    x = (c[:, None, :] + 0.5 * rng.uniform(0, 1, (8, per, 3))).reshape(-1, 3)
    _check(x, np.linspace(0.5, 1.5, len(x)), precision, uniform_depth=1, root=[0, 0, 0, 1])


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_long_u_list(precision):
    """A large empty-ish leaf next to a finely divided face has more than 64 U boxes:
    its near field against the same plan's order-independent part."""
    rng = np.random.default_rng(42)
    face = rng.uniform(0, 1, (3000, 3)) * [0.02, 1, 1] + [0.5, 0, 0]
    lone = np.array([[0.25, 0.3, 0.3], [0.26, 0.7, 0.7]])
    x = np.concatenate([lone, face])
    q = np.linspace(0.5, 1.5, len(x))
    pl = fmm.Plan(to_dev(x), 12, leaf_size=4, precision=precision)
    u = np.diff(pl.export_tree()["U_off"].astype(np.int64))
    phi = pl.evaluate(to_dev(q), want_field=False)[0].cpu().numpy()
    pl.close()
    say("  U lists up to %d" % u.max())
    assert u.max() > 64 and rel_l2(phi, _direct(x, q)[0]) <= 1e-5
