"""P2P of particles so close that 1/r^2 overflows although q/r^2 does not (r^2
subnormal), zero charges among them, against the direct sum in extended
precision."""
import numpy as np
import pytest

from gpu_util import say, to_dev
from paper_2508_02626_amd import fmm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [dict(), dict(kernel="softened", softening=0.0)], ids=["coulomb", "softened_eps0"])
@pytest.mark.parametrize("copies", [1, 40])
def test_tiny_separations(copies, kw):
    x = np.array([[0, 0, 0], [1e-155, 0, 0], [0, 3e-155, 0], [0.5, 0.25, 0.75]])
    q = np.array([0.0, 0.0, 1e-300, 1.0])
    far = np.random.default_rng(5).uniform(0.5, 1, (copies - 1, 3))  # (several lane groups and one)
    x, q = np.concatenate([x, far]), np.concatenate([q, np.ones(len(far))])
    X, Q = x.astype(np.longdouble), q.astype(np.longdouble)
    d = X[:, None, :] - X[None, :, :]
    r2 = (d * d).sum(-1)
    inv = np.where(r2 > 0, 1 / np.sqrt(np.where(r2 > 0, r2, 1)), 0)
    phi, fld = inv @ Q, (d * (Q[None, :] * inv ** 3)[:, :, None]).sum(1)
    pl = fmm.Plan(to_dev(x), 2, uniform_depth=0, root=[0, 0, 0, 1], **kw)
    g, e = (a.cpu().numpy() for a in pl.evaluate(to_dev(q)))
    pl.close()
    # r^2 near 1e-310 has 14 digits; its powers -1/2 and -3/2 in the terms
    ep = float((np.abs(g - phi) / np.abs(phi)).max())
    ef = float((np.abs(e - fld).max(1) / np.abs(fld).max(1)).max())
    say("  copies %d %s: phi %.2e field %.2e" % (copies, kw, ep, ef))
    assert np.isfinite(e).all() and ep <= 1e-12 and ef <= 1e-12
