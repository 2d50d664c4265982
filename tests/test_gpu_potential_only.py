"""Evaluations without a field array run the potential-only P2P, M2P and L2P
kernels; their potentials are the bits of an evaluation with the field."""
import numpy as np
import pytest

from gpu_util import to_dev
from paper_2508_02626_amd import inputs

pytestmark = pytest.mark.gpu

CASES = [
    ("plummer_p7", lambda: inputs.plummer(6000, 2), 7, dict(leaf_size=32)),          # W and X lists
    ("plummer_p13", lambda: inputs.plummer(4000, 3), 13, dict(leaf_size=32)),
    ("clusters_p4_mixed", lambda: inputs.clusters(4000, 4), 4, dict(leaf_size=70, precision="mixed")),
    ("uniform_p8_depth2", lambda: inputs.uniform(5000, 5), 8, dict(uniform_depth=2, root=[0, 0, 0, 1])),
    ("near_field_only", lambda: inputs.uniform(50, 6), 3, dict(leaf_size=64)),
    ("softened_plummer_p6", lambda: inputs.plummer(6000, 7), 6, dict(leaf_size=32, kernel="softened", softening=1e-3)),
    ("softened_p10", lambda: inputs.plummer(2000, 8), 10, dict(leaf_size=16, kernel="softened", softening=1e-2)),
]


@pytest.mark.parametrize("name,gen,p,kw", CASES, ids=[c[0] for c in CASES])
def test_potential_only_equals_potential_with_field(name, gen, p, kw):
    from paper_2508_02626_amd import fmm
    x, q = gen()
    pl = fmm.Plan(to_dev(x), p, **kw)
    phi, fld = pl.evaluate(to_dev(q))
    alone, none = pl.evaluate(to_dev(q), want_field=False)
    assert none is None
    assert np.array_equal(phi.cpu().numpy(), alone.cpu().numpy())
    pl.close()


def test_batch_without_field_equals_single():
    from paper_2508_02626_amd import fmm
    probs = [(gen(), p, kw) for _, gen, p, kw in CASES if kw.get("kernel") is None]
    plans = [fmm.Plan(to_dev(x), p, **kw) for (x, _), p, kw in probs]
    qs = [to_dev(q) for (_, q), _, _ in probs]
    singles = [pl.evaluate(q)[0].cpu().numpy() for pl, q in zip(plans, qs)]
    for (a, none), b in zip(fmm.evaluate_batch(plans, qs, want_field=False), singles):
        assert none is None
        assert np.array_equal(a.cpu().numpy(), b)
