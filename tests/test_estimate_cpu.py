"""Admission estimates: the slices of partial sums of small trees' M2L parts are
charged only where a plan can hold them (host only)."""
import ctypes

import pytest

from paper_2508_02626_amd import fmm


def _est(n, order, leaf_size=64, **opts):
    o = fmm.Options()
    fmm.lib().fmm_default_options(ctypes.byref(o))
    for k, v in opts.items():
        setattr(o, k, v)
    b = ctypes.c_size_t()
    assert fmm.lib().fmm_plan_estimate(n, order, leaf_size, ctypes.byref(o), ctypes.byref(b)) == 0
    return b.value


SOFT, ROTATION = dict(kernel=1, softening=1e-3), dict(m2l_method=1)

# (points, order, options, bytes of particles, lists and expansions alone)
WITHOUT = [
    (1000, 8, SOFT, 68621759), (10000, 8, SOFT, 87267682), (10000, 5, SOFT, 30495128),
    (1000, 8, ROTATION, 1901808), (10000, 8, ROTATION, 18952654), (10000, 5, ROTATION, 10481522),
    (1000, 8, dict(uniform_depth=3, kernel=1), 11433350), (1000, 8, dict(uniform_depth=2, m2l_method=1), 635710),
    (1000, 8, dict(uniform_depth=5), 272359230), (10000, 5, dict(uniform_depth=5), 144479670),
    (20000, 8, {}, 37898039), (100000, 12, {}, 429717030), (1000000, 8, {}, 1894545731), (4000000, 14, {}, 23568331202),
]


@pytest.mark.parametrize("n,p,opts,want", WITHOUT)
def test_plans_without_slices_are_not_charged(n, p, opts, want):
    """Softened and rotation plans have one part per tile, large trees the fixed
    number; a rounding of the double sum apart."""
    assert abs(_est(n, p, **opts) - want) <= 1


@pytest.mark.parametrize("n,p,alone", [(10000, 4, 8708494), (10000, 8, 18952654), (10000, 12, 42987030),
                                       (10000, 16, 78644586), (8000, 8, 15163577)])
def test_middling_adaptive_trees(n, p, alone):
    """Their slices fit into what the bound on the boxes leaves, or nearly."""
    assert alone <= _est(n, p) <= 1.15 * alone


def test_small_trees_are_charged_their_slices():
    # 585 boxes, 16 parts: 15 slices of 96 doubles, exactly
    assert _est(1000, 8, uniform_depth=3) == 4357950 + 15 * 585 * 96 * 8
    # 137 boxes of 1000 Plummer points: 0.86 MB and 1.58 MB of slices
    assert 2.44e6 <= _est(1000, 8) <= 3e6
