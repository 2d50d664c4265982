"""M2M and L2L at levels of many parents, where a wavefront takes all row tiles of
16 parents (M2M above 64 groups of 16, L2L from 2048) or several of them (L2L
from 2048 / row tiles, the next tile's operands carried over), and at levels of
fewer, where every row tile has its own: exported expansions of sampled parents
and children against the oracle's m2m and l2l, degree by degree.

Only the particles with x < 1/4 carry charge.  Boxes beyond x = 3/4 then receive
nothing but their parent's local expansion (their V and X lists hold zero
charges), so that one level's L2L stands alone."""
import numpy as np
import pytest

import oracle
from gpu_util import say, to_dev
from paper_2508_02626_amd import fmm, inputs

pytestmark = pytest.mark.gpu


def _centre(g, b):
    m, l = int(g["morton"][b]), int(g["level"][b])
    c = [sum(((m >> (3 * i + k)) & 1) << i for i in range(l)) for k in range(3)]
    return (np.array(c) + 0.5) / 2 ** l


def _axes():
    """Which of (x, y, z) each Morton bit of the trees below stands for."""
    x = np.array([[0.9, 0.1, 0.1], [0.1, 0.9, 0.1], [0.1, 0.1, 0.9]])
    pl = fmm.Plan(to_dev(x), 0, uniform_depth=1, root=[0, 0, 0, 1])
    g = pl.export_tree()
    pl.close()
    ax = []
    for i in range(3):
        b = next(b for b in range(1, 9) if i in g["perm"][g["first"][b]:g["first"][b] + g["count"][b]])
        ax.append([1, 2, 4].index(int(g["morton"][b])))
    return ax


def _check(p, n, levels, per, **kw):
    x, _ = inputs.uniform(n, 500 + p)
    q = np.where(x[:, 0] < 0.25, np.random.default_rng(p).uniform(0.5, 1.5, n), 0.0)
    pl = fmm.Plan(to_dev(x), p, root=[0, 0, 0, 1], **kw)
    pl.evaluate(to_dev(q))
    g = pl.export_tree()
    M, L = pl.export_expansions()
    pl.close()
    ax, deg = _axes(), oracle.exponents(p).sum(axis=1)
    cen = lambda b: _centre(g, b)[ax]
    rng = np.random.default_rng(p)
    worst = [0.0, 0.0]
    for lev in levels:
        parents = np.flatnonzero((g["level"] == lev) & (g["nchild"] > 0))
        px = np.array([cen(b)[0] for b in parents])
        kids = lambda b: range(g["child_begin"][b], g["child_begin"][b] + g["nchild"][b])
        for which, pick in (0, parents[px < 0.25]), (1, parents[px > 0.75]):
            pick = [pick[-1]] + list(rng.choice(pick[:-1], per - 1, replace=False))  # (the level's last among them)
            got, ref = [], []
            for b in pick:
                if which == 0:
                    got.append(M[b])
                    ref.append(sum(oracle.m2m(p, cen(c), cen(b), M[c]) for c in kids(b)))
                else:
                    got += [L[c] for c in kids(b)]
                    ref += [oracle.l2l(p, cen(b), cen(c), L[b]) for c in kids(b)]
            got, ref = np.array(got), np.array(ref)
            for d in range(p + 1):
                s = deg == d
                e = np.abs(got[:, s] - ref[:, s]).max() / np.abs(ref[:, s]).max()
                worst[which] = max(worst[which], e)
                assert e <= 1e-12, ("M2M" if which == 0 else "L2L", "level", lev, "degree", d, e)
        say("  p %d level %d, %d parents: M2M %.2e L2L %.2e" % (p, lev, len(parents), *worst))


@pytest.mark.parametrize("p", [5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16])
def test_thousands_of_parents(p):
    """512 and 4096 parents: M2M on both sides of its line, L2L by row tiles and
    by eight wavefronts for up to 23 tiles."""
    _check(p, 60000, [3, 4], 3 if p <= 12 else 1, uniform_depth=5)


@pytest.mark.parametrize("p", [6, 9])
def test_tens_of_thousands_of_parents(p):
    """32,768 parents: one wavefront takes every row tile of the L2L."""
    _check(p, 200000, [5], 3, uniform_depth=6)


@pytest.mark.parametrize("p", [10, 16])
def test_missing_children(p):
    """An adaptive tree: parents with fewer than eight children, a last group of
    fewer than 16 parents."""
    _check(p, 40000, [4], 3 if p <= 12 else 2, leaf_size=8)
