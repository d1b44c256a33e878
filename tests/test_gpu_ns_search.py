"""The near-singular pair search where its work is split: cells of more than
64 targets (cut between wavefronts), cells smaller than that, windows with and
without the wrap, fewer than 3 and fewer than 5 cells per axis, long segments
(the second grid), several targets per wavefront (8 and 16), targets and
midpoints beyond the packed period range.  The number of flagged pairs is a
brute-force count on the CPU in float64, exactly, and on the smaller sets the
correction itself is the oracle's, to the 1e-10 that its quadrature carries."""
import math

import numpy as np
import pytest

from oracle import oracle as O
from paper_2406_07366_amd import workloads as W
from tests.test_gpu_ns import make_plan, rel_l2

pytestmark = pytest.mark.gpu
L = 2 * math.pi


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2406_07366_amd import binding
    return binding


def rings(n, nodes, centre, spread, radius, seed, radius2=None):
    """Rings of given radius with centres in a cube of edge `spread`; every
    tenth with radius2, if given."""
    rng = np.random.default_rng(seed)
    t = 2 * np.pi * np.arange(nodes) / nodes
    fs = W.ellipses(nfil=n, n_per=nodes, seed=seed)
    out = []
    for k in range(n):
        q, _ = np.linalg.qr(rng.normal(size=(3, 3)))
        r = radius2 if radius2 and k % 10 == 0 else radius
        out.append(centre + spread * (rng.uniform(size=3) - 0.5) +
                   r * (np.cos(t)[:, None] * q[0] + np.sin(t)[:, None] * q[1]))
    fs.xyz = np.concatenate(out)
    fs.grid_n, fs.tol, fs.name = 64, 1e-6, f"{n} rings of {nodes}"
    return fs


def count(fs, ell, eta):
    """Non-adjacent segments whose chord passes within eta ell of a node."""
    from scipy.spatial import cKDTree
    x, off = np.asarray(fs.xyz), fs.offsets
    n = len(x)
    nxt = np.arange(1, n + 1)
    nxt[off[1:] - 1] = off[:-1]
    prv = np.empty(n, int)
    prv[nxt] = np.arange(n)
    e = x[nxt] - x
    mid, hc = x + 0.5 * e, 0.5 * np.sqrt((e ** 2).sum(1))
    reach = eta * ell + hc
    wrap = lambda v: np.minimum(np.mod(v, L), np.nextafter(L, 0))
    tree, total = cKDTree(wrap(x), boxsize=L), 0
    for j0 in range(0, n, 20000):
        js = np.arange(j0, min(n, j0 + 20000))
        cand = tree.query_ball_point(wrap(mid[js]), reach[js] * (1 + 1e-9))
        j = np.repeat(js, [len(c) for c in cand])
        o = np.concatenate([np.asarray(c, int) for c in cand])
        r = x[o] - mid[j]
        r -= L * np.rint(r / L)
        u = np.clip((r * e[j]).sum(1) / (e[j] ** 2).sum(1), -0.5, 0.5)
        d = np.sqrt(((r - u[:, None] * e[j]) ** 2).sum(1))
        total += int(((d < eta * ell[j]) & (o != j) & (prv[o] != j)).sum())
    return total


CASES = {
    # name: (filaments, eta, compare the correction)
    "three cells": (lambda: rings(6, 16, np.full(3, 6.2), 4.0, 2.9, 1), 1.0, True),
    "one cell": (lambda: rings(4, 8, np.zeros(3), 3.0, 2.8, 2), 2.0, True),
    "four cells": (lambda: rings(8, 16, np.full(3, 1.0), 6.0, 2.3, 3), 1.0, True),
    "dense": (lambda: rings(700, 16, np.array([6.25, 0.05, 3.0]), 0.6, 0.3, 4), 0.25, False),
    "dense with long segments": (lambda: rings(500, 16, np.zeros(3), 1.0, 0.25, 5, 1.2), 0.3, False),
    "sparse": (lambda: rings(40, 12, np.full(3, 3.0), 6.2, 0.05, 6), 1.0, True),
    "16 targets a wavefront": (lambda: W.tangle(nfil=700, n_per=100, seed=7), 1.0, False),
    "beyond the period range": (lambda: rings(60, 16, np.array([520 * L, -515 * L, 0.3]), 1.5, 0.3, 8),
                                0.6, True),
}


@pytest.mark.parametrize("name", CASES)
def test_search_flags_the_pairs_of_a_full_count(B, name):
    make, eta, values = CASES[name]
    fs = make()
    plan = make_plan(B, fs, ns_mode=B.BS_NS_ADAPTIVE, ns_eta=eta)
    ell = plan.geometry()["ell"].cpu().numpy()
    want = count(fs, ell, eta)
    got = plan.ns_counts()[0]
    print(f"  {name}: {got} pairs, counted {want}")
    plan.status()
    assert want > 0 and got == want
    if values:
        dv = plan.velocity_terms()["ns"].cpu().numpy()
        ref, cnt = O.Oracle(fs).ns_correction(eta=eta)
        assert int(cnt.sum()) == want and rel_l2(dv, ref) < 1e-10


def close_rings(gap, n):
    """Two coaxial rings of n nodes a gap apart, the second turned by a third
    of a segment (targets over the inside of segments), and a third ring far
    from both."""
    t = 2 * np.pi * np.arange(n) / n
    fs = W.ellipses(nfil=3, n_per=n, seed=9)
    ring = lambda z, s: np.stack([1.0 + 0.5 * np.cos(t + s), 2.0 + 0.5 * np.sin(t + s), z + 0 * t], 1)
    fs.xyz = np.concatenate([ring(3.0, 0.0), ring(3.0 + gap, 2 * np.pi / (3 * n)), ring(5.5, 0.1)])
    fs.grid_n, fs.tol, fs.name = 64, 1e-6, f"rings of {n}, gap {gap}"
    return fs


@pytest.mark.parametrize("order", [4, 6])
@pytest.mark.parametrize("gap,n", [(0.2, 6), (1e-2, 7), (1e-5, 11)])
def test_integrals_with_few_and_many_panels(B, order, gap, n):
    """From 2 panels a pair to over 20, pair counts that leave lanes idle: the
    correction is the oracle's, to the 1e-10 of the panels' quadrature, or to
    the float64 rounding of the distance in a pair's 1 / distance."""
    fs = close_rings(gap, n)
    plan = make_plan(B, fs, ns_mode=B.BS_NS_ADAPTIVE, spline_order=order)
    dv = plan.velocity_terms()["ns"].cpu().numpy()
    ref, cnt = O.Oracle(fs, order=order).ns_correction(eta=1.0)
    assert plan.ns_counts()[0] == int(cnt.sum()) > 0
    err = rel_l2(dv, ref)
    print(f"  order {order} gap {gap}: {cnt.sum()} pairs, rel_l2 {err:.2e}")
    assert err < max(1e-10, 1e-14 / gap)
