"""The sorts, the float64 row kernel and the spread's 4^3 tiles on small inputs, which
the grids that are multiples of 8 give to the direct path: here the grid is not one.
One cell, the fewest rows (5 per axis), more candidates than one chunk of start
marks holds, cells capped by the number of points, single bins; velocity and
streamfunction, closed and infinite filaments, cubic and quintic.

The short-range velocity against the oracle's sums over the same points, float64 in
another order: 1e-12 as for large inputs, of the sum or, where the terms cancel (the
straight lines), of one term at the distance r_c.  Velocity and streamfunction whole against
the oracle's direct Fourier sums over the same modes: with a kernel of w = 16 the
NUFFT's error is 1e-14 by its decay law, so 1e-11 leaves the rounding of the
deconvolved modes."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2406_07366_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2406_07366_amd import binding
    return binding


CASES = [
    # name, filaments, r_c / L, grid, spline order, psi too
    ("one cell", lambda: W.ellipses(3, 37, seed=3), 0.49, 36, 4, True),
    ("five rows per axis", lambda: W.ellipses(40, 21, seed=40), 0.3999, 36, 4, False),
    ("five rows, psi", lambda: W.ellipses(8, 21, seed=41), 0.3999, 36, 6, True),
    ("many candidates", lambda: W.ellipses(100, 40, seed=120), 0.33, 68, 4, False),
    ("cells capped", lambda: W.ellipses(1, 200, seed=1), 0.12, 36, 4, True),
    ("many rows", lambda: W.ellipses(10, 30, seed=7), 0.2, 44, 4, True),
    ("infinite lines", lambda: W.six_lines(40), 0.3, 36, 4, True),
    ("infinite helices", lambda: W.helices(48), 0.49, 36, 6, True),
    ("three nodes", lambda: W.ellipses(1, 3, seed=9), 0.49, 36, 4, True),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_general_path_on_small_inputs(B, case):
    name, make, rc_over_L, grid, order, whole = case
    fs = make()
    rc = rc_over_L * fs.L
    alpha = 3.5 / rc
    print(f"\n[case] {name}: N {fs.n_nodes} grid {grid} order {order}", flush=True)
    plan = B.Plan(B.make_params(L=fs.L, a=fs.a, tol=1e-6, grid_n=grid, w=16, alpha=alpha, rcut=rc,
                                spline_order=order))
    if fs.periods is not None:
        plan.set_periods(fs.periods)
    xyz, g = B.load_workload(fs)
    plan.set_profiling(True)
    plan.set_filaments(fs.offsets, xyz, g)
    plan.velocity()
    assert plan.stage_times()["binning"][1] == 1     # the sorts ran
    plan.set_profiling(False)
    plan.set_filaments(fs.offsets, xyz, g)
    t = {k: v.cpu().numpy() for k, v in plan.velocity_terms().items()}
    v = plan.velocity().cpu().numpy()
    E, psi = plan.energy()
    K = plan.params().K
    plan.status()
    plan.close()
    o = O.Oracle(fs, order=order)
    tg = np.arange(0, fs.n_nodes, max(1, fs.n_nodes // 400))
    ref, _ = o.shortrange(alpha, rc, targets=tg, psi=False)
    one = np.abs(fs.gamma).max() / (4 * np.pi * rc)
    scale = max(np.sqrt((ref ** 2).mean()), one)
    err = np.sqrt(((t["short"][tg] - ref) ** 2).mean()) / scale
    terms = np.linalg.norm(v - (t["local"] + t["short"] + t["long"] - t["self"])) / np.linalg.norm(v)
    print(f"  short {err:.2e}, sum of terms {terms:.2e}")
    assert err < 1e-12 and terms < 1e-12
    if not whole:
        return
    parts = [o.local(), o.shortrange(alpha, rc, psi=True), o.longrange(alpha, K, psi=True),
             o.selfcorr(alpha)]
    for what, got, i in (("v", v, 0), ("psi", psi.cpu().numpy(), 1)):
        ref = parts[0][i] + parts[1][i] + parts[2][i] - parts[3][i]
        err = np.sqrt(((got - ref) ** 2).mean()) / max(np.sqrt((ref ** 2).mean()), one)
        print(f"  {what} {err:.2e}")
        assert err < 1e-11, what
