"""The float64 short-range streamfunction to rounding.  With a splitting parameter so
small that the long-range part vanishes (alpha L = 0.5: the first mode's Gaussian is
below 1e-17) the streamfunction is local + short - self, formed here in 80 bits over
the plan's own points.  Every term is rounded a few times, so the errors of a
node's sum stay below 4 eps of the terms' root sum of squares, plus 4 eps of the
result (its own last additions).  The fitted polynomial with an exponential, good to
3e-15 of every term alike, does not pass."""
import math

import numpy as np
import pytest

from paper_2406_07366_amd import workloads as W

pytestmark = pytest.mark.gpu
LD = np.longdouble
PI = LD("3.14159265358979323846264338327950288")


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2406_07366_amd import binding
    return binding


def erf_small(x):
    """erf(x) for x < 1 by its Taylor series in 80 bits."""
    s, t = x.copy(), x.copy()
    for n in range(1, 40):
        t = -t * x * x / n
        s = s + t / (2 * n + 1)
    return 2 / np.sqrt(PI) * s


def reference(fs, geo, alpha, rc, Q):
    """psi at every node."""
    qp, qc = geo["qpos"].astype(LD), geo["qcharge"].astype(LD)
    sd, ell = geo["sdot"].astype(LD), geo["ell"].astype(LD)
    N, L, a = fs.n_nodes, LD(fs.L), LD(alpha)
    seg = np.arange(len(qp)) // Q
    prev = np.arange(N) - 1
    prev[fs.offsets[:-1]] = fs.offsets[1:] - 1
    gam = np.repeat(fs.gamma, np.diff(fs.offsets)).astype(LD)
    psi = np.zeros((N, 3), LD)
    for i in range(N):
        sn = np.sqrt((sd[i] ** 2).sum())
        lg = np.log(2 * np.sqrt(ell[prev[i]] * ell[i]) / LD(fs.a))
        terms = [gam[i] / (2 * PI) * (lg - (LD(fs.delta) - 1)) / sn * sd[i]]
        r = qp - fs.xyz[i].astype(LD)
        own = (seg == i) | (seg == prev[i])
        rr = np.sqrt((r[own] ** 2).sum(1))
        terms += list(-(erf_small(a * rr) / rr)[:, None] * qc[own] / (4 * PI))
        r = r[~own]
        r -= L * np.rint(r / L)
        rr = np.sqrt((r ** 2).sum(1))
        ok = rr < rc
        terms += list(((1 - erf_small(a * rr[ok])) / rr[ok])[:, None] * qc[~own][ok] / (4 * PI))
        psi[i] = np.array(terms).sum(0)
    return psi


@pytest.mark.parametrize("grid,rc_over_L,nfil,n,bound", [
    (64, 0.49, 5, 60, 1.25 * 2.61e-16),     # small input: pieces of filaments
    (68, 0.49, 5, 60, 1.25 * 1.81e-16),     # rows of cells: one cell
    (68, 0.2, 5, 60, 1.25 * 1.57e-16),      # many
    (68, 0.05, 30, 20, 1.25 * 4.52e-16),
])
def test_streamfunction_to_rounding(B, grid, rc_over_L, nfil, n, bound):
    fs = W.ellipses(nfil, n, seed=grid + nfil)
    alpha, rc = 0.5 / fs.L, rc_over_L * fs.L
    chord = np.linalg.norm(fs.xyz[1:n] - fs.xyz[:n - 1], axis=1).mean()
    fs.a = 2 * chord * math.exp(1 - fs.delta)
    print(f"\n[case] grid {grid}, rc/L {rc_over_L}, {fs.n_nodes} nodes", flush=True)
    plan = B.Plan(B.make_params(L=fs.L, a=fs.a, tol=1e-6, grid_n=grid, alpha=alpha, rcut=rc, beta=3.5))
    xyz, g = B.load_workload(fs)
    plan.set_filaments(fs.offsets, xyz, g)
    geo = {k: v.cpu().numpy() for k, v in plan.geometry().items()}
    Q = plan.params().Q
    _, psi = plan.energy()
    psi = psi.cpu().numpy()
    plan.status()
    plan.close()
    ref = reference(fs, geo, alpha, rc, Q)
    err = float(np.sqrt(((psi - ref) ** 2).mean() / (ref ** 2).mean()))
    print(f"  {err:.2e} (bound {bound:.2e})")
    assert err < bound
