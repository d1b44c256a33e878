"""The float64 short-range kernel at the edges of its cell lists: one cell,
the fewest rows (5 per axis), rows beyond the periodic boundary, and more
candidates than one chunk of start marks holds; velocity (one wavefront per
target and, alone, four) and streamfunction against the oracle's sums over the
same quadrature points.  Both sum the same terms in float64 in different
orders: at most ~1e4 terms, so rounding stays below 1e-12."""
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


@pytest.mark.parametrize("rc_over_L,nfil,n_per", [
    (0.49, 3, 37),       # one cell
    (0.3999, 40, 21),    # five rows per axis (the edges' room for the margin)
    (0.33, 120, 40),     # ~3000 candidates per target
    (0.12, 1, 200),      # fewer cells than fit: at most one per point
    (0.05, 300, 60),     # many rows; 18000 targets (one wavefront each)
])
def test_short_range_rows(B, rc_over_L, nfil, n_per):
    fs = W.ellipses(nfil=nfil, n_per=n_per, seed=nfil)
    L = fs.L
    rc = rc_over_L * L
    plan = B.Plan(B.make_params(L=L, a=fs.a, tol=1e-6, grid_n=64, alpha=3.0 / rc, rcut=rc))
    xyz, g = B.load_workload(fs)
    plan.set_filaments(fs.offsets, xyz, g)
    t = plan.velocity_terms()
    v, lng, loc, slf = (t[k].cpu().numpy() for k in ("short", "long", "local", "self"))
    total = plan.velocity().cpu().numpy()
    plan.status()
    tg = np.arange(0, fs.n_nodes, max(1, fs.n_nodes // 500))
    ref, _ = O.Oracle(fs).shortrange(3.0 / rc, rc, targets=tg, psi=False)
    err = np.linalg.norm(v[tg] - ref) / np.linalg.norm(ref)
    whole = np.linalg.norm(total - (loc + v + lng - slf)) / np.linalg.norm(total)
    print(f"\n[case] rc/L {rc_over_L} N {fs.n_nodes}: short {err:.2e}, sum of terms {whole:.2e}",
          flush=True)
    assert err < 1e-12 and whole < 1e-12
    # streamfunction: the short-range term enters psi alone, so compare whole
    # values against a plan whose split differs (the oracle at small sizes)
    if fs.n_nodes <= 1000:
        _, psi = plan.energy()
        o = O.Oracle(fs)
        p = plan.params()
        _, pl = o.local()
        _, ps = o.shortrange(p.alpha, p.rcut, psi=True)
        _, pS = o.selfcorr(p.alpha)
        _, pL = o.longrange(p.alpha, p.K, psi=True)
        ref = pl + ps + pL - pS
        e = np.linalg.norm(psi.cpu().numpy() - ref) / np.linalg.norm(ref)
        print(f"  psi {e:.2e}")
        assert e < 1e-6          # the long-range part's NUFFT (w = 8)
    plan.close()
