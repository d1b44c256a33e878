"""The direct path of small float64 inputs (no counting sorts) at the edges of
what it takes: filaments longer than the per-filament kernel holds, pieces cut
short, the largest point count and the first beyond it, the narrowest and
widest kernels, quintic splines beyond the LDS solve, infinite filaments.

Local, self and short-range terms against the oracle's over the same points
(float64 in another order: 1e-11 leaves room for cancellation between terms of
the quintic solve).  The spread against the general path: the vorticity's Fourier
coefficients are linear in the filaments, so those of the set are those of the
set with 140 more ellipses (too many points for the direct path) minus those
of the 140 alone, to the rounding of the larger sums (at most ~1e3 times the
set's own coefficients: 1e-12).  The whole velocity is the sum of the terms to
rounding."""
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
    # name, filaments, grid, w, spline order, Q
    ("one point run", lambda: W.ellipses(1, 3, seed=1), 32, 8, 4, 1),
    ("ragged pieces", lambda: W.ellipses(9, 33, seed=2), 40, 4, 4, 3),
    ("per-filament limit", lambda: W.ellipses(3, 128, seed=3), 64, 16, 4, 2),
    ("beyond it", lambda: W.ellipses(3, 129, seed=4), 64, 8, 4, 2),
    ("one long filament", lambda: W.trefoil(1000), 64, 8, 4, 4),
    ("quintic in LDS", lambda: W.ellipses(4, 64, seed=5), 32, 12, 6, 3),
    ("quintic beyond LDS", lambda: W.ellipses(4, 65, seed=6), 32, 12, 6, 3),
    ("infinite", lambda: W.helices(48), 32, 8, 4, 2),
    ("most points", lambda: W.ellipses(64, 64, seed=7), 64, 8, 4, 2),
    ("nearly as many", lambda: W.ellipses(63, 65, seed=8), 64, 8, 4, 2),
    ("two workgroups a filament", lambda: W.ellipses(100, 21, seed=10), 64, 8, 4, 2),
    ("one workgroup a filament", lambda: W.ellipses(200, 13, seed=11), 64, 8, 6, 3),
    ("larger grid", lambda: W.ellipses(20, 50, seed=9), 128, 6, 6, 2),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_terms_and_spread(B, case):
    import torch
    name, make, n, w, order, Q = case
    fs = make()
    print(f"\n[case] {name}: N {fs.n_nodes} grid {n} w {w} order {order}", flush=True)
    rc = 0.45 * fs.L if n < 64 else 0.2 * fs.L
    plan = B.Plan(B.make_params(L=fs.L, a=fs.a, tol=1e-6, grid_n=n, w=w, alpha=3.5 / rc, rcut=rc,
                                Q=Q, spline_order=order))
    if fs.periods is not None:
        plan.set_periods(fs.periods)
    xyz, g = B.load_workload(fs)
    plan.set_filaments(fs.offsets, xyz, g)
    t = {k: v.cpu().numpy() for k, v in plan.velocity_terms().items()}
    v = plan.velocity().cpu().numpy()
    plan.status()
    o = O.Oracle(fs, Q=Q, order=order)
    ref = {"local": o.local()[0], "self": o.selfcorr(3.5 / rc)[0]}
    tg = np.arange(0, fs.n_nodes, max(1, fs.n_nodes // 400))
    ref["short"] = np.zeros_like(v)
    ref["short"][tg] = o.shortrange(3.5 / rc, rc, targets=tg, psi=False)[0]
    scale = np.sqrt((v ** 2).mean())
    for k, r in ref.items():
        i = tg if k == "short" else slice(None)
        e = np.sqrt(((t[k][i] - r[i]) ** 2).mean()) / max(scale, np.sqrt((r[i] ** 2).mean()))
        print(f"  {k} {e:.2e}")
        assert e < 1e-11, k
    whole = np.linalg.norm(v - (t["local"] + t["short"] + t["long"] - t["self"])) / np.linalg.norm(v)
    print(f"  whole {whole:.2e}")
    assert whole < 1e-12
    m = plan.vorticity_modes().cpu().numpy()
    more = W.ellipses(140, 64, seed=99)
    off = np.concatenate([fs.offsets, fs.offsets[-1] + more.offsets[1:]])
    x2 = torch.cat([xyz, torch.from_numpy(more.xyz).cuda()])
    g2 = torch.cat([g, torch.from_numpy(more.gamma).cuda()])
    if fs.periods is not None:
        plan.set_periods(np.concatenate([fs.periods, np.zeros((140, 3), np.int64)]))
    plan.set_filaments(off, x2, g2)
    both = plan.vorticity_modes().cpu().numpy()
    plan.set_periods(None)
    plan.set_filaments(more.offsets, x2[fs.n_nodes:].contiguous(), g2[fs.n_fil:].contiguous())
    rest = plan.vorticity_modes().cpu().numpy()
    plan.status()
    e = np.linalg.norm(m - (both - rest)) / np.linalg.norm(m)
    print(f"  spread against the general path {e:.2e}")
    assert e < 1e-12
    plan.close()
