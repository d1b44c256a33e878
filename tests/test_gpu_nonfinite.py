"""A node that is not finite is reported by the status; what the short-range sums make of
it is the same on the direct path (64^3) and through the sorts (68^3): every target
within r_c of where such points fold to is not a number, the others are untouched."""
import numpy as np
import pytest

from paper_2406_07366_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2406_07366_amd import binding
    return binding


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("nfil,n", [(30, 40), (6, 300)])   # all of a filament's points, some
def test_short_range_with_a_bad_node(B, bad, nfil, n):
    fs = W.ellipses(nfil=nfil, n_per=n, seed=3)
    for f in (0, 1):                      # around the origin
        fs.xyz[f * n:(f + 1) * n] -= fs.xyz[f * n:(f + 1) * n].mean(0)
    fs.xyz[n + 5, 1] = bad
    rc = 0.2 * fs.L
    out = []
    for grid in (64, 68):
        print(f"\n[case] {bad} in a node, grid {grid}", flush=True)
        plan = B.Plan(B.make_params(L=fs.L, a=fs.a, tol=1e-6, grid_n=grid, alpha=3.5 / rc, rcut=rc))
        xyz, g = B.load_workload(fs)
        plan.set_filaments(fs.offsets, xyz, g)
        out.append(plan.velocity_terms()["short"].cpu().numpy())
        with pytest.raises(B.BsError):
            plan.status()
        plan.close()
    a, b = (np.isfinite(v).all(1) for v in out)
    print(f"  finite {a.sum()} {b.sum()} of {fs.n_nodes}")
    other = np.arange(fs.n_nodes) // n != 1
    assert np.array_equal(a[other], b[other])
    assert 0 < (~b[other]).sum() < other.sum()
    both = a & b & other
    assert np.abs(out[0][both] - out[1][both]).max() < 1e-12 * np.abs(out[1][both]).max()
