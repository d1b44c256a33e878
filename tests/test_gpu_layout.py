"""A plan whose filaments change: its buffers are laid out anew in one allocation, which
grows or stays, so whatever the other filaments left in it must not be read.  Larger,
smaller, longer filaments (spline scratch), inputs with and without sorts and, with
the near-singular term, other cell grids; every result equals a fresh plan's, velocity
and energy to the bit (all sums are ordered)."""
import numpy as np
import pytest

from paper_2406_07366_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2406_07366_amd import binding
    return binding


def sets():
    return [W.ellipses(nfil=6, n_per=40, seed=1), W.tangle(nfil=60, n_per=100, seed=2),
            W.ellipses(nfil=3, n_per=300, seed=3), W.ellipses(nfil=1, n_per=16, seed=4),
            W.ringpairs(npairs=40, n_ring=16, nbg=4, seed=5), W.tangle(nfil=90, n_per=96, seed=6)]


def evaluate(plan, B, fs):
    import torch
    xyz, gamma = B.load_workload(fs)
    v, psi = torch.empty_like(xyz), torch.empty_like(xyz)
    plan.set_filaments(fs.offsets, xyz, gamma)
    plan.velocity(v)
    e, _ = plan.energy(psi)
    return v.cpu().numpy(), psi.cpu().numpy(), e


@pytest.mark.parametrize("grid,order,mixed,ns", [
    (64, 4, False, "BS_NS_OFF"), (68, 6, False, "BS_NS_OFF"), (64, 4, True, "BS_NS_OFF"),
    (64, 6, False, "BS_NS_ADAPTIVE"), (64, 4, True, "BS_NS_MAPPED")])
def test_other_filaments_in_the_same_plan(B, grid, order, mixed, ns):
    def plan():
        return B.Plan(B.make_params(L=W.TWO_PI, grid_n=grid, tol=1e-5 if mixed else 1e-6, a=1e-4,
                                    spline_order=order, ns_mode=getattr(B, ns),
                                    precision=B.BS_FP32_MIXED if mixed else B.BS_FP64))
    one = plan()
    for fs in sets():
        got, want = evaluate(one, B, fs), evaluate(plan(), B, fs)
        for a, b in zip(got, want):
            assert np.array_equal(a, b), (fs.n_nodes, np.abs(np.asarray(a) - np.asarray(b)).max())
