"""The binning of few nodes where the node cells are many (a loose tolerance on a
fine grid: 98^3 cells for 1280 nodes): the bins of every array count for the choice
of the scan.  In float64 it may take at most 60 us more than in mixed precision,
which has as many cells (it took 240 more with one workgroup over all cells)."""
import pytest

from paper_2406_07366_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2406_07366_amd import binding
    return binding


def test_many_node_cells(B):
    fs = W.ellipses(nfil=20, n_per=64, seed=5)
    us = {}
    for precision in (B.BS_FP64, B.BS_FP32_MIXED):
        print(f"\n[case] 1280 nodes on 256^3 at 1e-3, precision {precision}", flush=True)
        plan = B.Plan(B.make_params(L=fs.L, a=fs.a, tol=1e-3, grid_n=256, precision=precision))
        assert plan.params().ncell == 98
        xyz, g = B.load_workload(fs)
        plan.set_profiling(True)
        t = []
        for _ in range(6):
            plan.stage_times(reset=True)
            plan.set_filaments(fs.offsets, xyz, g)
            t.append(1e3 * plan.stage_times(reset=True)["binning"][0])
        plan.status()
        plan.close()
        us[precision] = min(t)
    print(f"  {us}")
    assert us[B.BS_FP64] < us[B.BS_FP32_MIXED] + 60.0
