"""The transforms a plan says it runs, on every size with own ones: BS_FFT_AUTO
in float64 runs them, an explicit BS_FFT_LIBRARY, a plan made again from the
resolved parameters, and mixed precision below the powers of two do not; the
plan's answer is the host's.  Where the two differ their velocities differ too,
by rounding (a plan that silently fell back would give equal bits)."""
import numpy as np
import pytest

from paper_2406_07366_amd import workloads as W
from tests.test_gpu_fft_sizes import SIZES

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2406_07366_amd import binding
    return binding


@pytest.mark.parametrize("n", SIZES)
def test_a_plan_reports_the_transforms_it_runs(B, n):
    fs = W.ellipses(nfil=7, n_per=33, seed=n)
    rc = 0.45 * fs.L
    print(f"\n[case] grid {n}", flush=True)

    def run(prm):
        plan = B.Plan(prm)
        assert plan.transforms() == B.params_transforms(prm)
        xyz, g = B.load_workload(fs)
        plan.set_filaments(fs.offsets, xyz, g)
        v = plan.velocity_terms()["long"].cpu().numpy()
        out = plan.transforms(), v, plan.params()
        plan.close()
        return out

    def params(mode):
        return B.make_params(L=fs.L, a=fs.a, tol=1e-6, grid_n=n, w=4 if n < 32 else 8,
                             alpha=3.0 / rc, rcut=rc, fft_mode=mode)

    own, va, resolved = run(params(B.BS_FFT_AUTO))
    lib, vb, _ = run(params(B.BS_FFT_LIBRARY))
    assert own == B.BS_FFT_PRUNED and lib == B.BS_FFT_LIBRARY
    assert not np.array_equal(va, vb)
    assert np.linalg.norm(va - vb) < 1e-13 * np.linalg.norm(vb)
    again, vc, _ = run(resolved)
    assert again == B.BS_FFT_LIBRARY
    resolved.fft_mode = B.BS_FFT_AUTO
    again, vc, _ = run(resolved)
    assert again == own and np.array_equal(vc, va)


def test_mixed_precision_and_other_sizes(B):
    for n, precision, want in ((48, B.BS_FP32_MIXED, B.BS_FFT_LIBRARY), (64, B.BS_FP32_MIXED, B.BS_FFT_PRUNED),
                               (24, B.BS_FP64, B.BS_FFT_LIBRARY), (44, B.BS_FP64, B.BS_FFT_LIBRARY),
                               (88, B.BS_FP64, B.BS_FFT_LIBRARY), (64, B.BS_FP64, B.BS_FFT_PRUNED)):
        print(f"\n[case] grid {n} precision {precision}", flush=True)
        prm = B.make_params(L=6.0, a=1e-6, tol=1e-3, grid_n=n, w=4, alpha=2.0, rcut=2.0,
                            precision=precision)
        plan = B.Plan(prm)
        assert plan.transforms() == want == B.params_transforms(prm)
        plan.close()


def test_own_transforms_share_hipfft_memory(B):
    """At 384^3 in float64, where hipFFT needs no work area, a plan with its own
    transforms holds one array of 3 (2K+1) n (K+1) complex values more than one
    without, and no second one of 3 n^2 (K+1) beside the spectrum."""
    import torch
    n, used = 384, {}
    torch.zeros(1, device="cuda")
    for mode in (B.BS_FFT_LIBRARY, B.BS_FFT_AUTO, B.BS_FFT_LIBRARY, B.BS_FFT_AUTO):
        print(f"\n[case] plan at {n}, mode {mode}", flush=True)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        plan = B.Plan(B.make_params(L=6.0, a=1e-6, tol=1e-6, grid_n=n, fft_mode=mode))
        torch.cuda.synchronize()
        used[mode] = before - torch.cuda.mem_get_info()[0]
        K = plan.params().K
        plan.close()
    extra = used[B.BS_FFT_AUTO] - used[B.BS_FFT_LIBRARY]
    print(f"  {used}, extra {extra / 1e6:.0f} MB")
    assert extra < 3 * (2 * K + 1) * n * (K + 1) * 16 + (64 << 20)
