"""The float64 transforms on every grid size they are built for that is not a
power of two of at least 64 (which have a test of their own): velocity and
streamfunction against hipFFT's full transforms with the separate spectral
operator.  The two differ by the rounding of the transforms (at most nine
radix stages of a few 1e-16 each way): 1e-13 relative."""
import numpy as np
import pytest

from paper_2406_07366_amd import workloads as W

pytestmark = pytest.mark.gpu

SIZES = [16, 32, 40, 48, 56, 72, 80, 96, 112, 120, 144, 160, 168, 192, 200, 216, 224, 240, 280,
         288, 320, 336, 360, 384, 392, 400, 432, 448, 480, 504]


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available()
    from paper_2406_07366_amd import binding
    return binding


@pytest.mark.parametrize("n", SIZES)
def test_transforms_agree_with_hipfft(B, n):
    fs = W.ellipses(nfil=7, n_per=33, seed=n)
    rc = 0.45 * fs.L
    out = []
    print(f"\n[case] grid {n}", flush=True)
    for mode in (B.BS_FFT_AUTO, B.BS_FFT_LIBRARY):
        plan = B.Plan(B.make_params(L=fs.L, a=fs.a, tol=1e-6, grid_n=n, w=4 if n < 32 else 8,
                                    alpha=3.0 / rc, rcut=rc, fft_mode=mode))
        xyz, g = B.load_workload(fs)
        plan.set_filaments(fs.offsets, xyz, g)
        t = plan.velocity_terms()["long"].cpu().numpy()
        E, psi = plan.energy()
        plan.status()
        out.append((t, psi.cpu().numpy(), E))
        assert plan.params().fft_mode == (B.BS_FFT_LIBRARY)   # as it resolves on these grids
        plan.close()
    (va, pa, Ea), (vb, pb, Eb) = out
    dv = np.linalg.norm(va - vb) / np.linalg.norm(vb)
    dp = np.linalg.norm(pa - pb) / np.linalg.norm(pb)
    print(f"  v {dv:.2e} psi {dp:.2e}")
    assert dv < 1e-13 and dp < 1e-13 and abs(Ea - Eb) < 1e-13 * abs(Eb)
