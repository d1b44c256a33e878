// Pruned transforms in float64 on grids that are not powers of two (multiples of 8
// from 40 to 504 with no prime factor above 7), one of four sets of sizes.
#include "fft_kernels.h"

namespace bs {

const FftOps *mixed_ops_b(int n) {
    switch (n) {
        case 48: return fft_ops_for<double, 48>();
        case 96: return fft_ops_for<double, 96>();
        case 160: return fft_ops_for<double, 160>();
        case 216: return fft_ops_for<double, 216>();
        case 288: return fft_ops_for<double, 288>();
        case 384: return fft_ops_for<double, 384>();
        case 448: return fft_ops_for<double, 448>();
        default: return nullptr;
    }
}

}  // namespace bs
