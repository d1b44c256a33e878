// Pruned transforms in float64 on grids that are not powers of two (multiples of 8
// from 40 to 504 with no prime factor above 7), one of four sets of sizes.
#include "fft_kernels.h"

namespace bs {

const FftOps *mixed_ops_d(int n) {
    switch (n) {
        case 72: return fft_ops_for<double, 72>();
        case 120: return fft_ops_for<double, 120>();
        case 192: return fft_ops_for<double, 192>();
        case 240: return fft_ops_for<double, 240>();
        case 336: return fft_ops_for<double, 336>();
        case 400: return fft_ops_for<double, 400>();
        case 504: return fft_ops_for<double, 504>();
        default: return nullptr;
    }
}

}  // namespace bs
