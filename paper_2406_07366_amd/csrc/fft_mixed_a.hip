// Pruned transforms in float64 on grids that are not powers of two (multiples of 8
// from 40 to 504 with no prime factor above 7), one of four sets of sizes.
#include "fft_kernels.h"

namespace bs {

const FftOps *mixed_ops_a(int n) {
    switch (n) {
        case 40: return fft_ops_for<double, 40>();
        case 80: return fft_ops_for<double, 80>();
        case 144: return fft_ops_for<double, 144>();
        case 200: return fft_ops_for<double, 200>();
        case 280: return fft_ops_for<double, 280>();
        case 360: return fft_ops_for<double, 360>();
        case 432: return fft_ops_for<double, 432>();
        default: return nullptr;
    }
}

}  // namespace bs
