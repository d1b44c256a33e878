// Pruned transforms in float64 on grids that are not powers of two (multiples of 8
// from 40 to 504 with no prime factor above 7), one of four sets of sizes.
#include "fft_kernels.h"

namespace bs {

const FftOps *mixed_ops_c(int n) {
    switch (n) {
        case 56: return fft_ops_for<double, 56>();
        case 112: return fft_ops_for<double, 112>();
        case 168: return fft_ops_for<double, 168>();
        case 224: return fft_ops_for<double, 224>();
        case 320: return fft_ops_for<double, 320>();
        case 392: return fft_ops_for<double, 392>();
        case 480: return fft_ops_for<double, 480>();
        default: return nullptr;
    }
}

}  // namespace bs
