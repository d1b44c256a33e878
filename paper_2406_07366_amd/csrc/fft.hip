// Pruned transforms: which grids they serve, their batch sizes and dispatch,
// and the instantiations for the powers of two (the other sizes are in
// fft_mixed_*.hip, split so that they compile side by side).
#include <algorithm>

#include "fft_kernels.h"

namespace bs {

// power of two, and the z pass's smallest batch (2 twiddle tables + 3
// columns + pad) fits LDS
bool pruned_fft_ok(int n, size_t csize) {
    return n >= 16 && n <= 1024 && (n & (n - 1)) == 0 && (size_t)n * 6 * csize < kFftLds &&
           3 * fft_max_nj(n) <= kFftMaxThreads;
}

// 16, 32 and the sizes of fft_mixed_*.hip: multiples of 8 from 40 to 504 that are
// not powers of two and have no prime factor above 7
bool pruned_auto64(int n) {
    if (n == 16 || n == 32) return true;
    if (n < 40 || n > 504 || n % 8 != 0 || (n & (n - 1)) == 0) return false;
    for (int f : {2, 3, 5, 7})
        while (n % f == 0) n /= f;
    return n == 1;
}

template <typename R>
static const FftOps *ops_pow2(int n) {
    switch (n) {
        case 16: return fft_ops_for<R, 16>();
        case 32: return fft_ops_for<R, 32>();
        case 64: return fft_ops_for<R, 64>();
        case 128: return fft_ops_for<R, 128>();
        case 256: return fft_ops_for<R, 256>();
        case 512: return fft_ops_for<R, 512>();
        case 1024:   // float64: refused by pruned_fft_ok
            if constexpr (sizeof(R) == 4) return fft_ops_for<R, 1024>();
            return nullptr;
        default: return nullptr;
    }
}

const FftOps *pruned_ops(int n, bool fp32) {
    const FftOps *o = fp32 ? ops_pow2<float>(n) : ops_pow2<double>(n);
    if (o || fp32) return o;
    if ((o = mixed_ops_a(n)) || (o = mixed_ops_b(n)) || (o = mixed_ops_c(n))) return o;
    return mixed_ops_d(n);
}

bool grid_interleaved(bs_plan_t p) { return p->pruned && p->n > kFftXYMax; }

void pruned_forward(bs_plan_t p) { p->fft_ops->forward(p); }
void pruned_spectral_op(bs_plan_t p, int psi) { p->fft_ops->spectral(p, psi); }
void pruned_inverse(bs_plan_t p) { p->fft_ops->inverse(p); }


// Columns per workgroup of the z pass on planes (times 3 components): 3 kz
// sequences of mnj items, about 256 threads (128 in float64) of ipt items each and
// at most kFftMaxThreads, with 2 twiddle tables and 3 kz + 1 columns in the LDS.
int pruned_z_batch(int n, size_t csize) {
    const int mnj = fft_max_nj(n), ipt = z_ipt(n, (int)csize);
    const int threads = csize > 8 ? 128 : 256;
    const int lds = (int)(kFftLds / (csize * (n + n / 16 + 1))) - 2;
    const int b = std::max(1, std::min(threads / mnj, lds));
    int p2 = 1;   // the power of two below
    while (2 * p2 <= b) p2 *= 2;
    const size_t zlds = ipt > 1 ? kFftLdsZ : kFftLds;
    int z = std::max(1, ipt > 1 ? kFftMaxThreads * ipt / (3 * mnj) : p2 / 3);
    while (z > 1 && ((size_t)(2 * n + n * (3 * z + 1)) * csize > zlds ||
                     ceil_div(3 * z * mnj, ipt) > kFftMaxThreads))
        z--;
    return z;
}

}  // namespace bs
