// The graded panels of a near-singular integral over u in [0, 1], also compiled for
// the host by their test.
#pragma once
#include <math.h>

#ifndef BS_HD
#define BS_HD __host__ __device__ __forceinline__
#endif

namespace bs {

// Panel 0 is the centre panel [ub - delta, ub + delta], panels 1 .. left those to
// its left up to 0, each ending at three times the distance from ub at which it
// begins, the rest those to its right up to 1.  The outermost ones end at 0 and 1
// whatever the rounding of the distances: the count alone says how many there
// are, so that a bound formed with another rounding moves no panel.  None when
// the distance is not a number.
struct NsPanels {
    int n, left;
};
BS_HD NsPanels ns_panels(double ub, double delta) {
    const double a0 = ub - delta < 0.0 ? 0.0 : ub - delta, b0 = ub + delta > 1.0 ? 1.0 : ub + delta;
    NsPanels p = {0, 0};
    if (!(b0 > a0)) return p;
    p.n = 1;
    for (double e = a0, w = delta; e > 0.0; w *= 3.0, p.left++) e = ub - 3.0 * w;
    for (double e = b0, w = delta; e < 1.0; w *= 3.0, p.n++) e = ub + 3.0 * w;
    p.n += p.left;
    return p;
}
// bounds of panel k < p.n
BS_HD void ns_panel_bounds(double ub, double delta, NsPanels p, int k, double *lo, double *hi) {
    const double a0 = fmax(ub - delta, 0.0), b0 = fmin(ub + delta, 1.0);
    *lo = a0;
    *hi = b0;
    if (k == 0) return;
    const bool left = k <= p.left;
    const int j = left ? k : k - p.left, last = left ? p.left : p.n - 1 - p.left;
    double w = delta, in = left ? a0 : b0;   // the panel's inner bound
    for (int i = 1; i < j; i++, w *= 3.0) in = left ? fmax(ub - 3.0 * w, 0.0) : fmin(ub + 3.0 * w, 1.0);
    if (left) {
        *hi = in;
        *lo = j == last ? 0.0 : fmax(ub - 3.0 * w, 0.0);
    } else {
        *lo = in;
        *hi = j == last ? 1.0 : fmin(ub + 3.0 * w, 1.0);
    }
}

}  // namespace bs
