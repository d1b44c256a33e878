// C ABI of libbs.so: parameter resolution, plan and buffer management, and
// the order of the steps of one velocity / energy evaluation.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>

#include "bs_internal.h"
#include "direct.h"

namespace bs {

static thread_local std::string g_err = "no error";

int set_error(bs_plan_t p, int code, const std::string &msg) {
    if (p) p->err = msg;
    else g_err = msg;
    return code;
}

int check_hip(bs_plan_t p, hipError_t e, const char *what) {
    if (e == hipSuccess) return BS_OK;
    return set_error(p, e == hipErrorOutOfMemory ? BS_ENOMEM : BS_EDEVICE,
                     std::string(what) + ": " + hipGetErrorString(e));
}

// Gauss-Legendre rule on [-1, 1] by Newton iteration on the three-term
// recurrence of the Legendre polynomials; nodes ascending.
static void legendre_rule(int n, double *x, double *w) {
    for (int i = 0; i < n; i++) {
        double z = std::cos(kPi * (i + 0.75) / (n + 0.5)), dp = 1.0;
        for (int it = 0; it < 100; it++) {
            double p0 = 1.0, p1 = z;
            for (int k = 2; k <= n; k++) {
                double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
                p0 = p1; p1 = p2;
            }
            if (n == 1) { p1 = z; p0 = 1.0; }
            dp = n * (z * p1 - p0) / (z * z - 1.0);
            double dz = p1 / dp;
            z -= dz;
            if (std::fabs(dz) < 1e-16) break;
        }
        // recompute derivative at the converged node
        double p0 = 1.0, p1 = z;
        for (int k = 2; k <= n; k++) {
            double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
            p0 = p1; p1 = p2;
        }
        if (n == 1) { p1 = z; p0 = 1.0; }
        dp = n * (z * p1 - p0) / (z * z - 1.0);
        x[n - 1 - i] = z;
        w[n - 1 - i] = 2.0 / ((1.0 - z * z) * dp * dp);
    }
}

GLRule gl_rule(int Q) {
    GLRule r{};
    double x[kMaxQ], w[kMaxQ];
    if (Q == 1) { x[0] = 0.0; w[0] = 2.0; }
    else legendre_rule(Q, x, w);
    for (int i = 0; i < Q; i++) { r.h[i] = 0.5 * (x[i] + 1.0); r.w[i] = 0.5 * w[i]; }
    return r;
}

// Host copy of the normalised kernel phi(z) = sinh(zeta s)/(sinh(zeta) s),
// s = sqrt(1 - z^2) (same normalisation as the device kernel).
static double kb_phi_host(double z, double zeta) {
    double s2 = 1.0 - z * z;
    double den = -std::expm1(-2.0 * zeta);
    if (s2 <= 0.0) return 2.0 * zeta * std::exp(-zeta) / den;
    double s = std::sqrt(s2);
    return std::exp(zeta * (s - 1.0)) * (-std::expm1(-2.0 * zeta * s)) / s / den;
}

// F(m) = (w/2) int_{-1}^{1} phi(z) cos(pi m w z / n) dz, the transform of the
// spreading kernel per axis (Poisson summation of the grid sum; App. A).
// The integrand is analytic on [-1,1], so a 256-point Gauss-Legendre rule is
// exact to rounding.  (The closed form I0(sqrt(zeta^2 - kappa^2)) of
// eq:kaiser_bessel_bw is the transform of the kernel continued beyond
// |z| = 1 and differs from the truncated kernel's by ~e^{-zeta}.)
static void kernel_ft_table(int K, int w, int n, double zeta, double *F) {
    const int nq = 256;
    std::vector<double> x(nq), wt(nq), ph(nq);
    legendre_rule(nq, x.data(), wt.data());
    for (int i = 0; i < nq; i++) ph[i] = kb_phi_host(x[i], zeta);
    for (int m = 0; m <= K; m++) {
        double kap = kPi * m * w / n, s = 0.0;
        for (int i = 0; i < nq; i++) s += wt[i] * ph[i] * std::cos(kap * x[i]);
        F[m] = 0.5 * w * s;
    }
}

// Gauss-Legendre rules of the near-singular integrals: 16 points (the mapped
// rule, each side of the peak), 10 and 12 points (the graded panels on cubic
// and quintic segments)
struct NsRule {
    double x[16], w[16];
    double x10[10], w10[10];
    double x12[12], w12[12];
};
void ns_rule(NsRule *R) {
    static const NsRule cached = [] {
        NsRule r;
        legendre_rule(16, r.x, r.w);
        legendre_rule(10, r.x10, r.w10);
        legendre_rule(12, r.x12, r.w12);
        return r;
    }();
    *R = cached;
}

template <typename T>
static int ensure(bs_plan_t p, DBuf &b, size_t count) {
    size_t bytes = std::max<size_t>(count * sizeof(T), 256);
    if (b.bytes >= bytes) return BS_OK;
    if (b.p) { (void)hipFree(b.p); b.p = nullptr; b.bytes = 0; }
    hipError_t e = hipMalloc(&b.p, bytes);
    if (e != hipSuccess) { b.p = nullptr; return check_hip(p, e, "hipMalloc"); }
    b.bytes = bytes;
    return BS_OK;
}

static void release(DBuf &b) {
    if (b.p) (void)hipFree(b.p);
    b.p = nullptr;
    b.bytes = 0;
}

// Buffers that are parts of one allocation, P->points: they own nothing, and a new
// layout may move them all, so nothing in them outlives it.
struct Part {
    DBuf *buf;
    size_t bytes;
};
template <typename T>
static Part part(DBuf &b, size_t count) {
    return {&b, std::max<size_t>(count * sizeof(T), 256)};
}
static int lay_out(bs_plan_t p, const std::vector<Part> &parts) {
    constexpr size_t align = 4096;
    size_t total = 0;
    for (const Part &q : parts) {
        *q.buf = DBuf{};
        total += (q.bytes + align - 1) / align * align;
    }
    int rc = ensure<char>(p, p->points, total);
    if (rc) return rc;
    char *at = (char *)p->points.p;
    for (const Part &q : parts) {
        *q.buf = DBuf{at, q.bytes};
        at += (q.bytes + align - 1) / align * align;
    }
    return BS_OK;
}

__global__ void k_fill_f64(double *p, size_t n, double v) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

static void fill_f64(bs_plan_t p, double *ptr, size_t n, double v) {
    if (n == 0) return;
    hipLaunchKernelGGL(k_fill_f64, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, p->stream, ptr,
                       n, v);
}

__global__ void k_add_f64(double *__restrict__ y, const double *__restrict__ x, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] += x[i];
}

static void add_f64(bs_plan_t p, double *y, const double *x, size_t n) {
    if (n == 0) return;
    hipLaunchKernelGGL(k_add_f64, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, p->stream, y, x,
                       n);
}

static int launch_status(bs_plan_t p, const char *what) {
    return check_hip(p, hipGetLastError(), what);
}

// Table 1 of the paper: nominal tolerance -> beta and kernel width w.
static const double kTabTol[7] = {1e-3, 1e-4, 1e-6, 1e-8, 1e-10, 1e-12, 1e-14};
static const double kTabBeta[7] = {2.0, 2.5, 3.5, 4.0, 4.5, 5.0, 5.5};
static const int kTabW[7] = {4, 6, 8, 10, 12, 14, 16};

static double beta_from_tol(double tol) {
    for (int i = 0; i < 7; i++)
        if (kTabTol[i] <= tol * (1.0 + 1e-9)) return kTabBeta[i];
    return kTabBeta[6];
}

// a tolerance of the table takes the table's width; any other the App. A
// decay law 10^(-0.9 w)
static int width_from_tol(double tol) {
    for (int i = 0; i < 7; i++)
        if (std::fabs(tol - kTabTol[i]) <= 1e-9 * kTabTol[i]) return kTabW[i];
    double pe = -std::log10(tol);
    int w = (int)std::ceil(pe / 0.9 - 1e-9) + 1;
    return std::min(kMaxW, std::max(kMinW, w));
}

int resolve(const bs_params *in, bs_params *out) {
    if (!in || !out) return set_error(nullptr, BS_EINVAL, "null parameter pointer");
    bs_params r = *in;
    auto bad = [](const char *m) { return set_error(nullptr, BS_EINVAL, m); };
    if (!(std::isfinite(r.L) && r.L > 0)) return bad("L must be positive");
    if (!(std::isfinite(r.a) && r.a > 0 && r.a < r.L)) return bad("a must be in (0, L)");
    if (!std::isfinite(r.delta)) return bad("delta must be finite");
    if (!(r.tol > 0 && r.tol <= 0.5)) return bad("tol must be in (0, 0.5]");
    if (r.grid_n < 16 || r.grid_n % 4 != 0 || r.grid_n > 1024)
        return bad("grid_n must be a multiple of 4 in [16, 1024]");
    if (r.sigma == 0) r.sigma = 1.5;
    if (!(r.sigma > 1.0 && r.sigma <= 4.0)) return bad("sigma must be in (1, 4]");
    if (r.Q == 0) r.Q = 2;
    if (r.Q < 1 || r.Q > kMaxQ) return bad("Q must be in 1..4");
    if (r.spline_order == 0) r.spline_order = 4;
    if (r.spline_order != 4 && r.spline_order != 6)
        return bad("spline_order must be 4 (cubic) or 6 (quintic)");
    if (!(r.local_frac >= 0.0 && r.local_frac <= 1.0)) return bad("local_frac must be in [0, 1]");
    if (r.local_frac > 0.0 && r.local_frac < 1e-3)
        return bad("local_frac below 1e-3 (more than 10 panels per local segment)");
    if (r.precision != BS_FP64 && r.precision != BS_FP32_MIXED) return bad("unknown precision");
    if (r.ns_mode < BS_NS_OFF || r.ns_mode > BS_NS_MAPPED) return bad("unknown ns_mode");
    if (r.ns_mode == BS_NS_MLP && r.spline_order != 4)
        return bad("the learned near-singular correction is trained on cubic segments only");
    if (r.ns_eta == 0) r.ns_eta = 1.0;
    if (!(r.ns_eta > 0)) return bad("ns_eta must be positive");
    if (r.fft_mode < BS_FFT_AUTO || r.fft_mode > BS_FFT_PRUNED) return bad("unknown fft_mode");
    {
        const bool ok = pruned_fft_ok(r.grid_n, r.precision == BS_FP32_MIXED ? 8 : 16);
        if (r.fft_mode == BS_FFT_PRUNED && !ok)
            return bad("BS_FFT_PRUNED needs grid_n a power of two (at most 512 in float64)");
        // automatic choice: the pruned transforms win from 64^3 up (measured);
        // hipFFT on smaller grids
        if (r.fft_mode == BS_FFT_AUTO)
            r.fft_mode = (ok && r.grid_n >= 64) ? BS_FFT_PRUNED : BS_FFT_LIBRARY;
    }
    if (r.beta == 0) r.beta = beta_from_tol(r.tol);
    if (!(r.beta > 0)) return bad("beta must be positive");
    if (r.w == 0) r.w = width_from_tol(r.tol);
    if (r.w < kMinW || r.w > kMaxW) return bad("w must be in 4..16");
    {
        // every stencil must reach a spread tile at most once along an axis
        int T = (r.grid_n % 8 == 0) ? 8 : 4;
        if (r.grid_n < r.w + T) return bad("grid_n must be at least w + 8 (w + 4 if not a multiple of 8)");
    }
    int M = (int)std::floor(r.grid_n / r.sigma + 1e-9);
    r.K = (M - 1) / 2;
    if (r.K < 1) return bad("grid too small for one retained mode");
    bool derived = (in->alpha == 0 && in->rcut == 0);
    if (r.alpha == 0) r.alpha = r.K * (2.0 * kPi / r.L) / (2.0 * r.beta);
    if (!(r.alpha > 0)) return bad("alpha must be positive");
    if (r.rcut == 0) r.rcut = r.beta / r.alpha;
    if (!(r.rcut > 0)) return bad("rcut must be positive");
    if (r.rcut > 0.5 * r.L * (1.0 + 1e-12)) {
        if (derived)
            return set_error(nullptr, BS_ETOL,
                             "tolerance needs r_c = beta/alpha > L/2 on this grid; use a larger "
                             "grid_n");
        return set_error(nullptr, BS_EMINIMG, "rcut > L/2 violates the minimum-image convention");
    }
    r.zeta = 0.995 * r.w * kPi * (1.0 - 1.0 / (2.0 * r.sigma));
    double kap_max = kPi * r.K * r.w / r.grid_n;
    if (kap_max >= r.zeta)
        return set_error(nullptr, BS_EKB, "retained modes beyond the kernel's band (raise sigma)");
    // short-range cells of edge >= 2 r_c / 3: the points within r_c of any
    // target lie in a 4 x 4 x 4 block of cells (one cell when fewer than 4
    // fit along an axis)
    int nc = (int)std::floor(3.0 * r.L / (2.0 * r.rcut * (1.0 + 1e-6)));
    if (nc < 4) nc = 1;
    if (nc > 160) nc = 160;
    r.ncell = nc;
    *out = r;
    return BS_OK;
}

// Whether a plan of parameters in (resolved: r) runs its own transforms.
// BS_FFT_AUTO resolves to BS_FFT_LIBRARY on grids that are no power of two
// (BS_FFT_PRUNED refuses them) and below 64; in float64 the plan still runs
// its own transforms there where it has them: hipFFT's form all modes
// and need a pass of the spectral operator (384^3: 5.69 ms against 1.91;
// 160^3: 280 us, 162; 32^3: 20.5, 15).  In
// float32 their rounding would change results, so those stay on hipFFT, as
// does an explicit BS_FFT_LIBRARY, and 1024^3 in float64, which
// BS_FFT_PRUNED refuses (its arrays would add 29 GB).
static bool runs_pruned(const bs_params &in, const bs_params &r) {
    return r.fft_mode == BS_FFT_PRUNED ||
           (in.fft_mode == BS_FFT_AUTO && r.precision == BS_FP64 && pruned_auto64(r.grid_n));
}

void stage_collect(bs_plan_t p) {
    if (!p->prof) return;
    (void)hipStreamSynchronize(p->stream);
    for (int s = 0; s < BS_NSTAGES; s++) {
        if (!p->ev_used[s]) continue;
        float ms = 0.0f;
        if (hipEventElapsedTime(&ms, p->ev_beg[s], p->ev_end[s]) == hipSuccess) {
            p->stage_ms[s] += ms;
            p->stage_cnt[s] += 1;
        }
        p->ev_used[s] = false;
    }
}

}  // namespace bs

using namespace bs;

extern "C" {

int bs_set_profiling(bs_plan_t P, int enable) {
    if (!P) return set_error(nullptr, BS_EINVAL, "null plan");
    if (enable && !P->ev_beg[0]) {
        for (int s = 0; s < BS_NSTAGES; s++) {
            int rc = check_hip(P, hipEventCreate(&P->ev_beg[s]), "hipEventCreate");
            if (!rc) rc = check_hip(P, hipEventCreate(&P->ev_end[s]), "hipEventCreate");
            if (rc) return rc;
        }
    }
    P->prof = enable != 0;
    return BS_OK;
}

int bs_stage_times(bs_plan_t P, double *ms, int64_t *counts, int reset) {
    if (!P) return set_error(nullptr, BS_EINVAL, "null plan");
    for (int s = 0; s < BS_NSTAGES; s++) {
        if (ms) ms[s] = P->stage_ms[s];
        if (counts) counts[s] = P->stage_cnt[s];
        if (reset) { P->stage_ms[s] = 0.0; P->stage_cnt[s] = 0; }
    }
    return BS_OK;
}

int bs_resolve_params(const bs_params *p, bs_params *out) { return resolve(p, out); }

int bs_params_transforms(const bs_params *p) {
    bs_params r;
    const int rc = resolve(p, &r);
    if (rc) return rc;
    return runs_pruned(*p, r) ? BS_FFT_PRUNED : BS_FFT_LIBRARY;
}

const char *bs_last_error(bs_plan_t plan) { return plan ? plan->err.c_str() : g_err.c_str(); }

int bs_plan(const bs_params *p, void *hip_stream, bs_plan_t *out) {
    if (!out) return set_error(nullptr, BS_EINVAL, "null output handle");
    *out = nullptr;
    bs_params r;
    int rc = resolve(p, &r);
    if (rc) return rc;
    bs_plan_t P = new bs_plan_s();
    P->prm = r;
    P->stream = (hipStream_t)hip_stream;
    P->fp32 = (r.precision == BS_FP32_MIXED);
    P->real_size = P->fp32 ? 4 : 8;
    P->n = r.grid_n;
    P->T = (P->n % 8 == 0) ? 8 : 4;
    P->NT = P->n / P->T;
    P->nc = r.ncell;
    P->Q = r.Q;
    P->order = r.spline_order;
    (void)hipGetDevice(&P->device);
    const size_t n = (size_t)P->n, n3 = n * n * n, nc = n * n * (n / 2 + 1);
    auto fail = [&](int code) {
        g_err = P->err;
        bs_destroy(P);
        return code;
    };
    if ((rc = check_hip(P, hipStreamCreateWithFlags(&P->side, hipStreamNonBlocking),
                        "hipStreamCreateWithFlags")) ||
        (rc = check_hip(P, hipEventCreateWithFlags(&P->ev_fork, hipEventDisableTiming),
                        "hipEventCreateWithFlags")) ||
        (rc = check_hip(P, hipEventCreateWithFlags(&P->ev_join, hipEventDisableTiming),
                        "hipEventCreateWithFlags")) ||
        (rc = check_hip(P, hipEventCreateWithFlags(&P->ev_ns, hipEventDisableTiming),
                        "hipEventCreateWithFlags")))
        return fail(rc);
    if ((rc = ensure<char>(P, P->grid, 3 * n3 * P->real_size))) return fail(rc);
    if ((rc = ensure<char>(P, P->spec, 3 * nc * 2 * P->real_size))) return fail(rc);
    if ((rc = ensure<double>(P, P->deconv, 2 * (r.K + 1)))) return fail(rc);
    if ((rc = ensure<int>(P, P->d_status, 1))) return fail(rc);
    if ((rc = ensure<int>(P, P->red_tmp, 3 * 8192))) return fail(rc);
    if ((rc = ensure<int>(P, P->scan_tmp, 8192))) return fail(rc);
    if ((rc = check_hip(P, hipMemsetAsync(P->d_status.p, 0, sizeof(int), P->stream), "memset")))
        return fail(rc);
    // deconvolution table: [1/F(m)] then [1/F(m)^2], m = 0..K
    std::vector<double> F(r.K + 1), tab(2 * (r.K + 1));
    kernel_ft_table(r.K, r.w, P->n, r.zeta, F.data());
    for (int m = 0; m <= r.K; m++) {
        tab[m] = 1.0 / F[m];
        tab[r.K + 1 + m] = 1.0 / (F[m] * F[m]);
    }
    if ((rc = check_hip(P, hipMemcpy(P->deconv.p, tab.data(), tab.size() * sizeof(double),
                                     hipMemcpyHostToDevice), "copy table")))
        return fail(rc);
    P->kb.zeta = r.zeta;
    P->kb.c2 = exp(-2.0 * r.zeta);
    P->kb.inv_den = 1.0 / (-expm1(-2.0 * r.zeta));
    P->kb.edge = 2.0 * r.zeta * exp(-r.zeta) * P->kb.inv_den;
    // FFT plans: 3 transforms of n^3 (real) <-> n^2 (n/2+1) (complex)
    // (one work area for both, which the pruned transforms use too)
    int dims[3] = {P->n, P->n, P->n};
    size_t wsf = 0, wsi = 0;
    if (hipfftCreate(&P->fft_fwd) != HIPFFT_SUCCESS || hipfftCreate(&P->fft_inv) != HIPFFT_SUCCESS ||
        hipfftSetAutoAllocation(P->fft_fwd, 0) != HIPFFT_SUCCESS ||
        hipfftSetAutoAllocation(P->fft_inv, 0) != HIPFFT_SUCCESS)
        return fail(set_error(P, BS_EDEVICE, "hipfftCreate failed"));
    hipfftType tf = P->fp32 ? HIPFFT_R2C : HIPFFT_D2Z, ti = P->fp32 ? HIPFFT_C2R : HIPFFT_Z2D;
    if (hipfftMakePlanMany(P->fft_fwd, 3, dims, nullptr, 1, (int)n3, nullptr, 1, (int)nc, tf, 3,
                           &wsf) != HIPFFT_SUCCESS ||
        hipfftMakePlanMany(P->fft_inv, 3, dims, nullptr, 1, (int)nc, nullptr, 1, (int)n3, ti, 3,
                           &wsi) != HIPFFT_SUCCESS)
        return fail(set_error(P, BS_EDEVICE, "hipfftMakePlanMany failed"));
    if (hipfftSetStream(P->fft_fwd, P->stream) != HIPFFT_SUCCESS ||
        hipfftSetStream(P->fft_inv, P->stream) != HIPFFT_SUCCESS)
        return fail(set_error(P, BS_EDEVICE, "hipfftSetStream failed"));
    P->pruned = runs_pruned(*p, r);
    const size_t cs = 2 * P->real_size, K1 = r.K + 1, NY = 2 * r.K + 1;
    const size_t wsB = P->pruned ? 3 * NY * n * K1 * cs : 0;
    if ((rc = ensure<char>(P, P->fftwork, std::max({wsf, wsi, wsB})))) return fail(rc);
    if ((wsf && hipfftSetWorkArea(P->fft_fwd, P->fftwork.p) != HIPFFT_SUCCESS) ||
        (wsi && hipfftSetWorkArea(P->fft_inv, P->fftwork.p) != HIPFFT_SUCCESS))
        return fail(set_error(P, BS_EDEVICE, "hipfftSetWorkArea failed"));
    // pruned transforms: twiddles exp(-+2 pi i k / n), k < n, from float64
    if (P->pruned) {
        P->fft_ops = pruned_ops(P->n, P->fp32);
        P->fft_kz = pruned_z_batch(P->n, cs);
        // (A, 3 n^2 (K + 1) values, K + 1 <= n / 2, fits the spectrum's 3 n^2 (n / 2 + 1))
        if ((rc = ensure<char>(P, P->fft_tw, 2 * n * cs))) return fail(rc);
        // [n] exp(-2 pi i k / n), then [n] exp(+2 pi i k / n)
        std::vector<double> tw(4 * n);
        for (size_t k = 0; k < n; k++) {
            const double ang = 2.0 * kPi * (double)k / (double)n;
            const double c = cos(ang), sn = sin(ang);
            tw[2 * k] = c; tw[2 * k + 1] = -sn;
            tw[2 * n + 2 * k] = c; tw[2 * n + 2 * k + 1] = sn;
        }
        if (P->fp32) {
            std::vector<float> tf(tw.begin(), tw.end());
            rc = check_hip(P, hipMemcpy(P->fft_tw.p, tf.data(), tf.size() * 4,
                                        hipMemcpyHostToDevice), "copy twiddles");
        } else {
            rc = check_hip(P, hipMemcpy(P->fft_tw.p, tw.data(), tw.size() * 8,
                                        hipMemcpyHostToDevice), "copy twiddles");
        }
        if (rc) return fail(rc);
    }
    *out = P;
    return BS_OK;
}

static void drop_graph(bs_plan_t P);

// order the plan stream after the side stream's pending pair search (the
// calls that read its results or overwrite its inputs on the plan stream)
static int join_side(bs_plan_t P) {
    if (!P->side_pending) return BS_OK;
    int rc = check_hip(P, hipStreamWaitEvent(P->stream, P->ev_ns, 0), "hipStreamWaitEvent");
    if (!rc) P->side_pending = false;
    return rc;
}

int bs_set_periods(bs_plan_t P, int64_t nfil, const int64_t *periods) {
    if (!P) return set_error(nullptr, BS_EINVAL, "null plan");
    drop_graph(P);
    P->have_filaments = false;
    P->nper = 0;
    if (!periods) return BS_OK;
    if (nfil < 1) return set_error(P, BS_EINVAL, "need nfil >= 1");
    std::vector<double> sh(3 * nfil);
    bool any = false;
    for (int64_t k = 0; k < 3 * nfil; k++) {
        if (periods[k] < -(1 << 20) || periods[k] > (1 << 20))
            return set_error(P, BS_EINVAL, "period counts must lie in [-2^20, 2^20]");
        sh[k] = (double)periods[k] * P->prm.L;
        any = any || periods[k] != 0;
    }
    if (!any) return BS_OK;   // all closed
    int rc;
    if ((rc = ensure<double>(P, P->d_shift, 3 * nfil)) ||
        (rc = check_hip(P, hipMemcpyAsync(P->d_shift.p, sh.data(), sizeof(double) * 3 * nfil,
                                          hipMemcpyHostToDevice, P->stream), "copy shifts")) ||
        (rc = check_hip(P, hipStreamSynchronize(P->stream), "sync")))
        return rc;
    P->nper = nfil;
    return BS_OK;
}

// filaments at positions xyz, or xyz + c kstage (a Runge-Kutta stage)
static int set_filaments(bs_plan_t P, int64_t nfil, const int64_t *offsets, const double *xyz,
                         const double *kstage, double c, const double *gamma) {
    if (!P) return set_error(nullptr, BS_EINVAL, "null plan");
    if (nfil < 1 || !offsets || !xyz || !gamma)
        return set_error(P, BS_EINVAL, "need nfil >= 1 and non-null offsets, xyz, gamma");
    if (offsets[0] != 0) return set_error(P, BS_EINVAL, "offsets[0] must be 0");
    int64_t maxn = 0;
    for (int64_t f = 0; f < nfil; f++) {
        int64_t len = offsets[f + 1] - offsets[f];
        if (len < 3) return set_error(P, BS_EINVAL, "every filament needs at least 3 nodes");
        if (P->order == 6 && len < 6)
            return set_error(P, BS_EINVAL, "quintic splines need at least 6 nodes per filament");
        maxn = std::max(maxn, len);
    }
    const int64_t N = offsets[nfil], Nq = N * P->Q;
    if (Nq >= ((int64_t)1 << 31) / 4) return set_error(P, BS_EINVAL, "too many nodes");
    int rc0 = join_side(P);   // the previous search reads what this call rewrites
    if (rc0) return rc0;
    if (P->nper && P->nper != nfil)
        return set_error(P, BS_EINVAL, "periods were set for " + std::to_string(P->nper) +
                                           " filaments, not " + std::to_string(nfil));
    bool same = P->have_filaments && P->nfil == nfil &&
                std::equal(offsets, offsets + nfil + 1, P->off_host.begin());
    int rc;
    int ncx, ncy;
    pair_cells(P, Nq, &ncx, &ncy);
    const int ntiles = P->NT * P->NT * P->NT, nc3 = P->nc * P->nc * P->nc, ncp = ncx * ncy * ncy;
    const size_t rs = P->real_size;
    if (!same) {
        P->have_filaments = false;
        drop_graph(P);   // it holds the buffers that may move here, and their sizes
        // one allocation for all that the filaments' sizes decide: fifty of them took 0.5
        // to 4 ms, now 0.2 to 0.3 with the copies below (first evaluation of 1e5 nodes on
        // 256^3 2.1 to 4.0 ms, now 1.4 to 1.5)
        P->spline_tmp = P->d_piece = P->d_pfirst = DBuf{};   // not in every layout
        std::vector<Part> parts = {
            part<int>(P->d_off, nfil + 1), part<int>(P->d_fil, N), part<double>(P->d_gamma, nfil),
            part<double>(P->d_x, 3 * N), part<double>(P->d_xn, 3 * N), part<double>(P->d_dtau, N),
            part<double>(P->d_D, 3 * N), part<double>(P->d_sdd, 3 * N), part<double>(P->d_ell, N),
            part<double>(P->d_qpos, 3 * Nq), part<double>(P->d_qchg, 3 * Nq),
            part<double>(P->tmp3, 3 * N), part<double>(P->e_D, 3 * N), part<double>(P->e_S, 3 * N),
            part<double>(P->d_vls, 3 * N),
            part<int>(P->sp_key, Nq), part<int>(P->sp_cnt, ntiles + 1),
            part<int>(P->sp_start, ntiles + 1), part<int>(P->sp_fill, ntiles + 1),
            part<int>(P->sp_perm, Nq), part<int4>(P->sp_base, Nq),
            part<char>(P->sp_ker, Nq * 3 * P->prm.w * rs), part<char>(P->sp_q, Nq * 4 * rs),
            part<int>(P->pq_key, Nq), part<int>(P->pq_cnt, ncp + 1), part<int>(P->pq_start, ncp + 1),
            part<int>(P->pq_fill, ncp + 1), part<int>(P->pq_perm, Nq), part<double4>(P->pq_pos, Nq),
            part<char>(P->pq_chg, Nq * 4 * rs),
            part<int>(P->nd_key, N), part<int>(P->nd_cnt, nc3 + 1), part<int>(P->nd_start, nc3 + 1),
            part<int>(P->nd_fill, nc3 + 1), part<int>(P->nd_perm, N), part<double4>(P->nd_rec, N)};
        if (P->order == 4 && maxn > kPcrLds) parts.push_back(part<double>(P->spline_tmp, kPcrScratch * N));
        if (P->order == 6 && maxn > kPcr5Lds) parts.push_back(part<double>(P->spline_tmp, kBlkScratch * N));
        std::vector<int> pfirst(nfil + 1, 0);
        for (int64_t f = 0; f < nfil; f++)
            pfirst[f + 1] = pfirst[f] + (int)ceil_div(offsets[f + 1] - offsets[f], kPiece);
        if (direct_path(P, Nq)) {
            parts.push_back(part<Piece>(P->d_piece, pfirst[nfil]));
            parts.push_back(part<int>(P->d_pfirst, nfil + 1));
        }
        if (P->prm.ns_mode != BS_NS_OFF) {
            size_t mp = (size_t)N * P->ns_max_per_node;
            int ncmax = (int)cbrt(2.0 * (double)N);
            P->ns_ncmax = ncmax < 3 ? 3 : (ncmax > 128 ? 128 : ncmax);
            const size_t nb3 = (size_t)P->ns_ncmax * P->ns_ncmax * P->ns_ncmax;
            parts.insert(parts.end(),
                {part<double>(P->ns_red, 2 * 1024 + 1), part<int>(P->ns_nc, 4),
                 part<int>(P->ns_ckey, N), part<int>(P->ns_ccnt, 2 * nb3 + 1),
                 part<int>(P->ns_cstart, 2 * nb3 + 1), part<int>(P->ns_cfill, 2 * nb3 + 1),
                 part<int>(P->ns_cperm, N), part<int>(P->ns_tkey, N), part<int>(P->ns_tcnt, nb3 + 1),
                 part<int>(P->ns_tstart, nb3 + 1), part<int>(P->ns_tfill, nb3 + 1),
                 part<int>(P->ns_tperm, N), part<double4>(P->ns_segA, N), part<double4>(P->ns_segB, N),
                 part<float4>(P->ns_segM, N), part<float4>(P->ns_segH, N), part<float4>(P->ns_segP, N),
                 part<int2>(P->ns_slots, mp), part<int>(P->ns_cnt, N + 1), part<int>(P->ns_start, N + 1),
                 part<int2>(P->ns_pairs, mp), part<int>(P->ns_pnode, mp), part<double>(P->ns_pout, 3 * mp)});
            if (P->prm.ns_mode == BS_NS_MLP)
                parts.insert(parts.end(),
                    {part<float>(P->ns_X, 8 * mp), part<float>(P->ns_Y, 3 * mp),
                     part<int>(P->ns_fallback, 4), part<int>(P->ns_learn, mp),
                     part<int>(P->ns_fblist, mp), part<double>(P->ns_vs, 1 + 3 * 256)});
        }
        if ((rc = lay_out(P, parts))) return rc;
        // the bin counters start at zero; afterwards each call's per-bin
        // sort clears them for the next
        const size_t nb_t = sizeof(int) * (ntiles + 1), nb_c = sizeof(int) * (nc3 + 1),
                     nb_p = sizeof(int) * (ncp + 1);
        if ((rc = check_hip(P, hipMemsetAsync(P->sp_cnt.p, 0, nb_t, P->stream), "memset")) ||
            (rc = check_hip(P, hipMemsetAsync(P->sp_fill.p, 0, nb_t, P->stream), "memset")) ||
            (rc = check_hip(P, hipMemsetAsync(P->pq_cnt.p, 0, nb_p, P->stream), "memset")) ||
            (rc = check_hip(P, hipMemsetAsync(P->pq_fill.p, 0, nb_p, P->stream), "memset")) ||
            (rc = check_hip(P, hipMemsetAsync(P->nd_cnt.p, 0, nb_c, P->stream), "memset")) ||
            (rc = check_hip(P, hipMemsetAsync(P->nd_fill.p, 0, nb_c, P->stream), "memset")) ||
            (P->ns_fallback.p &&
             (rc = check_hip(P, hipMemsetAsync(P->ns_fallback.p, 0, P->ns_fallback.bytes,
                                               P->stream), "memset"))))
            return rc;
        std::vector<int> off32(nfil + 1), fil32(N);
        if (direct_path(P, Nq) &&
            (rc = check_hip(P, hipMemcpyAsync(P->d_pfirst.p, pfirst.data(), sizeof(int) * (nfil + 1),
                                              hipMemcpyHostToDevice, P->stream), "copy pieces")))
            return rc;
        for (int64_t f = 0; f <= nfil; f++) off32[f] = (int)offsets[f];
        for (int64_t f = 0; f < nfil; f++)
            for (int64_t j = offsets[f]; j < offsets[f + 1]; j++) fil32[j] = (int)f;
        if ((rc = check_hip(P, hipMemcpyAsync(P->d_off.p, off32.data(), sizeof(int) * (nfil + 1),
                                              hipMemcpyHostToDevice, P->stream), "copy offsets")) ||
            (rc = check_hip(P, hipMemcpyAsync(P->d_fil.p, fil32.data(), sizeof(int) * N,
                                              hipMemcpyHostToDevice, P->stream), "copy fil")))
            return rc;
        // the host vectors die at return: wait for the copies
        if ((rc = check_hip(P, hipStreamSynchronize(P->stream), "sync"))) return rc;
        P->off_host.assign(offsets, offsets + nfil + 1);
        P->nfil = nfil;
        P->ncx = ncx;
        P->ncy = ncy;
        P->direct = direct_path(P, Nq);
        P->npiece = (int)pfirst[nfil];
        P->N = N;
        P->Nq = Nq;
        P->max_fil_nodes = maxn;
    }
    stage_begin(P, 0);
    launch_filaments(P, xyz, kstage, c, gamma);   // also takes the plan's copies of xyz and gamma
    stage_end(P, 0);
    if (P->prm.ns_mode != BS_NS_OFF) {
        // the pair search needs only the geometry: it runs on the side stream,
        // beside the binning, and the velocity's short-range and
        // near-singular terms follow it there (per-stage timing keeps it on
        // the plan's stream)
        const bool side = !P->prof;
        if (side &&
            ((rc = check_hip(P, hipEventRecord(P->ev_fork, P->stream), "hipEventRecord")) ||
             (rc = check_hip(P, hipStreamWaitEvent(P->side, P->ev_fork, 0), "hipStreamWaitEvent"))))
            return rc;
        const hipStream_t plan_stream = P->stream;
        if (side) P->stream = P->side;
        stage_begin(P, 10);
        ns_build_pairs(P);
        stage_end(P, 10);
        P->stream = plan_stream;
        if (side) {
            if ((rc = check_hip(P, hipEventRecord(P->ev_ns, P->side), "hipEventRecord"))) return rc;
            P->side_pending = true;
        }
    }
    if (!P->direct) {
        stage_begin(P, 1);
        build_bins(P);
        stage_end(P, 1);
    }
    if ((rc = launch_status(P, "geometry kernels"))) return rc;
    P->have_filaments = true;
    stage_collect(P);
    return BS_OK;
}

int bs_set_filaments(bs_plan_t P, int64_t nfil, const int64_t *offsets, const double *xyz,
                     const double *gamma) {
    return set_filaments(P, nfil, offsets, xyz, nullptr, 0.0, gamma);
}

// out += near-singular correction; base: the velocity terms formed so far at
// the nodes (the learned path's velocity scale is their rms)
static int launch_ns(bs_plan_t P, double *out, const double *base) {
    if (P->prm.ns_mode == BS_NS_ADAPTIVE) {
        launch_ns_adaptive(P, out);
        return BS_OK;
    }
    if (P->prm.ns_mode == BS_NS_MAPPED) {
        launch_ns_mapped(P, out);
        return BS_OK;
    }
    if (!P->mlp) return set_error(P, BS_ESTATE, "BS_NS_MLP plan without bs_set_mlp");
    launch_ns_mlp(P, out, base);
    return BS_OK;
}

// out = base + long-range term (base NULL: out += long-range term); with
// join set, the interpolation waits for that event first; spread: whether the
// grid still has to be written
static int long_range(bs_plan_t P, int psi, const double *base, double *out,
                      hipEvent_t join = nullptr, bool spread = true) {
    int rc;
    if (spread) {
        stage_begin(P, 3);
        launch_spread(P);
        stage_end(P, 3);
    }
    if (P->pruned) {
        stage_begin(P, 4);
        pruned_forward(P);
        stage_end(P, 4);
        stage_begin(P, 5);
        pruned_spectral_op(P, psi);
        stage_end(P, 5);
        stage_begin(P, 6);
        pruned_inverse(P);
        stage_end(P, 6);
    } else {
        stage_begin(P, 4);
        if ((rc = fft_forward(P))) return rc;
        stage_end(P, 4);
        stage_begin(P, 5);
        launch_spectral(P, psi);
        stage_end(P, 5);
        stage_begin(P, 6);
        if ((rc = fft_inverse(P))) return rc;
        stage_end(P, 6);
    }
    if (join && (rc = check_hip(P, hipStreamWaitEvent(P->stream, join, 0), "hipStreamWaitEvent")))
        return rc;
    stage_begin(P, 7);
    launch_interp(P, base, out);
    stage_end(P, 7);
    return launch_status(P, "long-range kernels");
}

int bs_velocity(bs_plan_t P, double *v_out) {
    if (!P) return set_error(nullptr, BS_EINVAL, "null plan");
    if (!P->have_filaments) return set_error(P, BS_ESTATE, "bs_set_filaments not called");
    if (!v_out) return set_error(P, BS_EINVAL, "null output");
    if (P->prm.ns_mode == BS_NS_MLP && !P->mlp)
        return set_error(P, BS_ESTATE, "BS_NS_MLP plan without bs_set_mlp");
    // local - self was formed by set_filaments (d_vls).  The short-range sum
    // and the near-singular correction run on the side stream into
    // tmp3 = (local - self) + short (+ near-singular), concurrently with the
    // spread and the transforms on the plan stream.  Without the correction
    // the interpolation waits for them and writes v = tmp3 + long-range;
    // with it (the side stream's longer chain) the interpolation writes the
    // long-range term alone and tmp3 is added once the side work is in, so
    // that the correction's integrals can run beside the interpolation (the
    // same sum, bitwise).  With per-stage timing on, everything stays on the
    // plan stream, so that each stage's events bracket its own kernels only.
    double *t3 = (double *)P->tmp3.p;
    // Small inputs without the correction need no second stream: the pair sums
    // run in the spread's launch.
    const bool side = !P->prof;
    int rc;
    if (side && P->direct && P->prm.ns_mode == BS_NS_OFF) {
        launch_spread_pairs(P, (const double *)P->d_vls.p, t3);
        if ((rc = long_range(P, 0, t3, v_out, nullptr, false))) return rc;
        return launch_status(P, "velocity kernels");
    }
    if (!side && (rc = join_side(P))) return rc;
    if (side &&
        ((rc = check_hip(P, hipEventRecord(P->ev_fork, P->stream), "hipEventRecord")) ||
         (rc = check_hip(P, hipStreamWaitEvent(P->side, P->ev_fork, 0), "hipStreamWaitEvent"))))
        return rc;
    const hipStream_t plan_stream = P->stream;
    if (side) P->stream = P->side;   // launches below go to the side stream
    rc = BS_OK;
    stage_begin(P, 8);
    launch_pairs(P, 0, (const double *)P->d_vls.p, t3, false);
    stage_end(P, 8);
    if (P->prm.ns_mode != BS_NS_OFF) {
        stage_begin(P, 9);
        rc = launch_ns(P, t3, t3);   // t3 = local - self + short so far
        stage_end(P, 9);
    }
    P->stream = plan_stream;
    const hipError_t ej = side ? hipEventRecord(P->ev_join, P->side) : hipSuccess;
    if (rc || (rc = check_hip(P, ej, "hipEventRecord"))) return rc;
    if (side && P->prm.ns_mode != BS_NS_OFF) {
        fill_f64(P, v_out, 3 * (size_t)P->N, 0.0);
        if ((rc = long_range(P, 0, nullptr, v_out))) return rc;
        if ((rc = check_hip(P, hipStreamWaitEvent(P->stream, P->ev_join, 0), "hipStreamWaitEvent")))
            return rc;
        add_f64(P, v_out, t3, 3 * (size_t)P->N);
    } else if ((rc = long_range(P, 0, t3, v_out, side ? P->ev_join : nullptr))) {
        return rc;
    }
    P->side_pending = false;   // the plan stream now waits for all side work
    if ((rc = launch_status(P, "pair kernel"))) return rc;
    stage_collect(P);
    return BS_OK;
}

int bs_velocity_terms(bs_plan_t P, double *v_local, double *v_short, double *v_long,
                      double *v_self, double *v_ns) {
    if (!P) return set_error(nullptr, BS_EINVAL, "null plan");
    if (!P->have_filaments) return set_error(P, BS_ESTATE, "bs_set_filaments not called");
    int rc;
    if ((rc = join_side(P))) return rc;
    const size_t n3 = 3 * (size_t)P->N;
    if (v_local) launch_local_self(P, LS_VLOCAL | LS_ASSIGN, 1.0, v_local);
    if (v_self) launch_local_self(P, LS_VSELF | LS_ASSIGN, 1.0, v_self);
    if (v_long) {
        fill_f64(P, v_long, n3, 0.0);
        if ((rc = long_range(P, 0, nullptr, v_long))) return rc;
    }
    if (v_short) {
        fill_f64(P, v_short, n3, 0.0);
        launch_pairs(P, 0, nullptr, v_short, true);
    }
    if (v_ns) {
        fill_f64(P, v_ns, n3, 0.0);
        if (P->prm.ns_mode != BS_NS_OFF &&
            (rc = launch_ns(P, v_ns, (const double *)P->d_vls.p)))
            return rc;
    }
    return launch_status(P, "velocity terms");
}

int bs_energy(bs_plan_t P, double *E_out, double *psi_out) {
    if (!P) return set_error(nullptr, BS_EINVAL, "null plan");
    if (!P->have_filaments) return set_error(P, BS_ESTATE, "bs_set_filaments not called");
    int rc0 = join_side(P);
    if (rc0) return rc0;
    double *psi = psi_out ? psi_out : (double *)P->tmp3.p;
    launch_local_self(P, LS_VLOCAL | LS_VSELF | LS_PSI | LS_ASSIGN, 1.0, psi);
    int rc = long_range(P, 1, nullptr, psi);
    if (rc) return rc;
    launch_pairs(P, 1, nullptr, psi, true);
    if (!P->h_energy && (rc = check_hip(P, hipHostMalloc((void **)&P->h_energy, sizeof(double),
                                                         hipHostMallocMapped), "hipHostMalloc")))
        return rc;
    launch_energy(P, psi, (double *)P->red_tmp.p, P->h_energy);
    if ((rc = launch_status(P, "energy kernels"))) return rc;
    if ((rc = check_hip(P, hipStreamSynchronize(P->stream), "sync"))) return rc;
    if (E_out) *E_out = *(volatile double *)P->h_energy;
    return BS_OK;
}

int bs_vorticity_modes(bs_plan_t P, double *out) {
    if (!P) return set_error(nullptr, BS_EINVAL, "null plan");
    if (!P->have_filaments) return set_error(P, BS_ESTATE, "bs_set_filaments not called");
    if (!out) return set_error(P, BS_EINVAL, "null output");
    launch_spread(P);
    int rc = fft_forward(P);
    if (rc) return rc;
    launch_modes(P, out);
    return launch_status(P, "mode extraction");
}

int bs_geometry(bs_plan_t P, double *qpos, double *qcharge, double *sdot, double *sddot,
                double *ell) {
    if (!P) return set_error(nullptr, BS_EINVAL, "null plan");
    if (!P->have_filaments) return set_error(P, BS_ESTATE, "bs_set_filaments not called");
    const size_t N = P->N, Nq = P->Nq;
    struct { void *dst; const void *src; size_t bytes; } cp[5] = {
        {qpos, P->d_qpos.p, 3 * Nq * 8}, {qcharge, P->d_qchg.p, 3 * Nq * 8},
        {sdot, P->d_D.p, 3 * N * 8}, {sddot, P->d_sdd.p, 3 * N * 8}, {ell, P->d_ell.p, N * 8}};
    for (auto &c : cp) {
        if (!c.dst) continue;
        int rc = check_hip(P, hipMemcpyAsync(c.dst, c.src, c.bytes, hipMemcpyDeviceToDevice,
                                             P->stream), "copy geometry");
        if (rc) return rc;
    }
    return BS_OK;
}

int bs_status(bs_plan_t P) {
    if (!P) return set_error(nullptr, BS_EINVAL, "null plan");
    int st = 0, rc;
    if ((rc = join_side(P))) return rc;
    if ((rc = check_hip(P, hipMemcpyAsync(&st, P->d_status.p, sizeof(int), hipMemcpyDeviceToHost,
                                          P->stream), "read status")) ||
        (rc = check_hip(P, hipStreamSynchronize(P->stream), "sync")))
        return rc;
    if (st) {
        (void)hipMemsetAsync(P->d_status.p, 0, sizeof(int), P->stream);
        (void)hipStreamSynchronize(P->stream);
        return set_error(P, BS_EINVAL, (st & 1) ? "non-finite node position or zero-length segment"
                                                : "more than 64 near-singular segments at a node");
    }
    return BS_OK;
}

// classical RK4 update of [N][3] float64 positions
__global__ void k_rk4_final(size_t n, double *__restrict__ x, const double *__restrict__ k1,
                            const double *__restrict__ k2, const double *__restrict__ k3,
                            const double *__restrict__ k4, double dt) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] += dt / 6.0 * (k1[i] + 2.0 * k2[i] + 2.0 * k3[i] + k4[i]);
}

int bs_rk4_step(bs_plan_t P, int64_t nfil, const int64_t *offsets, double *xyz,
                const double *gamma, double dt) {
    if (!P) return set_error(nullptr, BS_EINVAL, "null plan");
    if (!offsets || nfil < 1 || !xyz || !gamma || !std::isfinite(dt))
        return set_error(P, BS_EINVAL, "bad arguments");
    const int64_t N = offsets[nfil];
    const size_t n3 = 3 * (size_t)N;
    int rc;
    if ((rc = ensure<double>(P, P->rk_k, 4 * n3))) return rc;
    double *k = (double *)P->rk_k.p;
    const dim3 g((unsigned)((n3 + 255) / 256)), b(256);
    const double c[4] = {0.0, 0.5 * dt, 0.5 * dt, dt};
    for (int st = 0; st < 4; st++) {
        // the stage's positions x + c k are formed as they are read
        if ((rc = set_filaments(P, nfil, offsets, xyz, st ? k + (st - 1) * n3 : nullptr, c[st],
                                gamma)))
            return rc;
        if ((rc = bs_velocity(P, k + st * n3))) return rc;
    }
    hipLaunchKernelGGL(k_rk4_final, g, b, 0, P->stream, n3, xyz, k, k + n3, k + 2 * n3, k + 3 * n3, dt);
    return launch_status(P, "rk4 kernels");
}

// ---------------------------------------------------------- graph replay
static void drop_graph(bs_plan_t P) {
    if (P->gexec) {
        (void)hipStreamSynchronize(P->stream);   // a replay may still run
        (void)hipGraphExecDestroy(P->gexec);
    }
    if (P->graph) (void)hipGraphDestroy(P->graph);
    P->gexec = nullptr;
    P->graph = nullptr;
}

int bs_set_graph(bs_plan_t P, int enable) {
    if (!P) return set_error(nullptr, BS_EINVAL, "null plan");
    if (enable && P->stream == nullptr)
        return set_error(P, BS_EINVAL, "graph replay needs a non-null plan stream");
    if (!enable) drop_graph(P);
    P->use_graph = enable != 0;
    return BS_OK;
}

int bs_step(bs_plan_t P, int64_t nfil, const int64_t *offsets, const double *xyz,
            const double *gamma, double *v_out) {
    if (!P) return set_error(nullptr, BS_EINVAL, "null plan");
    const bool same = P->gexec && P->have_filaments && P->g_xyz == xyz && P->g_gamma == gamma &&
                      P->g_v == v_out && P->g_fp32 == mlp_fp32(P->mlp) && P->nfil == nfil && offsets &&
                      std::equal(offsets, offsets + nfil + 1, P->off_host.begin());
    if (P->use_graph && !P->prof && same) {
        // a pair search of an earlier bs_set_filaments may still read, on the
        // side stream, what the replay rewrites
        int rc = join_side(P);
        return rc ? rc : check_hip(P, hipGraphLaunch(P->gexec, P->stream), "hipGraphLaunch");
    }
    // eager step (also sizes every buffer and uploads the filament structure)
    int rc = bs_set_filaments(P, nfil, offsets, xyz, gamma);
    if (!rc) rc = bs_velocity(P, v_out);
    if (rc || !P->use_graph || P->prof) return rc;
    // capture the same sequence; with unchanged offsets it has no host work
    drop_graph(P);
    hipError_t e = hipStreamBeginCapture(P->stream, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) { P->use_graph = false; return BS_OK; }
    int rc1 = bs_set_filaments(P, nfil, offsets, xyz, gamma);
    int rc2 = rc1 ? rc1 : bs_velocity(P, v_out);
    hipGraph_t g = nullptr;
    e = hipStreamEndCapture(P->stream, &g);
    if (rc2 || e != hipSuccess || !g) {
        if (g) (void)hipGraphDestroy(g);
        (void)hipGetLastError();
        P->use_graph = false;        // fall back to eager steps
        return BS_OK;
    }
    if (hipGraphInstantiate(&P->gexec, g, nullptr, nullptr, 0) != hipSuccess) {
        (void)hipGraphDestroy(g);
        P->gexec = nullptr;
        P->use_graph = false;
        return BS_OK;
    }
    P->graph = g;
    P->g_xyz = xyz; P->g_gamma = gamma; P->g_v = v_out;
    P->g_fp32 = mlp_fp32(P->mlp);
    return BS_OK;
}

int bs_graph_active(bs_plan_t P) { return P && P->gexec ? 1 : 0; }

int bs_set_mlp(bs_plan_t P, bs_mlp_t mlp, const float *err_table, int nbins) {
    if (!P) return set_error(nullptr, BS_EINVAL, "null plan");
    int want = 0;
    bs_ns_error_bins(nullptr, nullptr, &want);
    if (P->prm.ns_mode != BS_NS_MLP) return set_error(P, BS_ESTATE, "plan is not BS_NS_MLP");
    if (!mlp || !err_table || nbins != want)
        return set_error(P, BS_EINVAL, "need a network and an error table of bs_ns_error_bins bins");
    for (int b = 0; b < nbins; b++)
        if (!(err_table[b] >= 0.0f)) return set_error(P, BS_EINVAL, "error table entry < 0 or NaN");
    // a recorded bs_step graph holds the previous network's buffers and the
    // previous table in its kernel arguments
    drop_graph(P);
    P->mlp = mlp;
    for (int b = 0; b < nbins; b++) P->ns_err[b] = err_table[b];
    return BS_OK;
}

int bs_ns_counts(bs_plan_t P, int64_t *npairs, int64_t *nfallback) {
    if (!P) return set_error(nullptr, BS_EINVAL, "null plan");
    int np = 0, nf = 0, rc;
    if ((rc = join_side(P))) return rc;
    if (P->prm.ns_mode != BS_NS_OFF && P->have_filaments) {
        if ((rc = check_hip(P, hipMemcpyAsync(&np, (int *)P->ns_start.p + P->N, sizeof(int),
                                              hipMemcpyDeviceToHost, P->stream), "read count")))
            return rc;
        int c4[4] = {0, 0, 0, 0};
        if (P->prm.ns_mode == BS_NS_MLP && P->ns_fallback.p &&
            (rc = check_hip(P, hipMemcpyAsync(c4, P->ns_fallback.p, sizeof(c4),
                                              hipMemcpyDeviceToHost, P->stream), "read count")))
            return rc;
        if ((rc = check_hip(P, hipStreamSynchronize(P->stream), "sync"))) return rc;
        // the gate closed: every pair went to the plain integrator
        if (P->prm.ns_mode == BS_NS_MLP) nf = c4[2] ? c4[1] : (c4[3] ? np : 0);
    }
    if (npairs) *npairs = np;
    if (nfallback) *nfallback = nf;
    return BS_OK;
}

int bs_get_params(bs_plan_t P, bs_params *resolved) {
    if (!P || !resolved) return set_error(P, BS_EINVAL, "null argument");
    *resolved = P->prm;
    return BS_OK;
}

int bs_plan_transforms(bs_plan_t P) {
    if (!P) return set_error(nullptr, BS_EINVAL, "null plan");
    return P->pruned ? BS_FFT_PRUNED : BS_FFT_LIBRARY;
}

int bs_destroy(bs_plan_t P) {
    if (!P) return BS_OK;
    (void)hipStreamSynchronize(P->stream);
    if (P->side) {
        (void)hipStreamSynchronize(P->side);
        (void)hipStreamDestroy(P->side);
    }
    if (P->h_energy) (void)hipHostFree(P->h_energy);
    if (P->ev_fork) (void)hipEventDestroy(P->ev_fork);
    if (P->ev_join) (void)hipEventDestroy(P->ev_join);
    if (P->ev_ns) (void)hipEventDestroy(P->ev_ns);
    drop_graph(P);
    for (int s = 0; s < BS_NSTAGES; s++) {
        if (P->ev_beg[s]) (void)hipEventDestroy(P->ev_beg[s]);
        if (P->ev_end[s]) (void)hipEventDestroy(P->ev_end[s]);
    }
    if (P->fft_fwd) hipfftDestroy(P->fft_fwd);
    if (P->fft_inv) hipfftDestroy(P->fft_inv);
    DBuf *all[] = {&P->grid, &P->spec, &P->deconv, &P->fftwork, &P->fft_tw, &P->d_shift, &P->d_status,
                   &P->scan_tmp, &P->red_tmp, &P->points, &P->rk_k};
    for (DBuf *b : all) release(*b);
    delete P;
    return BS_OK;
}

}  // extern "C"
