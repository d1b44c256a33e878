// Float64 short-range sums: the pieces that the pair kernels share.
#pragma once
#include "bs_internal.h"
#include "bs_device.h"
#include "erfcx_fit.h"

namespace bs {

// g_sr(x) = erfc(x) + (2/sqrt(pi)) x exp(-x^2) = exp(-x^2) (erfcx(x) +
// (2/sqrt(pi)) x): one exponential, with erfcx = P(Z) / (4 + x),
// Z = (4 - x) / (4 + x), from its fitted polynomial (float64: relative
// error 3e-15 for x = alpha r below the beta of every tolerance in Table 1,
// 7e-14 where the term is below 1e-15 of its value at r = 0; float32:
// 4e-7, below the float32 rounding of exp(-x^2) for x near beta)
// float64: the polynomials' coefficients come as a kernel argument, so that they
// sit in scalar registers: as literals they took 130 moves per target and 50
// vector registers.  exp(y), y <= 0: y = n ln 2 + r, |r| <= ln 2 / 2, Taylor
// polynomial of degree 13 (remainder below 5e-18).
constexpr int kExpDeg = 13;
struct ShortFit {
    double p[kErfcxDeg + 1];
    double e[kExpDeg + 1];   // 1 / k!
    double log2e, ln2_hi, ln2_lo;
};
// scalars of the cell list, formed once on the host
struct PairGeom {
    double L, invL, rc2, rm, alpha;
    double fx, fy;          // cells per length along x and along y, z
    float ry, ratio;        // r_c in y cells with the margin, x cells per y cell
    int ncx, ncy;
};
__device__ __forceinline__ double g_short64(double x, const ShortFit &F) {
    constexpr double two_over_sqrtpi = 1.12837916709551257389615890312154517;
    const double inv = rcp_nr(kErfcxShift + x);
    const double z = (kErfcxShift - x) * inv;
    double p = F.p[kErfcxDeg];
#pragma unroll
    for (int k = kErfcxDeg - 1; k >= 0; k--)
        p = fma(p, z, F.p[k]);
    const double y = -x * x, n = rint(y * F.log2e);
    const double r = fma(-n, F.ln2_lo, fma(-n, F.ln2_hi, y));
    double e = F.e[kExpDeg];
#pragma unroll
    for (int k = kExpDeg - 1; k >= 0; k--) e = fma(e, r, k < 2 ? 1.0 : (k == 2 ? 0.5 : F.e[k]));
    e = ldexp(e, (int)n);
    return e * fma(p, inv, two_over_sqrtpi * x);
}

// rows of the cell list are found in float32 with this margin, in cells
constexpr float kRowMargin = 1e-4f;
ShortFit short_fit();
PairGeom pair_geom(bs_plan_t p);

// accepted candidates queued per wavefront (a ring of two steps' worth)
constexpr int kQueue = 128;

// A wavefront's queue of candidates within r_c (ring, positions [head, tail),
// wavefront-uniform) and the sums of their terms, run 64 at a time.
template <bool PSI>
struct PairQueue {
    double *qx, *qy, *qz;
    int *qp;
    const double4 *chg;
    double alpha;
    const ShortFit &fit;
    int head = 0, tail = 0;
    double acc0 = 0, acc1 = 0, acc2 = 0;

    __device__ __forceinline__ PairQueue(double (*q)[kQueue], int *qpid, const double4 *c, double a,
                                         const ShortFit &f)
        : qx(q[0]), qy(q[1]), qz(q[2]), qp(qpid), chg(c), alpha(a), fit(f) {}

    // the terms of the first n <= 64 queued ones, one per lane
    __device__ __forceinline__ void drain(int n) {
        const int lane = threadIdx.x & 63;
        if (lane < n) {
            const int sl = (head + lane) & (kQueue - 1);
            const double4 q = chg[qp[sl]];
            const double fx = qx[sl], fy = qy[sl], fz = qz[sl];
            const double r2 = fx * fx + fy * fy + fz * fz;
            if (PSI) {
                // (erfc and quotients to rounding: the fitted polynomial's error, 3e-15,
                // would be the streamfunction's, to which every term adds alike)
                const double rr = sqrt(r2), f = erfc(alpha * rr) / rr;
                acc0 += f * q.x; acc1 += f * q.y; acc2 += f * q.z;
            } else {
                const double ir = rsqrt_nr(r2);
                const double f = g_short64(alpha * (r2 * ir), fit) * (ir * ir * ir);
                acc0 += f * (fy * q.z - fz * q.y);
                acc1 += f * (fz * q.x - fx * q.z);
                acc2 += f * (fx * q.y - fy * q.x);
            }
        }
        head += n;
    }
    // one step of 64 candidates (converged): the accepted ones in lane order
    __device__ __forceinline__ void push(bool ok, double rx, double ry, double rz, int p) {
        const unsigned long long m = __ballot(ok);
        if (ok) {
            const int sl = (tail + bits_below(m)) & (kQueue - 1);
            qx[sl] = rx; qy[sl] = ry; qz[sl] = rz; qp[sl] = p;
        }
        tail += __popcll(m);
        if (tail - head >= 64) {
            wave_lds_sync();
            drain(64);
            wave_lds_sync();   // slots read before the next step writes them
        }
    }
    // the rest of the queue; the sums end in lane 63
    __device__ __forceinline__ void finish() {
        wave_lds_sync();
        drain(tail - head);
        acc0 = wave_total63(acc0);
        acc1 = wave_total63(acc1);
        acc2 = wave_total63(acc2);
    }
};

// candidates per chunk (start marks in LDS, one byte each)
constexpr int kMarkCap = 1024;
struct PairLds {
    __attribute__((aligned(16))) unsigned char mark[4][kMarkCap];
    double red[4][3];
    double qbuf[4][3][kQueue];
    int qpid[4][kQueue];
    int delta[4][64];
};

// The candidates of one target, given as ranges of points, one per lane: they are
// enumerated as one flattened range, with a mark at each range's start, so
// that a candidate's range is the number of marks up to it (one ballot and a
// bit count per 64 candidates) and every lane is busy whatever the ranges
// hold.  WPN wavefronts share a target: the steps of 64 are dealt round-robin.
template <bool PSI, int WPN>
struct PairScan {
    PairQueue<PSI> Q;
    unsigned char *mark;
    int *delta;
    const double4 *pos;
    double w0, w1, w2, od, pd, L, invL, rc2;
    bool inside;   // the sphere of radius r_c lies inside the box
    int part, st = 0;

    __device__ __forceinline__ PairScan(PairLds &lds, const double4 &tg, const PairGeom &G,
                                        const double4 *spos, const double4 *schg,
                                        const ShortFit &fit)
        : Q(lds.qbuf[threadIdx.x >> 6], lds.qpid[threadIdx.x >> 6], schg, G.alpha, fit),
          mark(lds.mark[threadIdx.x >> 6]), delta(lds.delta[threadIdx.x >> 6]), pos(spos) {
        part = WPN == 1 ? 0 : threadIdx.x >> 6;
        // wrapped position; node and its predecessor
        w0 = tg.x; w1 = tg.y; w2 = tg.z;
        od = (double)__double2loint(tg.w);
        pd = (double)__double2hiint(tg.w);
        L = G.L; invL = G.invL; rc2 = G.rc2;
        const double rm = G.rm;
        inside = w0 >= rm && w1 >= rm && w2 >= rm && w0 + rm < L && w1 + rm < L && w2 + rm < L;
        static_assert(kMarkCap == 64 * 16, "a lane clears 16 marks");
        *(uint4 *)(mark + 16 * (threadIdx.x & 63)) = make_uint4(0, 0, 0, 0);
    }

    // the lane's range: points cs .. cs + cn - 1 (converged)
    __device__ __forceinline__ void ranges(int cs, int cn) {
        const int lane = threadIdx.x & 63;
        const int incl = wave_incl_sum(cn);
        const int total = __builtin_amdgcn_readlane(incl, 63);
        const int excl = incl - cn;
        wave_lds_sync();   // marks cleared, deltas of the ranges before read
        {
            // the ranges in order: point = candidate + delta[range]
            const unsigned long long m = __ballot(cn > 0);
            if (cn > 0) delta[bits_below(m)] = cs - excl;
        }
        int seen = -1;   // ranges begun before the step, minus one
        for (int c0 = 0; c0 < total; c0 += kMarkCap) {
            const int cend = min(total, c0 + kMarkCap);
            const bool mine = cn > 0 && excl >= c0 && excl < cend;
            if (mine) mark[excl - c0] = 1;
            wave_lds_sync();
            // 64 candidates a step: separation (minimum image), the node's
            // two adjacent segments excluded, those within r_c queued in order
            for (int qb = c0; qb < cend; qb += 64, st++) {
                const int q = qb + lane;
                const bool mk = mark[q - c0] != 0;
                const unsigned long long mm = __ballot(mk);
                const int rg = seen + bits_below(mm) + (mk ? 1 : 0);
                seen += __popcll(mm);
                if (WPN > 1 && (st & (WPN - 1)) != part) continue;
                const bool in = q < cend;
                const int p = in ? q + delta[rg] : 0;
                const double4 sp = pos[p];
                double rx = sp.x - w0, ry = sp.y - w1, rz = sp.z - w2;
                if (!inside) {
                    rx -= L * rint(rx * invL);
                    ry -= L * rint(ry * invL);
                    rz -= L * rint(rz * invL);
                }
                const double r2 = rx * rx + ry * ry + rz * rz;
                Q.push(in && sp.w != od && sp.w != pd && r2 < rc2 && r2 != 0.0, rx, ry, rz, p);
            }
            wave_lds_sync();   // marks read before they are cleared
            if (mine) mark[excl - c0] = 0;
        }
    }

    // out = base + the target's sum (wavefront 0's lane 63 writes)
    __device__ __forceinline__ void store(PairLds &lds, const double *__restrict__ base,
                                          double *__restrict__ out) {
        const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, o = (int)od;
        Q.finish();
        double acc0 = Q.acc0, acc1 = Q.acc1, acc2 = Q.acc2;
        if (WPN > 1) {
            if (lane == 63) {
                lds.red[wave][0] = acc0; lds.red[wave][1] = acc1; lds.red[wave][2] = acc2;
            }
            __syncthreads();
            if (wave != 0) return;
            acc0 = (lds.red[0][0] + lds.red[1][0]) + (lds.red[2][0] + lds.red[3][0]);
            acc1 = (lds.red[0][1] + lds.red[1][1]) + (lds.red[2][1] + lds.red[3][1]);
            acc2 = (lds.red[0][2] + lds.red[1][2]) + (lds.red[2][2] + lds.red[3][2]);
        }
        if (lane == 63) {
            const double inv4pi = 1.0 / (4.0 * kPi);
            const double *b = base ? base : out;
            const double b0 = b[3 * o], b1 = b[3 * o + 1], b2 = b[3 * o + 2];
            out[3 * o] = b0 + acc0 * inv4pi;
            out[3 * o + 1] = b1 + acc1 * inv4pi;
            out[3 * o + 2] = b2 + acc2 * inv4pi;
        }
    }
};

}  // namespace bs
