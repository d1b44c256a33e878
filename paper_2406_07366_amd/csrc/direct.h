// The direct path of small float64 inputs: no counting sorts; the points and
// targets stay in index order, the spread's tiles scan every point's stencil
// base, and a target's candidates are the points of the filament pieces whose
// bounding boxes come near it.
#pragma once
#include "bs_internal.h"
#include "bs_device.h"
#include "pairs64.h"

namespace bs {

// filaments of at most this many nodes write the sorted copies' content in
// the per-filament kernel, longer ones through a launch of their own
constexpr int kDirectFil = 128;

// nodes per piece of a filament (the last piece of a filament may be shorter)
constexpr int kPiece = 32;
// bounding box of a piece's quadrature points (unwrapped): centre and half
// extents with a margin for their float32 rounding; its points
struct Piece {
    float c[3], e[3];
    int q0, nq;
};
struct PieceList {
    const Piece *p;
    int n;
};
inline PieceList piece_list(bs_plan_t p) { return {(const Piece *)p->d_piece.p, p->npiece}; }

struct DirectOut {
    unsigned *pack;     // stencil base per axis, 10 bits each
    double *ker;        // [Nq][3][w] kernel values
    double4 *q, *spos;  // charges; wrapped position and segment index
    double4 *tgt;       // wrapped position; node and its predecessor
    Piece *piece;
    const int *pfirst;  // first piece of each filament
    double L, inv_h, inv_half;
    KbPhi kb;
    int w, n;
};
inline DirectOut direct_out(bs_plan_t p) {
    DirectOut d;
    d.pack = (unsigned *)p->sp_base.p;
    d.ker = (double *)p->sp_ker.p;
    d.q = (double4 *)p->pq_chg.p;
    d.spos = (double4 *)p->pq_pos.p;
    d.tgt = (double4 *)p->nd_rec.p;
    d.piece = (Piece *)p->d_piece.p;
    d.pfirst = (const int *)p->d_pfirst.p;
    d.L = p->prm.L;
    d.inv_h = p->n / p->prm.L;
    d.inv_half = 2.0 / p->prm.w;
    d.kb = p->kb;
    d.w = p->prm.w;
    d.n = p->n;
    return d;
}

// point q on segment seg at position p[3] with charge c[3]
__device__ __forceinline__ void direct_point(int q, int seg, const double *p, const double *c,
                                             const DirectOut &d) {
    double xw[3], f;
    unsigned pk = 0;
#pragma unroll
    for (int a = 0; a < 3; a++) {
        xw[a] = wrap_box(p[a], d.L);
        pk |= (unsigned)stencil_base(xw[a], d.inv_h, d.w, d.n, &f) << (10 * a);
    }
    d.pack[q] = pk;
    d.spos[q] = make_double4(xw[0], xw[1], xw[2], (double)seg);
    d.q[q] = make_double4(c[0], c[1], c[2], 0.0);
}
// kernel value k of a point's coordinate x
__device__ __forceinline__ double direct_value(double x, int k, const DirectOut &d) {
    double f;
    stencil_base(wrap_box(x, d.L), d.inv_h, d.w, d.n, &f);
    return kb_phi64((k - f) * d.inv_half, d.kb);
}
// node i at x[3], predecessor ip
__device__ __forceinline__ void direct_node(int i, int ip, const double *x, const DirectOut &d) {
    d.tgt[i] = make_double4(wrap_box(x[0], d.L), wrap_box(x[1], d.L), wrap_box(x[2], d.L),
                            __hiloint2double(ip, i));
}

// box of the nq points at pos (unwrapped), by one wavefront; q0: their first index
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {   // lanes without a source keep v
    return __int_as_float(
        __builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float wave_max63(float v) {
    v = fmaxf(v, dpp_f<0x111>(v));
    v = fmaxf(v, dpp_f<0x112>(v));
    v = fmaxf(v, dpp_f<0x114>(v));
    v = fmaxf(v, dpp_f<0x118>(v));
    v = fmaxf(v, dpp_f<0x142>(v));
    v = fmaxf(v, dpp_f<0x143>(v));
    return v;
}
__device__ __forceinline__ void direct_piece(Piece *out, const double *pos, int q0, int nq,
                                             double L) {
    const int lane = threadIdx.x & 63;
    float hi[3] = {-3.0e38f, -3.0e38f, -3.0e38f}, lo[3] = {-3.0e38f, -3.0e38f, -3.0e38f};
    bool finite = true;   // (the maxima pass over NaN)
    for (int t = lane; t < nq; t += 64)
#pragma unroll
        for (int a = 0; a < 3; a++) {
            const float v = (float)pos[3 * t + a];
            finite = finite && fabsf(v) < 1.0e38f;
            hi[a] = fmaxf(hi[a], v);
            lo[a] = fmaxf(lo[a], -v);
        }
    const bool all = __ballot(!finite) == 0;
    Piece P;
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const float h = wave_max63(hi[a]), l = -wave_max63(lo[a]);
        // float32 rounding of the bounds and of the centre, and of the
        // target's offset from it: below 1e-6 of the magnitudes
        P.c[a] = 0.5f * (h + l);
        P.e[a] = 0.5f * (h - l) + 1e-6f * (fabsf(h) + fabsf(l) + (float)L);
        if (!all) {   // its points fold to 0: near every target
            P.c[a] = 0.0f;
            P.e[a] = INFINITY;
        }
    }
    P.q0 = q0;
    P.nq = nq;
    if (lane == 63) *out = P;
}

// Workgroup blk of 256 threads takes target blk (WPN = 4) or targets 4 blk ..
// 4 blk + 3.  64 pieces at a time, one per lane: those whose box comes within
// r_c of the target (nearest image) are its ranges.  Every piece is taken
// when its box or the target is not finite.
template <bool PSI, int WPN>
__device__ __forceinline__ void pairs_direct(int blk, int N, const PairGeom &G, const PieceList &pl,
                                             const double4 *__restrict__ tgt,
                                             const double4 *__restrict__ spos,
                                             const double4 *__restrict__ schg,
                                             const ShortFit &fit, const double *__restrict__ base,
                                             double *__restrict__ out, PairLds &lds) {
    static_assert(WPN == 1 || WPN == 4, "1 or 4 wavefronts per target");
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int t = WPN == 1 ? blk * 4 + wave : blk;
    if (t >= N) return;   // whole wavefronts (WPN = 1) or the whole workgroup
    PairScan<PSI, WPN> P(lds, tgt[t], G, spos, schg, fit);
    const float x[3] = {(float)P.w0, (float)P.w1, (float)P.w2};
    const float Lf = (float)G.L, iLf = (float)G.invL, rc = (float)G.rm;
    for (int p0 = 0; p0 < pl.n; p0 += 64) {
        int cs = 0, cn = 0;
        if (p0 + lane < pl.n) {
            const Piece pc = pl.p[p0 + lane];
            float d2 = 0.0f;
#pragma unroll
            for (int a = 0; a < 3; a++) {
                float d = x[a] - pc.c[a];
                d = fabsf(d - Lf * rintf(d * iLf)) - pc.e[a];
                d = fmaxf(d, 0.0f);
                d2 += d * d;
            }
            if (!(d2 > rc * rc * 1.00001f)) {
                cs = pc.q0;
                cn = pc.nq;
            }
        }
        P.ranges(cs, cn);
    }
    P.store(lds, base, out);
}

}  // namespace bs
