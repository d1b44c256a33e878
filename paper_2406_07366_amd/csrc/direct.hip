// Spread of the direct path (small float64 inputs), alone and in one launch with
// the short-range sums.
//
// A workgroup of four wavefronts per 8^3 tile.  The points are dealt to the
// wavefronts one by one (point i to wavefront i mod 4, so that the run of
// points where a filament crosses the tile is shared evenly); each wavefront
// tests its points' stencil bases against the tile, 64 a step, queues the
// indices of those that reach it, and takes them 32 at a time: their kernel
// values copied to LDS by consecutive lanes, then four candidates per matrix
// instruction as in k_spread.  The partial tiles are summed in wavefront order.
// Bound by latency (point bases, kernel values, instruction chains): on the
// 64^3 ellipses 31 us with the pair sums in the same
// launch, where the sorts took 14, the spread 22 and the pair kernel beside it 24.
#include <algorithm>

#include "direct.h"

namespace bs {

constexpr int kBatch = 32;   // candidates staged at a time
constexpr int kRing = 128;   // queued candidate indices per wavefront
constexpr int kTile = 8;

template <int W>
struct SpreadLds {
    static constexpr int SW = 3 * W + 4, STAGE = 4 * kBatch * SW, RED = 2 * 24 * 64;
    double st[STAGE > RED ? STAGE : RED];
    int soff[4][kBatch];
    unsigned short ring[4][kRing];
};

template <int W>
__device__ __forceinline__ void spread_direct(int tile, int n, int NT, int Nq,
                                              const unsigned *__restrict__ pack,
                                              const double *__restrict__ ker,
                                              const double4 *__restrict__ q,
                                              double *__restrict__ grid, SpreadLds<W> &lds) {
    constexpr int SW = SpreadLds<W>::SW, TT = kTile;
    typedef Mfma4<double>::V V4;
    const int tx = tile % NT, ty = (tile / NT) % NT, tz = tile / (NT * NT);
    const int t0[3] = {tx * TT, ty * TT, tz * TT};
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i16 = lane & 15, k4 = lane >> 4;
    double *st = lds.st + wave * kBatch * SW;
    unsigned short *ring = lds.ring[wave];
    int *soff = lds.soff[wave];
    V4 dacc[2][4];
#pragma unroll
    for (int a = 0; a < 2; a++)
#pragma unroll
        for (int b = 0; b < 4; b++) dacc[a][b] = V4{0.0, 0.0, 0.0, 0.0};
    // per axis, the stencil index of the tile's first cell, in [1 - T, W - 1]
    // when the stencil reaches the tile (the plan keeps n >= W + T)
    auto reach = [&](unsigned pk, int *o) {
        bool act = true;
#pragma unroll
        for (int a = 0; a < 3; a++) {
            int off = t0[a] - (int)((pk >> (10 * a)) & 1023u);
            if (off < 0) off += n;
            o[a] = off < W ? off : off - n;
            act = act && o[a] > -TT;
        }
        return act;
    };
    int head = 0, tail = 0;
    auto batch = [&](int nb) {
        wave_lds_sync();
        // kernel values: word j of candidate c by lane c 3W + j (mod 64)
        constexpr int NL = (kBatch * 3 * W + 63) / 64;
        double v[NL];
#pragma unroll
        for (int k = 0; k < NL; k++) {
            const int i = k * 64 + lane, c = i / (3 * W);
            if (c < nb) v[k] = ker[(size_t)ring[(head + c) & (kRing - 1)] * (3 * W) + (i - c * 3 * W)];
        }
        if (lane < nb) {
            const int p = ring[(head + lane) & (kRing - 1)];
            const double4 qq = q[p];
            int o[3];
            reach(pack[p], o);
            double *s = st + lane * SW + 3 * W;
            s[0] = qq.x; s[1] = qq.y; s[2] = qq.z;
            soff[lane] = (o[0] + TT) | (o[1] + TT) << 5 | (o[2] + TT) << 10;
        }
#pragma unroll
        for (int k = 0; k < NL; k++) {
            const int i = k * 64 + lane, c = i / (3 * W);
            if (c < nb) st[c * SW + (i - c * 3 * W)] = v[k];
        }
        wave_lds_sync();
        for (int c0 = 0; c0 < nb; c0 += 4) {
            const int c = c0 + k4;
            double a0 = 0.0, a1 = 0.0, bv[4] = {0.0, 0.0, 0.0, 0.0};
            if (c < nb) {
                const double *s = st + c * SW;
                const int op = soff[c];
                const int kx = (op & 31) - TT + (i16 & 7), ky = ((op >> 5) & 31) - TT + (i16 >> 3),
                          kz = ((op >> 10) & 31) - TT + (i16 & 7);
                const double wx = (unsigned)kx < (unsigned)W ? s[kx] : 0.0;
                const double wz = (unsigned)kz < (unsigned)W ? s[2 * W + kz] : 0.0;
                a0 = s[3 * W + (i16 >> 3)] * wz;
                if (i16 < 8) a1 = s[3 * W + 2] * wz;
#pragma unroll
                for (int b = 0; b < 4; b++) {
                    const int k = ky + 2 * b;
                    bv[b] = ((unsigned)k < (unsigned)W ? s[W + k] : 0.0) * wx;
                }
            }
#pragma unroll
            for (int b = 0; b < 4; b++) {
                dacc[0][b] = Mfma4<double>::op(a0, bv[b], dacc[0][b]);
                dacc[1][b] = Mfma4<double>::op(a1, bv[b], dacc[1][b]);
            }
        }
        head += nb;
        wave_lds_sync();
    };
    // four steps' bases loaded together; point 256 k + 4 lane + wave
    for (int k0 = 0; k0 < Nq; k0 += 1024) {
        unsigned pk[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const int p = k0 + 256 * k + 4 * lane + wave;
            pk[k] = p < Nq ? pack[p] : 0u;
        }
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const int p = k0 + 256 * k + 4 * lane + wave;
            int o[3];
            const bool act = reach(pk[k], o) && p < Nq;
            const unsigned long long m = __ballot(act);
            if (act) ring[(tail + bits_below(m)) & (kRing - 1)] = (unsigned short)p;
            tail += __popcll(m);
            while (tail - head >= kBatch) batch(kBatch);   // at most 31 + 64 queued
        }
    }
    if (tail > head) batch(tail - head);
    const size_t n3 = (size_t)n * n * n;
    // element i = (component, z) row i / 64, (y, x) column i % 64
    auto put = [&](int i, double v) {
        const int r = i >> 6, cell = i & 63;
        const size_t gi = ((size_t)(t0[2] + (r & 7)) * n + (t0[1] + (cell >> 3))) * n +
                          (t0[0] + (cell & 7));
        grid[(size_t)(r >> 3) * n3 + gi] = v;
    };
    if (!__syncthreads_or(tail > 0)) {   // no point reaches the tile
        for (int i = threadIdx.x; i < 1536; i += 256) put(i, 0.0);
        return;
    }
    // wavefronts 2, 3 onto 0, 1, then 0 + 1
    auto each = [&](auto f) {
#pragma unroll
        for (int a = 0; a < 2; a++)
#pragma unroll
            for (int b = 0; b < 4; b++)
#pragma unroll
                for (int v = 0; v < 4; v++) {
                    const int r = 16 * a + Mfma4<double>::row(k4, v);
                    if (r < 24) f(r * 64 + 16 * b + i16, dacc[a][b][v]);
                }
    };
    double *half = lds.st + (wave & 1) * 1536;
    if (wave >= 2) each([&](int i, double v) { half[i] = v; });
    __syncthreads();
    if (wave < 2) each([&](int i, double v) { half[i] += v; });   // own elements only
    __syncthreads();
    for (int i = threadIdx.x; i < 1536; i += 256) put(i, lds.st[i] + lds.st[1536 + i]);
}

template <int W>
__global__ __launch_bounds__(256) void k_spread_direct(int n, int NT, int Nq,
                                                       const unsigned *__restrict__ pack,
                                                       const double *__restrict__ ker,
                                                       const double4 *__restrict__ q,
                                                       double *__restrict__ grid) {
    __shared__ SpreadLds<W> lds;
    spread_direct<W>(blockIdx.x, n, NT, Nq, pack, ker, q, grid, lds);
}

// The spread's workgroups first (the transforms wait for them), then the
// pair sums' (four targets each), which fill the chip beside them: a second
// stream with its fork and join costs 22 us of host time per evaluation.
template <int W>
__global__ __launch_bounds__(256) void k_spread_pairs(int n, int NT, int ntiles, int N, int Nq,
                                                      PieceList pl,
                                                      const unsigned *__restrict__ pack,
                                                      const double *__restrict__ ker,
                                                      const double4 *__restrict__ q,
                                                      double *__restrict__ grid, PairGeom G,
                                                      const double4 *__restrict__ tgt,
                                                      const double4 *__restrict__ spos, ShortFit fit,
                                                      const double *__restrict__ base,
                                                      double *__restrict__ out) {
    __shared__ union U {
        SpreadLds<W> s;
        PairLds p;
        __device__ U() {}
    } lds;
    if ((int)blockIdx.x < ntiles)
        spread_direct<W>(blockIdx.x, n, NT, Nq, pack, ker, q, grid, lds.s);
    else
        pairs_direct<false, 1>((int)blockIdx.x - ntiles, N, G, pl, tgt, spos, q, fit, base, out,
                               lds.p);
}

__global__ __launch_bounds__(256) void k_direct_gather(int N, int Nq, int Q,
                                                       const double *__restrict__ x,
                                                       const double *__restrict__ qpos,
                                                       const double *__restrict__ qchg,
                                                       const int *__restrict__ off,
                                                       const int *__restrict__ fil, DirectOut d,
                                                       int nfil) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    // a wavefront per piece: its filament is the last one that starts at or before
    const int np = d.pfirst[nfil];
    for (int pc = t >> 6; pc < np; pc += (int)(gridDim.x * blockDim.x) >> 6) {
        int f = 0;
        for (int lo = 0, hi = nfil; hi - lo > 1;) {
            const int mid = (lo + hi) >> 1;
            if (d.pfirst[mid] <= pc) lo = mid; else hi = mid;
            f = lo;
        }
        const int j = pc - d.pfirst[f], b0 = off[f] + j * kPiece, e0 = min(b0 + kPiece, off[f + 1]);
        direct_piece(d.piece + pc, qpos + 3 * (size_t)b0 * Q, b0 * Q, (e0 - b0) * Q, d.L);
    }
    if (t < Nq * 3 * d.w) d.ker[t] = direct_value(qpos[t / d.w], t % d.w, d);
    if (t < Nq) direct_point(t, t / Q, qpos + 3 * t, qchg + 3 * t, d);
    if (t < N) direct_node(t, prev_node_d(off, fil, t), x + 3 * t, d);
}

void launch_direct_gather(bs_plan_t p) {
    const int items = (int)p->Nq * 3 * p->prm.w;   // more than Nq >= N
    hipLaunchKernelGGL(k_direct_gather, dim3(ceil_div(items, 256)), dim3(256), 0, p->stream,
                       (int)p->N, (int)p->Nq, p->Q, (const double *)p->d_x.p,
                       (const double *)p->d_qpos.p, (const double *)p->d_qchg.p,
                       (const int *)p->d_off.p, (const int *)p->d_fil.p, direct_out(p), (int)p->nfil);
}

template <int W>
static void spread_w(bs_plan_t p, const double *base, double *out) {
    const int nt = p->NT * p->NT * p->NT, N = (int)p->N, Nq = (int)p->Nq;
    const DirectOut d = direct_out(p);
    double *grid = (double *)p->grid.p;
    if (!out) {
        hipLaunchKernelGGL(k_spread_direct<W>, dim3(nt), dim3(256), 0, p->stream, p->n, p->NT, Nq,
                           (const unsigned *)d.pack, (const double *)d.ker, (const double4 *)d.q,
                           grid);
        return;
    }
    hipLaunchKernelGGL(k_spread_pairs<W>, dim3(nt + ceil_div(N, 4)), dim3(256), 0, p->stream, p->n,
                       p->NT, nt, N, Nq, piece_list(p), (const unsigned *)d.pack, (const double *)d.ker,
                       (const double4 *)d.q, grid, pair_geom(p), (const double4 *)d.tgt,
                       (const double4 *)d.spos, short_fit(), base, out);
}

static void spread_any(bs_plan_t p, const double *base, double *out) {
    switch (p->prm.w) {
        case 4: return spread_w<4>(p, base, out);
        case 5: return spread_w<5>(p, base, out);
        case 6: return spread_w<6>(p, base, out);
        case 7: return spread_w<7>(p, base, out);
        case 8: return spread_w<8>(p, base, out);
        case 9: return spread_w<9>(p, base, out);
        case 10: return spread_w<10>(p, base, out);
        case 11: return spread_w<11>(p, base, out);
        case 12: return spread_w<12>(p, base, out);
        case 13: return spread_w<13>(p, base, out);
        case 14: return spread_w<14>(p, base, out);
        case 15: return spread_w<15>(p, base, out);
        case 16: return spread_w<16>(p, base, out);
        default: return;
    }
}

void launch_spread_direct(bs_plan_t p) { spread_any(p, nullptr, nullptr); }
void launch_spread_pairs(bs_plan_t p, const double *base, double *out) { spread_any(p, base, out); }

// Taken where scanning every point per tile and per target costs less than the
// four launches of the sorts and the second stream: evaluations of rings of 64 nodes
// in us, through the sorts and direct,
//              64 nodes   640       1280      2560      4096      6400
//   32^3 w 8   76  37     84  47    100  55   138  93   189 151   312 268
//   64^3 w 8   80  46     85  52     88  57    97  73   109  93   127 130
//   96^3 w 8  119  82    131  89    131  94   139 108   146 127   155 161
//   128^3 w 8 149 123    155 134    160 145   168 168   174 198
//   160^3 w 8 213 196    223 215    226 235   232 271
//   192^3 w 8 310 312    318 339
//   128^3 w 12 164 134   173 149    179 162   202 191   213 227
//   64^3 w 16  94  62    104  75    114  87   134 121   156 169
//   128^3 w 16 166 157   179 193    189 222   223 278   239 346
//   160^3 w 16 231 248   250 298
//   256^3 w 16 745 928   778 1100
// so up to 8192 points on up to 8192 tiles with up to 2^24 tests of a point against a
// tile; wide kernels, whose staging leaves few workgroups per CU, up to 4096 tiles
// and 3 2^20 tests.
constexpr int64_t kDirectPoints = 8192;
constexpr int64_t kDirectTiles = 8192, kDirectTests = (int64_t)1 << 24;
constexpr int64_t kDirectTilesWide = 4096, kDirectTestsWide = (int64_t)3 << 20;
constexpr int kDirectWide = 13;
bool direct_path(bs_plan_t p, int64_t Nq) {
    const int64_t nt = (int64_t)p->NT * p->NT * p->NT;
    const bool wide = p->prm.w >= kDirectWide;
    return !p->fp32 && p->T == kTile && Nq <= kDirectPoints &&
           nt <= (wide ? kDirectTilesWide : kDirectTiles) &&
           nt * Nq <= (wide ? kDirectTestsWide : kDirectTests);
}

}  // namespace bs
