// Binning of quadrature points and nodes (counting sort), and the sorted
// structure-of-arrays copies that the spread, interpolation and pair kernels
// read.
//
//   spread bins : tile of T^3 grid cells containing a point's stencil base
//                 (lowest grid index of its w-point support per axis);
//   pair cells  : the cell-list idea of Sec. 5.3 (pair_cells): in float64
//                 cells of edges >= r_c / 3 along x and r_c / 2 along y, z; in
//                 float32 ncell^3 cells of edge L/ncell >= 2 r_c / 3, so that
//                 the 4 x 4 x 4 cells from the cell of x - r_c on hold every
//                 point within r_c of x;
//   node order  : nodes sorted by cell (ncell^3), so neighbouring threads share
//                 cells in the pair and interpolation kernels.
//
// Within a bin, entries are ordered by original index so that every sum the
// later kernels form has a fixed order (bitwise reproducible results).
#include <algorithm>

#include "bs_internal.h"
#include "bs_device.h"

namespace bs {

// ------------------------------------------------------------ scan (int32)
constexpr int kScanBlock = 256, kScanItems = 8, kScanTile = kScanBlock * kScanItems;

__device__ int block_exclusive_scan(int v, int *sh, int *total) {
    // Hillis-Steele scan over the block in LDS
    int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int o = 1; o < blockDim.x; o <<= 1) {
        int add = (t >= o) ? sh[t - o] : 0;
        __syncthreads();
        sh[t] += add;
        __syncthreads();
    }
    int incl = sh[t];
    *total = sh[blockDim.x - 1];
    __syncthreads();
    return incl - v;
}

// up to three arrays scanned side by side: array a has its blocks
// [blk[a], blk[a + 1]) of the reduce and apply launches and its own part of
// the block sums (starting at blk[a])
struct ScanSet {
    const int *in[3];
    int *out[3];
    int n[3], blk[4];
    const int *lim;   // when set: the arrays' sizes, decided on the device (at most n)
};
__device__ __forceinline__ int scan_size(const ScanSet &S, int a) {
    return S.lim ? S.lim[a] : S.n[a];
}

__device__ __forceinline__ int scan_array(const ScanSet &S) {
    return (int)blockIdx.x >= S.blk[2] ? 2 : ((int)blockIdx.x >= S.blk[1] ? 1 : 0);
}

__global__ void k_scan_reduce(ScanSet S, int *__restrict__ sums) {
    __shared__ int sh[kScanBlock];
    const int a = scan_array(S), n = scan_size(S, a);
    if (((int)blockIdx.x - S.blk[a]) * kScanTile >= n) return;
    const int *in = S.in[a];
    int base = ((int)blockIdx.x - S.blk[a]) * kScanTile + threadIdx.x * kScanItems;
    int s = 0;
    for (int k = 0; k < kScanItems; k++)
        if (base + k < n) s += in[base + k];
    int tot;
    block_exclusive_scan(s, sh, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// one workgroup per array; out[n] = total
__global__ void k_scan_sums(ScanSet S, int *__restrict__ sums) {
    __shared__ int sh[kScanBlock];
    const int a = blockIdx.x, n = scan_size(S, a), nb = (n + kScanTile - 1) / kScanTile;
    // nb <= kScanTile
    int *sa = sums + S.blk[a];
    int base = threadIdx.x * kScanItems;
    int v[kScanItems], s = 0;
    for (int k = 0; k < kScanItems; k++) {
        v[k] = (base + k < nb) ? sa[base + k] : 0;
        s += v[k];
    }
    int tot;
    int ex = block_exclusive_scan(s, sh, &tot);
    for (int k = 0; k < kScanItems; k++) {
        if (base + k < nb) sa[base + k] = ex;
        ex += v[k];
    }
    if (threadIdx.x == 0) S.out[a][n] = tot;
}

__global__ void k_scan_apply(ScanSet S, const int *__restrict__ sums) {
    __shared__ int sh[kScanBlock];
    const int a = scan_array(S), n = scan_size(S, a);
    if (((int)blockIdx.x - S.blk[a]) * kScanTile >= n) return;
    const int *in = S.in[a];
    int *out = S.out[a];
    int base = ((int)blockIdx.x - S.blk[a]) * kScanTile + threadIdx.x * kScanItems;
    int v[kScanItems], s = 0;
    for (int k = 0; k < kScanItems; k++) {
        v[k] = (base + k < n) ? in[base + k] : 0;
        s += v[k];
    }
    int tot;
    int ex = block_exclusive_scan(s, sh, &tot) + sums[blockIdx.x];
    for (int k = 0; k < kScanItems; k++) {
        if (base + k < n) out[base + k] = ex;
        ex += v[k];
    }
}

void scan_arrays(bs_plan_t p, int na, const int *const *in, int *const *out, const int *n,
                 int *sums, const int *lim) {
    ScanSet S{};
    S.lim = lim;
    for (int a = 0; a < 3; a++) {
        if (a < na) { S.in[a] = in[a]; S.out[a] = out[a]; S.n[a] = n[a]; }
        S.blk[a + 1] = S.blk[a] + (a < na ? ceil_div(n[a], kScanTile) : 0);
    }
    const dim3 g(S.blk[3]), b(kScanBlock);
    hipLaunchKernelGGL(k_scan_reduce, g, b, 0, p->stream, S, sums);
    hipLaunchKernelGGL(k_scan_sums, dim3(na), b, 0, p->stream, S, sums);
    hipLaunchKernelGGL(k_scan_apply, g, b, 0, p->stream, S, (const int *)sums);
}

// out[0..n-1] = exclusive scan of in, out[n] = total (n: S.lim's, if set).  in
// and out may not alias.  Requires n <= kScanTile^2 (4.2 M bins); sums: kScanTile ints of
// scratch, private to the stream.
void exclusive_scan(bs_plan_t p, const int *in, int *out, int n, int *sums) {
    scan_arrays(p, 1, &in, &out, &n, sums, nullptr);
}

// ------------------------------------------------------- fused bin passes
// The three sorts (quadrature points by spread tile, quadrature points by pair
// cell, nodes by pair cell) run side by side: each pass below is one launch
// covering all three.
struct SortSet {
    int *key[3], *cnt[3], *start[3], *fill[3], *perm[3];
    int nbins[3], nitems[3];
    int share[3], nwave[3];   // the per-bin sort: entries per wavefront, wavefronts
    int *tmp[3];              // scratch of the array's size, free until the gather
};


// one workgroup per array: exclusive scan of cnt into start (start[n] =
// total).  Wavefront w owns the contiguous segment [w seg, (w + 1) seg) and
// takes it 256 entries at a time, four consecutive ones per lane: a first
// pass sums it, the segment offsets are formed from the 16 sums in LDS, and a
// second pass scans each 256-entry chunk by data-parallel moves while writing
// (one entry per lane took 12.1 us for 14112 bins, four 5.0).
__global__ __launch_bounds__(1024) void k_scan_small(SortSet S) {
    __shared__ int wsum[16];
    const int a = blockIdx.x;
    const int n = S.nbins[a];
    const int *in = S.cnt[a];
    int *out = S.start[a];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int seg = ((n + nw - 1) / nw + 255) / 256 * 256;
    const int b0 = min(wave * seg, n), b1 = min(b0 + seg, n);
    auto load = [&](int i) {   // in[i .. i + 3], zero beyond the segment; i is a multiple of 4
        if (i + 3 < b1) return *(const int4 *)(in + i);
        return make_int4(i < b1 ? in[i] : 0, i + 1 < b1 ? in[i + 1] : 0, i + 2 < b1 ? in[i + 2] : 0, 0);
    };
    int sum = 0;
    for (int i = b0 + 4 * lane; i < b1; i += 256) {
        const int4 v = load(i);
        sum += v.x + v.y + v.z + v.w;
    }
    sum = __builtin_amdgcn_readlane(wave_incl_sum(sum), 63);
    if (lane == 0) wsum[wave] = sum;
    __syncthreads();
    int carry = 0;
    for (int w = 0; w < wave; w++) carry += wsum[w];
    for (int c0 = b0; c0 < b1; c0 += 256) {
        const int i = c0 + 4 * lane;
        const int4 v = load(i);
        const int s = v.x + v.y + v.z + v.w, incl = wave_incl_sum(s), e = carry + incl - s;
        const int4 r = make_int4(e, e + v.x, e + v.x + v.y, e + v.x + v.y + v.z);
        if (i + 3 < b1) {
            *(int4 *)(out + i) = r;
        } else {
            if (i < b1) out[i] = r.x;
            if (i + 1 < b1) out[i + 1] = r.y;
            if (i + 2 < b1) out[i + 2] = r.z;
        }
        carry += __builtin_amdgcn_readlane(incl, 63);
    }
    if (threadIdx.x == 0) {
        int tot = 0;
        for (int w = 0; w < nw; w++) tot += wsum[w];
        out[n] = tot;
    }
}

__global__ void k_scatter_all(SortSet S) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    int a = 0;
    if (i >= S.nitems[0]) { i -= S.nitems[0]; a = 1; }
    if (a == 1 && i >= S.nitems[1]) { i -= S.nitems[1]; a = 2; }
    const bool valid = !(a == 2 && i >= S.nitems[2]);
    const int k = valid ? S.key[a][i] : 0;
    const bool one = S.nbins[a] == 1;   // one bin: already in index order
    if (one && valid) S.perm[a][i] = i;
    // one atomic per (set, bin) group of the wavefront, all issued together
    const bool act = valid && !one;
    const WaveGroup g = wave_group(k, a, act);
    int old = 0;
    if (act && (int)(threadIdx.x & 63) == g.leader) old = atomicAdd(S.fill[a] + k, g.size);
    const int slot = __shfl(old, g.leader) + g.rank;
    if (act) S.perm[a][S.start[a][k] + slot] = i;
}

// Orders every bin's entries by original index.  A wavefront takes the bins that
// begin in its share of the array's entries, so that neither many empty bins nor a
// few full ones, wherever they lie, leave work to one wavefront (groups of up to
// 64 bins each, with the counting below for every bin, took 1.8 ms instead of 0.24
// and 133 ms instead of 0.31 for clusters of 20000 and 1e5 nodes on 512^3; on the
// 1e6-node tangle both take 0.40).  Those bins' entries form one contiguous range, of which
// only the last bin may reach beyond the share.  Up to kSortLds entries: staged
// in LDS, each counts the smaller ones of its own bin.  Beyond: so the bins but
// the last, and the last one by digits (radix_sort_bin).  The other wavefronts
// may be moving entries meanwhile, but only within their bins: a position's bin
// can be read at any time.
constexpr int kSortLds = 1024;
// entries per wavefront of the per-bin sort: 16 to 64 on small inputs, up to 256 where
// that leaves more wavefronts than the chip holds (eight per SIMD).  A wavefront's
// last bin reaches beyond its share, so 16 saves a round of counting (1134 nodes
// 7.7 -> 6.6 us), but not where it only makes more wavefronts (1e5 nodes 9.4 -> 12.9)
constexpr int kSortShare = 16, kSortFew = 512, kSortWaves = 8192, kSortShareMax = 256;
static_assert(kSortShareMax <= kSortLds && 256 <= kSortLds, "a share, or the digits, in LDS");

// LDS of the per-bin sort: the staged entries (or the digits' counts) and, of those in
// the share, where their bin begins and ends among them
struct SortLds {
    int v[kSortLds];
    int range[kSortShareMax];
};
static_assert(kSortLds < 1 << 15, "both ends in an int");

// n distinct entries below 2^nbits at a, in ascending order, by one wavefront:
// stable passes over eight bits at a time between a and t (n values of scratch).
// Counting the smaller ones, as the bins in LDS do, took 1.5 s where 20000 nodes
// fill a handful of bins, against 0.7 ms (all of the binning).
__device__ __forceinline__ void radix_sort_bin(int *a, int *t, int n, int nbits, SortLds &S) {
    const int lane = threadIdx.x & 63;
    int *cnt = S.v;   // 256 counts, then the digits' next positions
    int *src = a, *dst = t;
    for (int sh = 0; sh < nbits; sh += 8) {
        for (int i = lane; i < 256; i += 64) cnt[i] = 0;
        wave_lds_sync();
        // (four steps' loads in flight)
        for (int i0 = 0; i0 < n; i0 += 256) {
            int x[4];
#pragma unroll
            for (int u = 0; u < 4; u++) x[u] = src[min(i0 + 64 * u + lane, n - 1)];
#pragma unroll
            for (int u = 0; u < 4; u++)
                if (i0 + 64 * u + lane < n) atomicAdd(&cnt[(x[u] >> sh) & 255], 1);
        }
        wave_lds_sync();
        int c[4], s = 0;
        for (int k = 0; k < 4; k++) { c[k] = cnt[4 * lane + k]; s += c[k]; }
        int e = wave_incl_sum(s) - s;
        for (int k = 0; k < 4; k++) { cnt[4 * lane + k] = e; e += c[k]; }
        wave_lds_sync();
        int next[4];
#pragma unroll
        for (int u = 0; u < 4; u++) next[u] = src[min(64 * u + lane, n - 1)];
        for (int i0 = 0; i0 < n; i0 += 256) {
            int x[4];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                x[u] = next[u];
                next[u] = src[min(i0 + 256 + 64 * u + lane, n - 1)];
            }
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const bool act = i0 + 64 * u + lane < n;
                const int d = (x[u] >> sh) & 255;
                // the lanes with the same digit
                unsigned long long m = __ballot(act);
#pragma unroll
                for (int k = 0; k < 8; k++) {
                    const unsigned long long bit = __ballot((d >> k) & 1);
                    m &= ((d >> k) & 1) ? bit : ~bit;
                }
                const int base = cnt[d], r = bits_below(m);
                wave_lds_sync();   // read before the group's last lane moves it on
                if (act) {
                    dst[base + r] = x[u];
                    if (r + 1 == __popcll(m)) cnt[d] = base + r + 1;
                }
                wave_lds_sync();
            }
        }
        __threadfence();   // the pass's stores before the next one's loads
        int *const p = src; src = dst; dst = p;
    }
    if (src != a) {
        for (int i = lane; i < n; i += 64) a[i] = src[i];
    }
}

__global__ __launch_bounds__(64) void k_sort_all(SortSet S) {
    int w = blockIdx.x, a = 0;
    if (w >= S.nwave[0]) { w -= S.nwave[0]; a = 1; }
    if (a == 1 && w >= S.nwave[1]) { w -= S.nwave[1]; a = 2; }
    __shared__ SortLds L;
    const int lane = threadIdx.x;
    int *perm = S.perm[a], *cnt = S.cnt[a], *fill = S.fill[a];
    const int *key = S.key[a], *start = S.start[a];
    // the bins' counters are not read again: those of the bins that hold entries are
    // cleared for the next call (the per-filament kernel counts into them)
    if (S.nbins[a] == 1) {   // one bin: the scatter wrote the identity
        if (lane == 0) cnt[0] = fill[0] = 0;
        return;
    }
    // the share's entries and their bins, up to four per lane (three round trips to
    // memory; with its ends looked up first, six, 1e4 nodes took 7.4 us instead of 5.8)
    constexpr int U = kSortShareMax / 64;
    const int share = S.share[a], v0 = w * share, v1 = min(v0 + share, S.nitems[a]);
    int x[U], b[U], lo[U], hi[U];
#pragma unroll
    for (int u = 0; u < U; u++)
        if (64 * u < share) x[u] = perm[min(v0 + 64 * u + lane, v1 - 1)];
#pragma unroll
    for (int u = 0; u < U; u++)
        if (64 * u < share) b[u] = key[x[u]];
    int bl = 0, lol = 0, e0 = 0;   // the bin of the share's last entry, its range
#pragma unroll
    for (int u = 0; u < U; u++)
        if (64 * u < share) {
            lo[u] = start[b[u]];
            hi[u] = start[b[u] + 1];
            bl = b[u]; lol = lo[u]; e0 = hi[u];
        }
    bl = __shfl(bl, 63);
    lol = __shfl(lol, 63);
    e0 = __shfl(e0, 63);
    const int first = __shfl(lo[0], 0), s0 = first == v0 ? v0 : __shfl(hi[0], 0);
    if (s0 >= v1) return;
    if (e0 - s0 > kSortLds) {
        if (lane == 0) cnt[bl] = fill[bl] = 0;
        const int nbits = 32 - __clz(S.nitems[a] - 1);
        radix_sort_bin(perm + lol, S.tmp[a] + lol, e0 - lol, nbits, L);
        e0 = lol;   // at most a share is left
        __syncthreads();   // the LDS is free
    }
    // beyond m - s0, the last bin's entries outside the share
    const int m = min(e0, v1), total = e0 - s0;
#pragma unroll
    for (int u = 0; u < U; u++) {
        const int i = v0 + 64 * u + lane;
        if (64 * u < share && i >= s0 && i < m) {
            L.v[i - s0] = x[u];
            L.range[i - s0] = (lo[u] - s0) | (hi[u] - s0) << 16;
            cnt[b[u]] = 0;
            fill[b[u]] = 0;
        }
    }
    for (int i = v1 + lane; i < e0; i += 64) L.v[i - s0] = perm[i];
    wave_lds_sync();
    for (int i = lane; i < total; i += 64) {
        const int y = L.v[i], g = i < m - s0 ? L.range[i] : (lol - s0) | total << 16;
        const int l = g & 0xffff, h = g >> 16;
        int r = l;
#pragma unroll 8
        for (int j = l; j < h; j++) r += (L.v[j] < y);
        perm[s0 + r] = y;
    }
}

// sorted copies for the spread (by tile) and the pairs (by cell), one pass;
// thread (p, d) handles axis d of sorted entry p (its stencil base and w
// kernel values, and component d of the charges and pair position).  A
// separate launch from the per-bin sort: there a heavy bin's workgroup would
// gather its entries alone (measured 5.5 + 6.4 us -> 21.6 us fused).
struct GatherOut {
    int4 *base;
    void *ker, *q, *schg;
    double4 *spos;   // w: the point's segment index
    double4 *tgt;    // nodes in cell order: wrapped position, node and its predecessor
};

// (the w kernel values of thread t go to lk[0 .. w-1]; the caller writes them
// to ker[t w ..])
template <typename R>
__device__ __forceinline__ void gather_one(int t, int w, int Q, const int *__restrict__ sperm,
                                           const int *__restrict__ pperm,
                                           const double *__restrict__ pos,
                                           const double *__restrict__ chg, double L, double inv_h,
                                           int n, const KbPhi &kb, const GatherOut &G, R *lk) {
    const int p = t / 3, d = t - 3 * p;
    R *q = (R *)G.q, *schg = (R *)G.schg;
    int o = sperm[p];
    double f;
    const int b = stencil_base(wrap_box(pos[3 * o + d], L), inv_h, w, n, &f);
    const double half = 0.5 * w;
    for (int k = 0; k < w; k++) lk[k] = kb_value<R>((k - f) / half, kb);
    int *bp = (int *)(G.base + p);
    bp[d] = b;
    q[4 * (size_t)p + d] = (R)chg[3 * o + d];
    o = pperm[p];
    double *sp = (double *)(G.spos + p);
    sp[d] = wrap_box(pos[3 * o + d], L);
    schg[4 * (size_t)p + d] = (R)chg[3 * o + d];
    if (d == 0) {
        bp[3] = 0;
        q[4 * (size_t)p + 3] = (R)0;
        sp[3] = (double)(o / Q);
        schg[4 * (size_t)p + 3] = (R)0;
    }
}

// Thread t = 3 p + d writes its kernel values at ker[t w ..], so those of a
// workgroup form one contiguous range: they are staged in LDS and written out
// with consecutive threads on consecutive words (a thread writing its own w
// values touched a cache line per lane in each store).  256 threads, w <= 16.
// The last workgroups write the nodes' records (a thread per node), from which
// the pair and interpolation kernels take their target in one load.
constexpr int kGatherBlock = 256;
template <typename R>
__global__ __launch_bounds__(kGatherBlock) void k_gather_all(int M, int w, int Q,
                                                             const int *__restrict__ sperm,
                                                             const int *__restrict__ pperm,
                                                             const double *__restrict__ pos,
                                                             const double *__restrict__ chg,
                                                             double L, double inv_h, int n,
                                                             KbPhi kb, GatherOut G, int N,
                                                             const int *__restrict__ nperm,
                                                             const double *__restrict__ x,
                                                             const int *__restrict__ off,
                                                             const int *__restrict__ fil) {
    __shared__ R lk[kGatherBlock * 16];
    const int npt = (3 * M + kGatherBlock - 1) / kGatherBlock;   // workgroups of the points
    if ((int)blockIdx.x >= npt) {
        const int t = ((int)blockIdx.x - npt) * kGatherBlock + (int)threadIdx.x;
        if (t >= N) return;
        const int o = nperm[t];
        G.tgt[t] = make_double4(wrap_box(x[3 * o], L), wrap_box(x[3 * o + 1], L),
                                wrap_box(x[3 * o + 2], L),
                                __hiloint2double(prev_node_d(off, fil, o), o));
        return;
    }
    const int t0 = blockIdx.x * kGatherBlock, t = t0 + (int)threadIdx.x;
    if (t < 3 * M)
        gather_one<R>(t, w, Q, sperm, pperm, pos, chg, L, inv_h, n, kb, G, lk + threadIdx.x * w);
    __syncthreads();
    const int nt = 3 * M - t0 < kGatherBlock ? 3 * M - t0 : kGatherBlock;
    R *ker = (R *)G.ker + (size_t)t0 * w;
    for (int i = threadIdx.x; i < nt * w; i += kGatherBlock) ker[i] = lk[i];
}

// arrays of at most this many bins are scanned by one workgroup each (one
// launch, 5.0 us at 14112 bins and 7.4 at 21312, but 240 at the 98^3 node cells of a
// loose tolerance on 256^3; the three launches of the blocked scan take 14 us)
constexpr int kScanSmall = 32768;

void build_bins(bs_plan_t p) {
    const int bs = 256;
    const int M = (int)p->Nq, N = (int)p->N;
    const double L = p->prm.L, inv_h = p->n / L;
    const int w = p->prm.w, n = p->n;
    const int ntiles = p->NT * p->NT * p->NT, nc3 = p->nc * p->nc * p->nc,
              ncp = p->ncx * p->ncy * p->ncy;
    SortSet S;
    S.key[0] = (int *)p->sp_key.p; S.cnt[0] = (int *)p->sp_cnt.p; S.start[0] = (int *)p->sp_start.p;
    S.fill[0] = (int *)p->sp_fill.p; S.perm[0] = (int *)p->sp_perm.p;
    S.key[1] = (int *)p->pq_key.p; S.cnt[1] = (int *)p->pq_cnt.p; S.start[1] = (int *)p->pq_start.p;
    S.fill[1] = (int *)p->pq_fill.p; S.perm[1] = (int *)p->pq_perm.p;
    S.key[2] = (int *)p->nd_key.p; S.cnt[2] = (int *)p->nd_cnt.p; S.start[2] = (int *)p->nd_start.p;
    S.fill[2] = (int *)p->nd_fill.p; S.perm[2] = (int *)p->nd_perm.p;
    S.nbins[0] = ntiles; S.nbins[1] = ncp; S.nbins[2] = nc3;
    S.nitems[0] = M; S.nitems[1] = M; S.nitems[2] = N;
    S.tmp[0] = (int *)p->sp_q.p; S.tmp[1] = (int *)p->pq_pos.p; S.tmp[2] = (int *)p->nd_rec.p;
    for (int a = 0; a < 3; a++) {
        int sh = kSortShare;
        while (sh < kSortShareMax &&
               (int64_t)sh * (sh < 64 ? kSortFew : kSortWaves) < S.nitems[a])
            sh *= 2;
        S.share[a] = sh;
        S.nwave[a] = S.nbins[a] == 1 ? 1 : ceil_div(S.nitems[a], sh);
    }
    const int maxb = std::max({ntiles, ncp, nc3});
    GatherOut G;
    G.base = (int4 *)p->sp_base.p;
    G.ker = p->sp_ker.p;
    G.q = p->sp_q.p;
    G.spos = (double4 *)p->pq_pos.p;
    G.schg = p->pq_chg.p;
    G.tgt = (double4 *)p->nd_rec.p;
    const double *qp = (const double *)p->d_qpos.p, *qc = (const double *)p->d_qchg.p;
    // keys and counts come from the per-filament kernel (bin_keys)
    if (maxb <= kScanSmall) {
        hipLaunchKernelGGL(k_scan_small, dim3(3), dim3(1024), 0, p->stream, S);
    } else {
        scan_arrays(p, 3, S.cnt, S.start, S.nbins, (int *)p->red_tmp.p, nullptr);
    }
    hipLaunchKernelGGL(k_scatter_all, dim3(ceil_div(2 * (int64_t)M + N, bs)), dim3(bs), 0, p->stream, S);
    hipLaunchKernelGGL(k_sort_all, dim3(S.nwave[0] + S.nwave[1] + S.nwave[2]), dim3(64), 0, p->stream, S);
    const dim3 gg(ceil_div(3 * (int64_t)M, kGatherBlock) + ceil_div(N, kGatherBlock));
    const double *x = (const double *)p->d_x.p;
    const int *off = (const int *)p->d_off.p, *fil = (const int *)p->d_fil.p;
    auto gather = p->fp32 ? k_gather_all<float> : k_gather_all<double>;
    hipLaunchKernelGGL(gather, gg, dim3(kGatherBlock), 0, p->stream, M, w, p->Q, S.perm[0],
                       S.perm[1], qp, qc, L, inv_h, n, p->kb, G, N, S.perm[2], x, off, fil);
}

BinKeys bin_keys(bs_plan_t p) {
    BinKeys k;
    k.key[0] = (int *)p->sp_key.p; k.cnt[0] = (int *)p->sp_cnt.p;
    k.key[1] = (int *)p->pq_key.p; k.cnt[1] = (int *)p->pq_cnt.p;
    k.key[2] = (int *)p->nd_key.p; k.cnt[2] = (int *)p->nd_cnt.p;
    k.L = p->prm.L;
    k.inv_h = p->n / p->prm.L;
    k.w = p->prm.w; k.n = p->n; k.T = p->T; k.NT = p->NT; k.nc = p->nc;
    k.ncx = p->ncx; k.ncy = p->ncy;
    return k;
}

}  // namespace bs
