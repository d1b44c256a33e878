// Small MLP 8 -> 64 -> 64 -> 64 -> 3 (SiLU hidden activations) on BF16 MFMA
// with FP32 accumulation: inference, loss gradient and Adam training.  Used
// by the learned near-singular correction (no counterpart in the paper).  A
// debug mode (bs_mlp_set_fp32) runs the same kernels with FP32 weights and
// activations on FP32 MFMA, leaving only FP32 rounding in the gradients.
//
// Master parameters are FP32, packed W1[64][8] b1[64] W2[64][64] b2[64]
// W3[64][64] b3[64] W4[3][64] b4[3] (9091 values).  The kernels read a padded
// BF16 image of the weights:
//   W1p[64][16]: columns 0..7 and 8..15 both hold W1, so that the input
//                vector can be fed as (hi, lo) BF16 halves of each FP32
//                feature: W1 x = W1 hi + W1 lo keeps ~16 mantissa bits of x;
//   W2[64][64], W3[64][64];  W4p[16][64]: rows 3..15 zero;
// and FP32 biases b1, b2, b3 and b4p[16].
//
// One wavefront handles 16 samples at a time with v_mfma_f32_16x16x16_bf16
// in the transposed orientation Z^T = W H^T: the MFMA result layout (lane l
// holds rows 4(l/16)..4(l/16)+3 of column l%16) is exactly the B-operand
// layout of the next layer, so activations never leave registers in the
// forward pass.  Backward: dH^T = W^T dZ^T by MFMA in the same orientation;
// dW = dZ^T H by MFMA over a workgroup's samples, both factors transposed
// through LDS, each wavefront owning a share of the output blocks in registers.
// The workgroup partials are added in a fixed order by a second kernel, which
// writes the gradient (or takes the Adam step).
#include <algorithm>

#include "bs_internal.h"
#include "bs_device.h"

namespace bs {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kH = 64;                       // hidden width
constexpr int kNP = 9091;                    // master parameter count
// padded image offsets (in elements)
constexpr int kW1p = 0, kW2 = kW1p + 64 * 16, kW3 = kW2 + 64 * 64, kW4p = kW3 + 64 * 64;
constexpr int kWpad = kW4p + 16 * 64;        // 10240 bf16 weights
constexpr int kB1 = 0, kB2 = 64, kB3 = 128, kB4p = 192, kBpad = 208;   // fp32 biases
constexpr int kGpad = kWpad + kBpad;         // padded gradient length (fp32)
// the same image in LDS, rows padded by 4 elements against bank conflicts
constexpr int kLd1 = 20, kLd = 68;
constexpr int kL1 = 0, kL2 = kL1 + 64 * kLd1, kL3 = kL2 + 64 * kLd, kL4 = kL3 + 64 * kLd;
constexpr int kLpad = kL4 + 16 * kLd;

__device__ __forceinline__ unsigned short f2bf(float f) {
    unsigned int u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);          // round to nearest even
    return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf2f(unsigned short h) {
    return __uint_as_float(((unsigned int)h) << 16);
}
// SiLU and its derivative with the hardware exp2 and reciprocal (1 ulp in
// float32; the activations are rounded to bf16 right after)
__device__ __forceinline__ float sigmoid_f(float z) {
    return __builtin_amdgcn_rcpf(1.0f + __expf(-z));
}
__device__ __forceinline__ float silu(float z) { return z * sigmoid_f(z); }
__device__ __forceinline__ float dsilu(float z) {
    const float s = sigmoid_f(z);
    return s * (1.0f + z * (1.0f - s));
}

// Precision of a kernel instance: F = false, BF16 operands on
// v_mfma_f32_16x16x16_bf16 (the product); F = true, FP32 weights and
// activations on v_mfma_f32_16x16x4_f32, four per 16x16x16 product (a debug
// mode that leaves only FP32 rounding, for checking the gradients tightly).
// The operand registers hold the same k indices in both: lane l, element j
// is k = 4(l/16) + j; the j-th FP32 MFMA sums k = j, 4 + j, 8 + j, 12 + j.
template <bool F> struct Prec {
    typedef unsigned short W;   // stored weights and tiles
    typedef bf16x4 Op;          // MFMA operand
    static __device__ __forceinline__ W store(float v) { return f2bf(v); }
    static __device__ __forceinline__ float elem(W w) { return bf2f(w); }
    static __device__ __forceinline__ f32x4 mfma(Op a, Op b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ void set(Op &o, int r, W w) { o[r] = (short)w; }
};
template <> struct Prec<true> {
    typedef float W;
    typedef f32x4 Op;
    static __device__ __forceinline__ W store(float v) { return v; }
    static __device__ __forceinline__ float elem(W w) { return w; }
    static __device__ __forceinline__ f32x4 mfma(Op a, Op b, f32x4 c) {
#pragma unroll
        for (int j = 0; j < 4; j++) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[j], c, 0, 0, 0);
        return c;
    }
    static __device__ __forceinline__ void set(Op &o, int r, W w) { o[r] = w; }
};

template <bool F>
__device__ __forceinline__ f32x4 mfma16(typename Prec<F>::Op a, typename Prec<F>::Op b, f32x4 c) {
    return Prec<F>::mfma(a, b, c);
}

// A operand: 16x16 tile of a row-major matrix M (row stride ld), rows r0..,
// columns c0..: lane l reads M[r0 + l%16][c0 + 4(l/16) .. +3] (M and ld
// multiples of 4 elements: one 8- or 16-byte read).
template <bool F>
__device__ __forceinline__ typename Prec<F>::Op load_a(const typename Prec<F>::W *M, int ld,
                                                       int r0, int c0, int l) {
    return *(const typename Prec<F>::Op *)(M + (r0 + (l & 15)) * ld + c0 + 4 * (l >> 4));
}
// A operand of the transpose: A[i][k] = M[k][i], i.e. lane l reads
// M[c0 + 4(l/16) + j][r0 + l%16], j = 0..3.
template <bool F>
__device__ __forceinline__ typename Prec<F>::Op load_at(const typename Prec<F>::W *M, int ld,
                                                        int r0, int c0, int l) {
    typename Prec<F>::Op v;
    int i = r0 + (l & 15), k = c0 + 4 * (l >> 4);
    for (int r = 0; r < 4; r++) Prec<F>::set(v, r, M[(k + r) * ld + i]);
    return v;
}
template <bool F>
__device__ __forceinline__ typename Prec<F>::Op to_op(f32x4 x) {
    typename Prec<F>::Op v;
    for (int r = 0; r < 4; r++) Prec<F>::set(v, r, Prec<F>::store(x[r]));
    return v;
}

template <bool F>
struct Fwd {
    f32x4 z1[4], z2[4], z3[4];   // pre-activations, blocks of 16 features
    typename Prec<F>::Op x;      // input operand (BF16: hi/lo halves; FP32: x, 0)
    f32x4 y;                     // outputs (rows 0..2 valid in lanes 0..15)
};

// input operand of the samples s0 .. s0+15: lanes 0..31 carry features 0..7,
// lanes 32..63 (the duplicated columns of W1p) the BF16 remainder x - hi, or
// zero in FP32
template <bool F>
__device__ __forceinline__ typename Prec<F>::Op input_op(const float *__restrict__ X, int64_t B,
                                                         int64_t s0, int l) {
    const int g = l >> 4;
    const int64_t s = s0 + (l & 15);
    float xv[4] = {0.f, 0.f, 0.f, 0.f};
    if (s < B) {
        const float *xs = X + 8 * s + 4 * (g & 1);
        for (int r = 0; r < 4; r++) {
            const float v = xs[r];
            if (F) {
                xv[r] = (g < 2) ? v : 0.f;
            } else {
                const float hi = bf2f(f2bf(v));
                xv[r] = (g < 2) ? hi : v - hi;
            }
        }
    }
    typename Prec<F>::Op x;
    for (int r = 0; r < 4; r++) Prec<F>::set(x, r, Prec<F>::store(xv[r]));
    return x;
}

// forward pass for samples s0 .. s0+15 (tail masked by B)
template <bool F>
__device__ __forceinline__ void mlp_tile_forward(const typename Prec<F>::W *W, const float *b,
                                                 const float *__restrict__ X, int64_t B,
                                                 int64_t s0, int l, Fwd<F> &f) {
    const int g = l >> 4;
    f.x = input_op<F>(X, B, s0, l);
    typename Prec<F>::Op h[4];
    for (int ob = 0; ob < 4; ob++) {
        f32x4 acc;
        for (int r = 0; r < 4; r++) acc[r] = b[kB1 + 16 * ob + 4 * g + r];
        acc = mfma16<F>(load_a<F>(W + kL1, kLd1, 16 * ob, 0, l), f.x, acc);
        f.z1[ob] = acc;
    }
    for (int ob = 0; ob < 4; ob++) {
        f32x4 a = f.z1[ob];
        for (int r = 0; r < 4; r++) a[r] = silu(a[r]);
        h[ob] = to_op<F>(a);
    }
    for (int ob = 0; ob < 4; ob++) {
        f32x4 acc;
        for (int r = 0; r < 4; r++) acc[r] = b[kB2 + 16 * ob + 4 * g + r];
        for (int kb = 0; kb < 4; kb++) acc = mfma16<F>(load_a<F>(W + kL2, kLd, 16 * ob, 16 * kb, l), h[kb], acc);
        f.z2[ob] = acc;
    }
    for (int ob = 0; ob < 4; ob++) {
        f32x4 a = f.z2[ob];
        for (int r = 0; r < 4; r++) a[r] = silu(a[r]);
        h[ob] = to_op<F>(a);
    }
    for (int ob = 0; ob < 4; ob++) {
        f32x4 acc;
        for (int r = 0; r < 4; r++) acc[r] = b[kB3 + 16 * ob + 4 * g + r];
        for (int kb = 0; kb < 4; kb++) acc = mfma16<F>(load_a<F>(W + kL3, kLd, 16 * ob, 16 * kb, l), h[kb], acc);
        f.z3[ob] = acc;
    }
    for (int ob = 0; ob < 4; ob++) {
        f32x4 a = f.z3[ob];
        for (int r = 0; r < 4; r++) a[r] = silu(a[r]);
        h[ob] = to_op<F>(a);
    }
    f32x4 acc;
    for (int r = 0; r < 4; r++) acc[r] = b[kB4p + 4 * g + r];
    for (int kb = 0; kb < 4; kb++) acc = mfma16<F>(load_a<F>(W + kL4, kLd, 0, 16 * kb, l), h[kb], acc);
    f.y = acc;
}

// weights (16 bytes at a time; rows of 16 in W1p, of 64 in the others) and
// biases into LDS
template <typename WT>
__device__ __forceinline__ void load_weights_lds(const WT *__restrict__ wg,
                                                 const float *__restrict__ bg, WT *W, float *b) {
    typedef WT V4 __attribute__((ext_vector_type(4)));
    constexpr int E = 16 / (int)sizeof(WT);   // elements per 16 bytes
    struct V16 { V4 v[E / 4]; };
    const V16 *src = (const V16 *)wg;
    for (int i = threadIdx.x; i < kWpad / E; i += blockDim.x) {
        const int e = i * E;
        const V16 v = src[i];
        const int at = e < kW2 ? (e >> 4) * kLd1 + (e & 15)
                               : kL2 + ((e - kW2) >> 6) * kLd + ((e - kW2) & 63);
#pragma unroll
        for (int k = 0; k < E / 4; k++) *(V4 *)(W + at + 4 * k) = v.v[k];
    }
    for (int i = threadIdx.x; i < kBpad; i += blockDim.x) b[i] = bg[i];
}

// ------------------------------------------------------------- inference
// The same arithmetic as mlp_tile_forward, with every weight operand and
// bias of the network held in registers across the wavefront's tiles (40
// A operands and 13 bias blocks, read from LDS once): a tile then costs its
// 40 MFMAs, 192 SiLUs per sample and the input and output accesses only (1e6
// samples in 74 us).
template <bool F>
__global__ __launch_bounds__(256) void k_mlp_infer(int64_t B, const int *__restrict__ Bdev,
                                                   const float *__restrict__ X,
                                                   const typename Prec<F>::W *__restrict__ wg,
                                                   const float *__restrict__ bg,
                                                   float *__restrict__ Y) {
    typedef typename Prec<F>::Op Op;
    __shared__ __attribute__((aligned(16))) typename Prec<F>::W W[kLpad];
    __shared__ float b[kBpad];
    if (Bdev) B = *Bdev;
    // a workgroup without a tile returns before staging the weights (the
    // launch is sized for the largest count; the device-side one is often
    // far smaller, or zero)
    if ((int64_t)blockIdx.x * (blockDim.x >> 6) >= (B + 15) / 16) return;
    load_weights_lds(wg, bg, W, b);
    __syncthreads();
    const int l = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int g = l >> 4;
    Op A1[4], A2[4][4], A3[4][4], A4[4];
    f32x4 C1[4], C2[4], C3[4], C4;
#pragma unroll
    for (int ob = 0; ob < 4; ob++) {
        A1[ob] = load_a<F>(W + kL1, kLd1, 16 * ob, 0, l);
        A4[ob] = load_a<F>(W + kL4, kLd, 0, 16 * ob, l);
#pragma unroll
        for (int kb = 0; kb < 4; kb++) {
            A2[ob][kb] = load_a<F>(W + kL2, kLd, 16 * ob, 16 * kb, l);
            A3[ob][kb] = load_a<F>(W + kL3, kLd, 16 * ob, 16 * kb, l);
        }
#pragma unroll
        for (int r = 0; r < 4; r++) {
            C1[ob][r] = b[kB1 + 16 * ob + 4 * g + r];
            C2[ob][r] = b[kB2 + 16 * ob + 4 * g + r];
            C3[ob][r] = b[kB3 + 16 * ob + 4 * g + r];
        }
    }
#pragma unroll
    for (int r = 0; r < 4; r++) C4[r] = b[kB4p + 4 * g + r];
    const int64_t ntiles = (B + 15) / 16;
    for (int64_t t = (int64_t)blockIdx.x * nw + wave; t < ntiles; t += (int64_t)gridDim.x * nw) {
        const int64_t s = 16 * t + (l & 15);
        const Op x = input_op<F>(X, B, 16 * t, l);
        Op h[4], hn[4];
#pragma unroll
        for (int ob = 0; ob < 4; ob++) {
            f32x4 a = mfma16<F>(A1[ob], x, C1[ob]);
#pragma unroll
            for (int r = 0; r < 4; r++) a[r] = silu(a[r]);
            h[ob] = to_op<F>(a);
        }
#pragma unroll
        for (int ob = 0; ob < 4; ob++) {
            f32x4 acc = C2[ob];
#pragma unroll
            for (int kb = 0; kb < 4; kb++) acc = mfma16<F>(A2[ob][kb], h[kb], acc);
#pragma unroll
            for (int r = 0; r < 4; r++) acc[r] = silu(acc[r]);
            hn[ob] = to_op<F>(acc);
        }
#pragma unroll
        for (int ob = 0; ob < 4; ob++) {
            f32x4 acc = C3[ob];
#pragma unroll
            for (int kb = 0; kb < 4; kb++) acc = mfma16<F>(A3[ob][kb], hn[kb], acc);
#pragma unroll
            for (int r = 0; r < 4; r++) acc[r] = silu(acc[r]);
            h[ob] = to_op<F>(acc);
        }
        f32x4 y = C4;
#pragma unroll
        for (int kb = 0; kb < 4; kb++) y = mfma16<F>(A4[kb], h[kb], y);
        if (g == 0 && s < B)
            for (int r = 0; r < 3; r++) Y[3 * s + r] = y[r];
    }
}

// ------------------------------------------------------------- training
// A workgroup of NW wavefronts takes 16 NW samples at a time, each wavefront
// the forward and backward chains of 16.  Both factors of a layer's dW = dZ^T H
// go through LDS transposed ([feature][sample], so that an operand is one
// read), and the wavefronts share the products by output blocks, which they
// accumulate in registers over all the workgroup's samples.  Bias gradients are
// summed per lane and reduced once.  Bound by latency at the training batch of
// 8192 samples (128 workgroups): 14 us, and 4 for the reduction (one wavefront per
// workgroup with its gradient in LDS, bias sums by shuffles and unaligned operand
// reads took 56, the reduction over 512 partials 32, a fold and two copies 14).
template <bool F> constexpr int train_waves() { return F ? 2 : 4; }
template <bool F> constexpr int tile_ld() { return 16 * train_waves<F>() + 4; }

// store a D-layout block (features 16 ob + 4 g + r of sample l % 16 of the
// wavefront) into a [feature][sample] tile
template <bool F>
__device__ __forceinline__ void store_tile(typename Prec<F>::W *T, int ob, f32x4 v, int s, int g) {
#pragma unroll
    for (int r = 0; r < 4; r++) T[(16 * ob + 4 * g + r) * tile_ld<F>() + s] = Prec<F>::store(v[r]);
}

// acc += block (ob, ib) of dZ^T H over the workgroup's samples
template <bool F>
__device__ __forceinline__ f32x4 acc_dw(const typename Prec<F>::W *Tz, int ob,
                                        const typename Prec<F>::W *Th, int ib, f32x4 acc, int l) {
#pragma unroll
    for (int st = 0; st < train_waves<F>(); st++)
        acc = mfma16<F>(load_a<F>(Tz, tile_ld<F>(), 16 * ob, 16 * st, l),
                        load_a<F>(Th, tile_ld<F>(), 16 * ib, 16 * st, l), acc);
    return acc;
}

// sum of a lane's value over its row of 16 lanes, in the row's last lane
__device__ __forceinline__ float row_sum15(float v) {
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x118, 0xf, 0xf, true));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x114, 0xf, 0xf, true));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x112, 0xf, 0xf, true));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x111, 0xf, 0xf, true));
    return v;
}

template <bool F>
__global__ __launch_bounds__(64 * train_waves<F>()) void k_mlp_train(
    int64_t B, const float *__restrict__ X, const float *__restrict__ T, float scale,
    const typename Prec<F>::W *__restrict__ wg, const float *__restrict__ bg,
    float *__restrict__ partial, float *__restrict__ loss_partial) {
    typedef typename Prec<F>::W WT;
    constexpr int NW = train_waves<F>(), PB = 4 / NW;   // output blocks of a row per wavefront
    __shared__ __attribute__((aligned(16))) WT W[kLpad];
    __shared__ __attribute__((aligned(16))) WT Tz[64 * tile_ld<F>()], Th[64 * tile_ld<F>()];
    __shared__ float b[kBpad], dbs[NW][kBpad];
    load_weights_lds(wg, bg, W, b);
    __syncthreads();
    const int l = threadIdx.x & 63, wave = threadIdx.x >> 6, g = l >> 4, ts = 16 * wave + (l & 15);
    const int64_t ntiles = (B + 16 * NW - 1) / (16 * NW);
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    // dW blocks: layers 3, 2: rows ob = wave PB + p; layer 4: columns; layer 1: rows
    f32x4 g3[PB][4], g2[PB][4], g4[PB], g1[PB], db1[4], db2[4], db3[4], db4 = zero;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        db1[i] = db2[i] = db3[i] = zero;
#pragma unroll
        for (int p = 0; p < PB; p++) g3[p][i] = g2[p][i] = zero;
    }
#pragma unroll
    for (int p = 0; p < PB; p++) g4[p] = g1[p] = zero;
    float lsum = 0.f;
    // dZ of the layer below: (W^T dZ) * silu'(z)
    auto back = [&](int woff, int nk, const f32x4 (&zp)[4], f32x4 (&dz)[4]) {
        typename Prec<F>::Op dzb[4];
#pragma unroll
        for (int k = 0; k < 4; k++)
            if (k < nk) dzb[k] = to_op<F>(dz[k]);
#pragma unroll
        for (int ob = 0; ob < 4; ob++) {
            f32x4 acc = zero;
#pragma unroll
            for (int k = 0; k < 4; k++)
                if (k < nk) acc = mfma16<F>(load_at<F>(W + woff, kLd, 16 * ob, 16 * k, l), dzb[k], acc);
#pragma unroll
            for (int r = 0; r < 4; r++) acc[r] *= dsilu(zp[ob][r]);
            dz[ob] = acc;
        }
    };
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        Fwd<F> f;
        const int64_t s0 = 16 * NW * t + 16 * wave, s = s0 + (l & 15);
        mlp_tile_forward<F>(W, b, X, B, s0, l, f);
        const bool valid = s < B;
        auto store_h = [&](const f32x4 (&z)[4]) {
#pragma unroll
            for (int ob = 0; ob < 4; ob++) {
                f32x4 h = z[ob];
#pragma unroll
                for (int r = 0; r < 4; r++) h[r] = valid ? silu(h[r]) : 0.f;
                store_tile<F>(Th, ob, h, ts, g);
            }
        };
        // dZ4 = (y - t) * scale on rows 0..2
        f32x4 dz[4] = {zero, zero, zero, zero};
        if (g == 0 && valid)
#pragma unroll
            for (int r = 0; r < 3; r++) {
                const float d = f.y[r] - T[3 * s + r];
                lsum += 0.5f * d * d * scale;
                dz[0][r] = d * scale;
            }
        db4 += dz[0];
        store_h(f.z3);
        store_tile<F>(Tz, 0, dz[0], ts, g);
        __syncthreads();
#pragma unroll
        for (int p = 0; p < PB; p++) g4[p] = acc_dw<F>(Tz, 0, Th, wave * PB + p, g4[p], l);
        back(kL4, 1, f.z3, dz);
        __syncthreads();
        auto layer = [&](const f32x4 (&z)[4], f32x4 (&db)[4], f32x4 (&gw)[PB][4]) {
            store_h(z);
#pragma unroll
            for (int ob = 0; ob < 4; ob++) {
                db[ob] += dz[ob];
                store_tile<F>(Tz, ob, dz[ob], ts, g);
            }
            __syncthreads();
#pragma unroll
            for (int p = 0; p < PB; p++)
#pragma unroll
                for (int ib = 0; ib < 4; ib++)
                    gw[p][ib] = acc_dw<F>(Tz, wave * PB + p, Th, ib, gw[p][ib], l);
        };
        layer(f.z2, db3, g3);
        back(kL3, 4, f.z2, dz);
        __syncthreads();
        layer(f.z1, db2, g2);
        back(kL2, 4, f.z1, dz);
        __syncthreads();
        // layer 1: dW1p (64 x 16) += dZ1^T Xp
#pragma unroll
        for (int r = 0; r < 4; r++) Th[(4 * g + r) * tile_ld<F>() + ts] = (WT)f.x[r];
#pragma unroll
        for (int ob = 0; ob < 4; ob++) {
            db1[ob] += dz[ob];
            store_tile<F>(Tz, ob, dz[ob], ts, g);
        }
        __syncthreads();
#pragma unroll
        for (int p = 0; p < PB; p++) g1[p] = acc_dw<F>(Tz, wave * PB + p, Th, 0, g1[p], l);
        __syncthreads();
    }
    // element r of a block: row 4 g + r, column l % 16
    float *out = partial + (size_t)blockIdx.x * kGpad;
    const int c = l & 15;
#pragma unroll
    for (int p = 0; p < PB; p++) {
        const int ob = wave * PB + p;
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int row = 16 * ob + 4 * g + r;
            out[kW1p + row * 16 + c] = g1[p][r];
            out[kW4p + (4 * g + r) * 64 + 16 * ob + c] = g4[p][r];
#pragma unroll
            for (int ib = 0; ib < 4; ib++) {
                out[kW2 + row * 64 + 16 * ib + c] = g2[p][ib][r];
                out[kW3 + row * 64 + 16 * ib + c] = g3[p][ib][r];
            }
        }
    }
#pragma unroll
    for (int r = 0; r < 4; r++) {
#pragma unroll
        for (int ob = 0; ob < 4; ob++) {
            const float v1 = row_sum15(db1[ob][r]), v2 = row_sum15(db2[ob][r]),
                        v3 = row_sum15(db3[ob][r]);
            if (c == 15) {
                dbs[wave][kB1 + 16 * ob + 4 * g + r] = v1;
                dbs[wave][kB2 + 16 * ob + 4 * g + r] = v2;
                dbs[wave][kB3 + 16 * ob + 4 * g + r] = v3;
            }
        }
        const float v4 = row_sum15(db4[r]);
        if (c == 15) dbs[wave][kB4p + 4 * g + r] = v4;
    }
    for (int m = 1; m < 64; m <<= 1) lsum += __shfl_xor(lsum, m, 64);
    if (l == 0) b[wave] = lsum;   // the biases are no longer read
    __syncthreads();
    for (int i = threadIdx.x; i < kBpad; i += blockDim.x) {
        float v = dbs[0][i];
        for (int w = 1; w < NW; w++) v += dbs[w][i];
        out[kWpad + i] = v;
    }
    if (threadIdx.x == 0) {
        float v = b[0];
        for (int w = 1; w < NW; w++) v += b[w];
        loss_partial[blockIdx.x] = v;
    }
}

// Sum of the workgroup partials in a fixed order: block j < kGpad / 64 owns
// 64 consecutive entries of the padded gradient image; its 4 thread groups
// sum 4 contiguous quarters of the partials (coalesced rows, eight loads in
// flight) and the quarter sums are added in order.  The entries of the master
// layout go to grad (W1's two copies of a column added), or, with ADAM, into
// the Adam step: moments, parameters and the kernels' padded images.  The extra
// last block sums the loss partials (fixed per-thread strides, then a fixed
// tree).
constexpr int kRedCols = 64;
constexpr int kRedBlocks = (kGpad + kRedCols - 1) / kRedCols;
static_assert(kGpad == kRedCols * kRedBlocks - 48, "the last block is cut short");

struct AdamArgs {
    float *P, *m, *v, *wf, *bg;
    unsigned short *wg;
    float lr, b1, b2, eps, c1, c2;
};

// master index of padded entry i, or -1 (padding, and W1's second copy)
__device__ __forceinline__ int master_index(int i) {
    if (i < kW2) return (i & 15) < 8 ? (i >> 4) * 8 + (i & 15) : -1;
    if (i < kW3) return 576 + (i - kW2);
    if (i < kW4p) return 4736 + (i - kW3);
    if (i < kWpad) return i - kW4p < 192 ? 8896 + (i - kW4p) : -1;
    const int j = i - kWpad;
    if (j < kB2) return 512 + j;
    if (j < kB3) return 4672 + (j - kB2);
    if (j < kB4p) return 8832 + (j - kB3);
    return j - kB4p < 3 ? 9088 + (j - kB4p) : -1;
}

__device__ __forceinline__ void sum_loss(int nb, const float *__restrict__ loss_partial, float *sh,
                                         float *__restrict__ loss) {
    const int t = threadIdx.x;
    float s = 0.f;
    for (int k = t; k < nb; k += 256) s += loss_partial[k];
    sh[t] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (t < o) sh[t] += sh[t + o];
        __syncthreads();
    }
    if (t == 0) *loss = sh[0];
}

__global__ __launch_bounds__(256) void k_mlp_loss(int nb, const float *__restrict__ loss_partial,
                                                  float *__restrict__ loss) {
    __shared__ float sh[256];
    sum_loss(nb, loss_partial, sh, loss);
}

template <bool ADAM>
__global__ __launch_bounds__(256) void k_mlp_reduce(int nb, const float *__restrict__ partial,
                                                   const float *__restrict__ loss_partial,
                                                   float *__restrict__ grad,
                                                   float *__restrict__ loss, AdamArgs A) {
    __shared__ float sh[256], tot[64];
    const int t = threadIdx.x;
    if (blockIdx.x == kRedBlocks) {
        if (loss) sum_loss(nb, loss_partial, sh, loss);
        return;
    }
    const int c = t % kRedCols, g = t / kRedCols;
    const int i = blockIdx.x * kRedCols + c;
    const int q = (nb + 3) / 4, k0 = g * q, k1 = k0 + q < nb ? k0 + q : nb;
    float s = 0.f;
    if (i < kGpad) {
#pragma unroll 8
        for (int k = k0; k < k1; k++) s += partial[(size_t)k * kGpad + i];
    }
    sh[t] = s;
    __syncthreads();
    if (g == 0) tot[c] = (sh[c] + sh[64 + c]) + (sh[128 + c] + sh[192 + c]);
    __syncthreads();
    if (g != 0 || i >= kGpad) return;
    const int j = master_index(i);
    if (j < 0) return;
    const float v = i < kW2 ? tot[c] + tot[c + 8] : tot[c];
    if constexpr (!ADAM) {
        grad[j] = v;
    } else {
        const float mi = A.b1 * A.m[j] + (1.f - A.b1) * v;
        const float vi = A.b2 * A.v[j] + (1.f - A.b2) * v * v;
        A.m[j] = mi;
        A.v[j] = vi;
        const float p = A.P[j] - A.lr * (mi / A.c1) / (sqrtf(vi / A.c2) + A.eps);
        A.P[j] = p;
        if (i < kWpad) {
            A.wg[i] = f2bf(p);
            A.wf[i] = p;
            if (i < kW2) {
                A.wg[i + 8] = f2bf(p);
                A.wf[i + 8] = p;
            }
        } else {
            A.bg[i - kWpad] = p;
        }
    }
}

// master FP32 -> padded BF16 weights (and the same image in FP32, for the
// FP32 debug mode) + FP32 biases
__global__ void k_mlp_pack(const float *__restrict__ P, unsigned short *__restrict__ wg,
                           float *__restrict__ wf, float *__restrict__ bg) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kWpad) {
        float v = 0.f;
        if (i < kW2) { int o = i / 16, c = i % 16; v = P[o * 8 + (c & 7)]; }
        else if (i < kW3) v = P[576 + (i - kW2)];
        else if (i < kW4p) v = P[4736 + (i - kW3)];
        else { int o = (i - kW4p) / 64, c = (i - kW4p) % 64; v = o < 3 ? P[8896 + o * 64 + c] : 0.f; }
        wg[i] = f2bf(v);
        wf[i] = v;
    }
    if (i < kBpad) {
        float v;
        if (i < 64) v = P[512 + i];
        else if (i < 128) v = P[4672 + i - 64];
        else if (i < 192) v = P[8832 + i - 128];
        else v = (i - 192) < 3 ? P[9088 + i - 192] : 0.f;
        bg[i] = v;
    }
}

}  // namespace bs

// ------------------------------------------------------------------ C ABI
using namespace bs;

struct bs_mlp_s {
    hipStream_t stream = nullptr;
    float *P = nullptr, *m = nullptr, *v = nullptr;
    unsigned short *wg = nullptr;
    float *wf = nullptr;     // FP32 image of the padded weights (debug mode)
    float *bg = nullptr;
    int fp32 = 0;            // 1: FP32 weights and activations (debug mode)
    float *partial = nullptr, *loss_partial = nullptr;
    int nb = 256;            // workgroups of a training pass, at most (one per CU)
    int64_t step = 0;
    std::string err;
};

namespace bs {
hipStream_t mlp_stream(bs_mlp_t M) { return M->stream; }
int mlp_fp32(bs_mlp_t M) { return M ? M->fp32 : 0; }

void mlp_forward_device(bs_mlp_t M, const int *Bdev, int64_t Bmax, const float *X, float *Y,
                        hipStream_t stream) {
    int64_t tiles = (Bmax + 15) / 16;
    int blocks = (int)std::min<int64_t>(std::max<int64_t>((tiles + 3) / 4, 1), 2048);
    if (M->fp32)
        hipLaunchKernelGGL(k_mlp_infer<true>, dim3(blocks), dim3(256), 0, stream, Bmax, Bdev, X,
                           (const float *)M->wf, M->bg, Y);
    else
        hipLaunchKernelGGL(k_mlp_infer<false>, dim3(blocks), dim3(256), 0, stream, Bmax, Bdev, X,
                           (const unsigned short *)M->wg, M->bg, Y);
}
}  // namespace bs

extern "C" {

int bs_mlp_nparams(void) { return kNP; }

int bs_mlp_create(const float *params_host, void *hip_stream, bs_mlp_t *out) {
    if (!out || !params_host) return BS_EINVAL;
    bs_mlp_t M = new bs_mlp_s();
    M->stream = (hipStream_t)hip_stream;
    hipError_t e = hipSuccess;
    auto al = [&](void **p, size_t bytes) { if (e == hipSuccess) e = hipMalloc(p, bytes); };
    al((void **)&M->P, kNP * 4); al((void **)&M->m, kNP * 4); al((void **)&M->v, kNP * 4);
    al((void **)&M->wg, kWpad * 2); al((void **)&M->bg, kBpad * 4);
    al((void **)&M->wf, kWpad * 4);
    al((void **)&M->partial, (size_t)M->nb * kGpad * 4);
    al((void **)&M->loss_partial, M->nb * 4);
    if (e != hipSuccess) { bs_mlp_destroy(M); return BS_ENOMEM; }
    (void)hipMemcpy(M->P, params_host, kNP * 4, hipMemcpyHostToDevice);
    (void)hipMemset(M->m, 0, kNP * 4);
    (void)hipMemset(M->v, 0, kNP * 4);
    hipLaunchKernelGGL(k_mlp_pack, dim3(ceil_div(kWpad, 256)), dim3(256), 0, M->stream, M->P,
                       M->wg, M->wf, M->bg);
    *out = M;
    return hipGetLastError() == hipSuccess ? BS_OK : BS_EDEVICE;
}

int bs_mlp_forward(bs_mlp_t M, int64_t B, const float *X, float *Y) {
    if (!M || B < 0 || (B > 0 && (!X || !Y))) return BS_EINVAL;
    if (B == 0) return BS_OK;
    int64_t tiles = (B + 15) / 16;
    int blocks = (int)std::min<int64_t>((tiles + 3) / 4, 4096);
    if (M->fp32)
        hipLaunchKernelGGL(k_mlp_infer<true>, dim3(blocks), dim3(256), 0, M->stream, B,
                           (const int *)nullptr, X, (const float *)M->wf, M->bg, Y);
    else
        hipLaunchKernelGGL(k_mlp_infer<false>, dim3(blocks), dim3(256), 0, M->stream, B,
                           (const int *)nullptr, X, (const unsigned short *)M->wg, M->bg, Y);
    return hipGetLastError() == hipSuccess ? BS_OK : BS_EDEVICE;
}

// the workgroup partials of the loss and its gradient; their number
static int mlp_partials(bs_mlp_t M, int64_t B, const float *X, const float *T) {
    const int waves = M->fp32 ? train_waves<true>() : train_waves<false>();
    const int64_t tiles = (B + 16 * waves - 1) / (16 * waves);
    const int blocks = (int)std::min<int64_t>(tiles, M->nb);
    if (M->fp32)
        hipLaunchKernelGGL(k_mlp_train<true>, dim3(blocks), dim3(64 * waves), 0, M->stream, B, X, T,
                           1.0f / (float)B, (const float *)M->wf, M->bg, M->partial,
                           M->loss_partial);
    else
        hipLaunchKernelGGL(k_mlp_train<false>, dim3(blocks), dim3(64 * waves), 0, M->stream, B, X,
                           T, 1.0f / (float)B, (const unsigned short *)M->wg, M->bg, M->partial,
                           M->loss_partial);
    return blocks;
}

int bs_mlp_loss_grad(bs_mlp_t M, int64_t B, const float *X, const float *T, float *loss_dev,
                     float *grad_dev) {
    if (!M || B <= 0 || !X || !T) return BS_EINVAL;
    if (!loss_dev && !grad_dev) return BS_OK;
    const int blocks = mlp_partials(M, B, X, T);
    if (hipGetLastError() != hipSuccess) return BS_EDEVICE;
    AdamArgs A{};
    if (grad_dev)
        hipLaunchKernelGGL(k_mlp_reduce<false>, dim3(kRedBlocks + 1), dim3(256), 0, M->stream,
                           blocks, M->partial, M->loss_partial, grad_dev, loss_dev, A);
    else
        hipLaunchKernelGGL(k_mlp_loss, dim3(1), dim3(256), 0, M->stream, blocks, M->loss_partial,
                           loss_dev);
    return hipGetLastError() == hipSuccess ? BS_OK : BS_EDEVICE;
}

int bs_mlp_adam_step(bs_mlp_t M, int64_t B, const float *X, const float *T, float lr,
                     float beta1, float beta2, float eps, float *loss_dev) {
    if (!M || B <= 0 || !X || !T) return BS_EINVAL;
    const int blocks = mlp_partials(M, B, X, T);
    if (hipGetLastError() != hipSuccess) return BS_EDEVICE;   // no step was taken
    M->step++;
    AdamArgs A;
    A.P = M->P; A.m = M->m; A.v = M->v; A.wf = M->wf; A.bg = M->bg; A.wg = M->wg;
    A.lr = lr; A.b1 = beta1; A.b2 = beta2; A.eps = eps;
    A.c1 = 1.f - powf(beta1, (float)M->step);
    A.c2 = 1.f - powf(beta2, (float)M->step);
    hipLaunchKernelGGL(k_mlp_reduce<true>, dim3(kRedBlocks + 1), dim3(256), 0, M->stream, blocks,
                       M->partial, M->loss_partial, (float *)nullptr, loss_dev, A);
    return hipGetLastError() == hipSuccess ? BS_OK : BS_EDEVICE;
}

int bs_mlp_set_fp32(bs_mlp_t M, int enable) {
    if (!M) return BS_EINVAL;
    M->fp32 = enable ? 1 : 0;
    return BS_OK;
}

int bs_mlp_get_params(bs_mlp_t M, float *params_host) {
    if (!M || !params_host) return BS_EINVAL;
    (void)hipStreamSynchronize(M->stream);
    return hipMemcpy(params_host, M->P, kNP * 4, hipMemcpyDeviceToHost) == hipSuccess ? BS_OK
                                                                                   : BS_EDEVICE;
}

int bs_mlp_destroy(bs_mlp_t M) {
    if (!M) return BS_OK;
    (void)hipStreamSynchronize(M->stream);
    void *all[] = {M->P, M->m, M->v, M->wg, M->wf, M->bg, M->partial, M->loss_partial};
    for (void *p : all)
        if (p) (void)hipFree(p);
    delete M;
    return BS_OK;
}

}  // extern "C"
