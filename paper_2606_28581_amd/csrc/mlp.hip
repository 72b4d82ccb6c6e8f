// Learned sun-visibility surrogate on gfx950 MFMA (not in the paper; a stand-in for the
// geometric shadow pass of Sec. 3.1 / 3.3, trained on that pass's labels).
//
// Network: Fourier features of the normalised surfel centre (16 frequencies x sin/cos
// x 3 coordinates) + (cos phi, sin phi, sin theta, cos theta) padded to 128, then
// 128 -> 64 -> 64 -> 64 (ReLU) -> 1.  BF16 weights and activations, FP32 accumulation
// with v_mfma_f32_16x16x32_bf16.  Parameters are one FP32 master vector
// [W1 (64x128), b1, W2 (64x64), b2, W3 (64x64), b3, w4 (64), b4].
//
// Forward: one wave step owns 64 points (four 16-point MFMA tiles, so that every weight
// fragment read from LDS feeds four independent accumulation chains).  Each lane computes
// exactly the 8 features its operand needs (point l%16, features 32 ks + 8 (l/16) .. +7),
// so the 96 sin/cos values of a point are spread over 4 lanes with no duplication and no
// LDS staging; the layers are computed transposed so that hidden activations stay in
// registers (see k_mlp_forward).  Weights live in LDS, row-major [out][in], so a weight
// operand is 16 contiguous bytes.  Training is one kernel that runs forward and backward
// of 128 points per block step (see k_mlp_train) and one that sums its partial gradients.
#include "ss_internal.h"
#include "ss_mlp.h"

namespace ss {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16;

// the forward takes kFwdPT tiles of 16 points per wave step: each weight fragment read
// from LDS feeds kFwdPT independent MFMA chains
constexpr int kFwdPT = 4;
constexpr int kFwdPts = 16 * kFwdPT;
constexpr int kMlpThreads = 256;
constexpr int kMlpWaves = kMlpThreads / 64;

// FP32 -> BF16, round to nearest even (gfx950 converts in hardware, two values per
// instruction when the compiler pairs them)
__device__ __forceinline__ u16 f2bf(float x)
{
    const __bf16 h = (__bf16)x;
    return __builtin_bit_cast(u16, h);
}
__device__ __forceinline__ float bf2f(u16 b) { return __uint_as_float((uint32_t)b << 16); }

union Frag {
    bf16x8 v;
    u16 h[8];
    uint4 q;
};

__device__ __forceinline__ f32x4 mfma(const Frag &a, const Frag &b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, c, 0, 0, 0);
}

// --------------------------------------------------------------- weight prep
// FP32 master -> BF16 copies (W1, W2, W3, w4) and FP32 biases, in the MLP workspace.
__global__ void k_mlp_prep(const float *__restrict__ w, u16 *__restrict__ wb, float *__restrict__ wf)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kMlpW1 + kMlpW2 + kMlpW3 + kMlpWidth) {
        int src;
        if (i < kMlpW1) src = kOffW1 + i;
        else if (i < kMlpW1 + kMlpW2) src = kOffW2 + (i - kMlpW1);
        else if (i < kMlpW1 + kMlpW2 + kMlpW3) src = kOffW3 + (i - kMlpW1 - kMlpW2);
        else src = kOffW4 + (i - kMlpW1 - kMlpW2 - kMlpW3);
        wb[i] = f2bf(w[src]);
    }
    if (i < 3 * kMlpWidth + 1) {
        int src = i < 64 ? kOffB1 + i : i < 128 ? kOffB2 + i - 64 : i < 192 ? kOffB3 + i - 128 : kOffB4;
        wf[i] = w[src];
    }
}

// Feature chunk of one lane for the k-step ks < 3 (coordinate ks of the point p_hat) and
// lane group g: 8 bf16 values, features 32 ks + 8 g .. + 7.
__device__ __forceinline__ void feature_chunk(float p_hat, int g, Frag &out)
{
    // frequency 4 g from the hardware sine and cosine: x = x0 2^(4g) is exact (a
    // power-of-two scaling), r = x - 2 rint(x / 2) in [-1, 1] too, and their argument
    // is in revolutions (r / 2, exact); frequencies 4 g + 1 .. 4 g + 3 by the double
    // angle, sin 2a = 2 sin a cos a, cos 2a = 1 - 2 sin^2 a, which grows the error at
    // most eightfold, still far below the BF16 rounding that follows
    const float x = p_hat * (float)(1u << (4 * g));
    const float r = x - 2.f * rintf(0.5f * x);
    float s = __builtin_amdgcn_sinf(0.5f * r);
    float c = __builtin_amdgcn_cosf(0.5f * r);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        out.h[2 * q] = f2bf(s);
        out.h[2 * q + 1] = f2bf(c);
        if (q < 3) {
            const float s2 = 2.f * s * c;
            c = __fmaf_rn(-2.f * s, s, 1.f);
            s = s2;
        }
    }
}

// The last k-step: features 96 .. 99 are the sun's (cos phi, sin phi, sin theta, cos theta)
// in lane group 0, the rest of the 128 is zero padding.  Angles go through the hardware
// sine and cosine (argument in revolutions).
__device__ __forceinline__ void sun_chunk(float phi, float theta, int g, Frag &out)
{
    constexpr float kRev = 0.15915494309189535f;   // 1 / (2 pi)
    phi *= kRev;
    theta *= kRev;
    out.q = make_uint4(0, 0, 0, 0);
    if (g == 0) {
        out.h[0] = f2bf(__builtin_amdgcn_cosf(phi));
        out.h[1] = f2bf(__builtin_amdgcn_sinf(phi));
        out.h[2] = f2bf(__builtin_amdgcn_sinf(theta));
        out.h[3] = f2bf(__builtin_amdgcn_cosf(theta));
    }
}

// Forward, transposed: every layer computes C^T = W X^T (rows = neurons, columns =
// points), so lane l of an accumulator tile holds neurons 4 (l / 16) + 0..3 of point
// l % 16 - four consecutive neurons of one point.  The next layer's B operand needs 8
// consecutive inputs of one point per lane; numbering that layer's inputs so that its
// k-step ks, lane group q, element e is neuron 16 (2 ks + e / 4) + 4 q + e % 4 (the
// columns of W2 and W3 are permuted once when they are copied to LDS) makes those 8 the
// lane's own accumulator values of tiles 2 ks and 2 ks + 1.  Hidden activations never
// leave registers.  Features are computed directly in the B layout (point l % 16,
// features 32 ks + 8 (l / 16) .. + 7), as for the first layer.
// A weight operand read takes 16 rows at one column: at the plain strides of 256 and 128
// bytes all 16 lie on the same LDS banks, so rows are padded by 16 bytes, which spreads
// them over all 64 banks (20M points: 0.727 -> 0.688 ms for the whole network pass).
constexpr int kLdIn = kMlpIn + 8, kLdWidth = kMlpWidth + 8;

struct MlpLds {
    u16 W1[kMlpWidth * kLdIn];
    u16 W2[kMlpWidth * kLdWidth];   // columns permuted (see above)
    u16 W3[kMlpWidth * kLdWidth];
    float b[3 * kMlpWidth + 1];
};

// input index k of a hidden layer -> neuron of the previous layer
__device__ __forceinline__ int hidden_input(int k)
{
    const int ks = k >> 5, q = (k >> 3) & 3, e = k & 7;
    return 16 * (2 * ks + (e >> 2)) + 4 * q + (e & 3);
}

// ... and back: neuron -> the input index that names it (two bit fields swapped)
__device__ __forceinline__ int hidden_slot(int j)
{
    return (j & 0x23) | ((j & 0x0C) << 1) | ((j & 0x10) >> 2);
}

__device__ __forceinline__ void load_weights(MlpLds &L, const u16 *wb, const float *wf)
{
    const uint4 *src = reinterpret_cast<const uint4 *>(wb);
    for (int i = threadIdx.x; i < kMlpW1 / 8; i += blockDim.x)
        *reinterpret_cast<uint4 *>(L.W1 + (i / (kMlpIn / 8)) * kLdIn + 8 * (i % (kMlpIn / 8))) = src[i];
    const u16 *w2 = wb + kMlpW1, *w3 = wb + kMlpW1 + kMlpW2;
    for (int i = threadIdx.x; i < kMlpW2; i += blockDim.x) {
        const int o = i / kMlpWidth, k = i % kMlpWidth;
        const int j = o * kMlpWidth + hidden_input(k);
        L.W2[o * kLdWidth + k] = w2[j];
        L.W3[o * kLdWidth + k] = w3[j];
    }
    for (int i = threadIdx.x; i < 3 * kMlpWidth + 1; i += blockDim.x) L.b[i] = wf[i];
}

// One layer, transposed: acc[ot][pt] (neurons 16 ot.., points 16 pt..) = bias (zero when
// null) + W[ot rows] x[pt] over KSTEPS k-steps; W row-major [out][in] (in LDS).
template <int KSTEPS, int PT>
__device__ __forceinline__ void layer_t(const u16 *W, int ldw, const float *bias,
                                        const Frag (&x)[PT][KSTEPS], int lane, f32x4 (&acc)[4][PT])
{
#pragma unroll
    for (int ot = 0; ot < 4; ++ot) {
        f32x4 b0 = f32x4{0.f, 0.f, 0.f, 0.f};
        if (bias) {
            const float *bo = bias + ot * 16 + 4 * (lane >> 4);
            b0 = f32x4{bo[0], bo[1], bo[2], bo[3]};
        }
#pragma unroll
        for (int pt = 0; pt < PT; ++pt) acc[ot][pt] = b0;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            Frag w;
            w.q = *reinterpret_cast<const uint4 *>(W + (ot * 16 + (lane & 15)) * ldw + ks * 32 +
                                                   8 * (lane >> 4));
#pragma unroll
            for (int pt = 0; pt < PT; ++pt) acc[ot][pt] = mfma(w, x[pt][ks], acc[ot][pt]);
        }
    }
}

// ReLU + bf16 of a layer's accumulators into the next layer's B operands: two values are
// rounded to one packed bf16 pair, then the ReLU is one packed 16-bit integer max (a
// negative bf16, -0 included, is a negative int16 and becomes +0; rounding commutes with
// the ReLU, so the pair is bit-identical to bf16(max(x, 0))).
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short i16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t relu_bf16x2(float a, float b)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const bf16x2 v = __builtin_convertvector((f32x2){a, b}, bf16x2);
    const i16x2 z = {0, 0};
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(i16x2, v), z));
}

template <int PT>
__device__ __forceinline__ void relu_to_operand(const f32x4 (&acc)[4][PT], Frag (&h)[PT][2])
{
#pragma unroll
    for (int pt = 0; pt < PT; ++pt)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const f32x4 &lo = acc[2 * ks][pt], &hi = acc[2 * ks + 1][pt];
            h[pt][ks].q = make_uint4(relu_bf16x2(lo[0], lo[1]), relu_bf16x2(lo[2], lo[3]),
                                     relu_bf16x2(hi[0], hi[1]), relu_bf16x2(hi[2], hi[3]));
        }
}

// Forward over M points.  Point i uses position pts[i % G] and sun[i / G] when G > 0
// (every surfel under every sun), or pts[i] and sun[i] when G == 0.
__global__ __launch_bounds__(kMlpThreads) __attribute__((amdgpu_waves_per_eu(3))) void k_mlp_forward(
    const u16 *__restrict__ wb, const float *__restrict__ wf, const float *__restrict__ pts,
    const float *__restrict__ sun, int64_t M, int64_t G, MlpNorm nz, int prob,
    float *__restrict__ out)
{
    __shared__ MlpLds L;
    load_weights(L, wb, wf);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr int PT = kFwdPT;
    const int64_t ntile = (M + kFwdPts - 1) / kFwdPts;
    // output weights as an MFMA weight operand: row 0 (lanes n % 16 == 0) holds w4 in the
    // hidden layers' input numbering, rows 1..15 are zero
    Frag a4[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e)
            a4[ks].h[e] = (lane & 15) == 0
                              ? wb[kMlpW1 + kMlpW2 + kMlpW3 + hidden_input(32 * ks + 8 * (lane >> 4) + e)]
                              : (u16)0;
    for (int64_t tile = (int64_t)blockIdx.x * kMlpWaves + wave; tile < ntile;
         tile += (int64_t)gridDim.x * kMlpWaves) {
        // weight fragments are read from LDS per tile (held across tiles they would take
        // 128 VGPRs)
        asm volatile("" ::: "memory");
        const int64_t base = tile * kFwdPts;
        // all-pairs mode: one division per tile; lanes carry into the next sun
        const int64_t is0 = G > 0 ? base / G : 0, ip0 = base - is0 * G;
        // ---- features in the B layout.  In all-pairs mode a tile that lies under one sun
        // (all but one in G / 64) computes the sun's features once instead of per point:
        // the four sines and cosines are 4 of the 10 quarter-rate instructions of a point
        // (network pass over 20M points: 0.688 -> 0.667 ms)
        const bool one_sun = G > 0 && ip0 + kFwdPts <= G;
        Frag fsun;
        if (one_sun) sun_chunk(sun[2 * is0], sun[2 * is0 + 1], lane >> 4, fsun);
        Frag fa[PT][4];
#pragma unroll
        for (int pt = 0; pt < PT; ++pt) {
            int64_t i = base + pt * 16 + (lane & 15);
            if (i >= M) i = M - 1;
            int64_t ip = i, is = i;
            if (G > 0) {
                ip = ip0 + (i - base);
                is = is0;
                while (ip >= G) { ip -= G; ++is; }
            }
            const float ph[3] = {__fmul_rn(__fsub_rn(pts[3 * ip], nz.cx), nz.inv_half),
                                 __fmul_rn(__fsub_rn(pts[3 * ip + 1], nz.cy), nz.inv_half),
                                 __fmul_rn(__fsub_rn(pts[3 * ip + 2], nz.cz), nz.inv_half)};
#pragma unroll
            for (int ks = 0; ks < 3; ++ks) feature_chunk(ph[ks], lane >> 4, fa[pt][ks]);
            if (!one_sun) sun_chunk(sun[2 * is], sun[2 * is + 1], lane >> 4, fa[pt][3]);
            else fa[pt][3] = fsun;
        }
        f32x4 acc[4][PT];
        Frag h[PT][2];
        layer_t<4>(L.W1, kLdIn, L.b, fa, lane, acc);
        relu_to_operand(acc, h);
        layer_t<2>(L.W2, kLdWidth, L.b + kMlpWidth, h, lane, acc);
        relu_to_operand(acc, h);
        layer_t<2>(L.W3, kLdWidth, L.b + 2 * kMlpWidth, h, lane, acc);
        relu_to_operand(acc, h);
        // ---- output: logit = w4 . h3 + b4, one more transposed MFMA layer whose weight
        // operand holds w4 in row 0: lane n < 16 gets point n's logit in element 0
        float part[PT];
#pragma unroll
        for (int pt = 0; pt < PT; ++pt) {
            f32x4 o = {0.f, 0.f, 0.f, 0.f};
            o = mfma(a4[0], h[pt][0], o);
            o = mfma(a4[1], h[pt][1], o);
            part[pt] = o[0];
        }
        if (lane < 16) {
#pragma unroll
            for (int pt = 0; pt < PT; ++pt) {
                const int64_t i = base + pt * 16 + lane;
                if (i < M) {
                    const float lg = part[pt] + L.b[3 * kMlpWidth];
                    out[i] = prob ? 1.f / (1.f + expf(-lg)) : lg;
                }
            }
        }
    }
}

// ------------------------------------------------------------------- training
// Loss and weight gradients of M paired points.  Per point: dlogit = (sigmoid(logit) - y)
// scale or d_logits scale, da3 = bf16(dlogit w4 [h3 > 0]), da2 = bf16((W3^T da3) [h2 > 0]),
// da1 = bf16((W2^T da2) [h1 > 0]); dW_l = sum da_l h_(l-1)^T, db_l = sum da_l, dw4 = sum
// dlogit h3, db4 = sum dlogit.
//
// A wave takes a 16-point tile through forward and backward, the block's eight waves 128
// points per step.  Activations and their gradients go to LDS twice: transposed [neuron]
// [point], where 8 consecutive points of a neuron are an operand of the weight-gradient
// products (the contraction runs over points), and the gradients also as [point][neuron],
// the operand of the next layer's product.  Each wave owns 16 rows of half of every dW in registers
// over all of its block's steps, so partial gradients leave the chip once per block, and
// features and activations never do.  Biases come from a column of ones.
// The step is bound by latency (3 forward and 2 backward layers, each a chain of LDS
// writes, a barrier and MFMAs), so the grid is one block per CU with two waves per SIMD
// (four waves of two tiles each: 36.4 and 19.9 us against 30.2 and 16.6).
// One forward + backward + Adam: 65,536 points 32.6 us, 6,001 points
// 21.2 us (as separate forward, output, weight-gradient and activation-gradient kernels per
// layer with serial reductions: 525 and 260 us).
constexpr int kTrThreads = 512, kTrWaves = kTrThreads / 64, kTrPT = 1;
static_assert(kTrBlockPts == 16 * kTrPT * kTrWaves, "points per block step");
constexpr int kLdPts = kTrBlockPts + 8;      // padded [neuron][point] rows

struct MlpTrainLds {
    u16 W1[kMlpWidth * kLdIn];
    u16 W2[kMlpWidth * kLdWidth], W3[kMlpWidth * kLdWidth];     // columns permuted
    u16 W2t[kMlpWidth * kLdWidth], W3t[kMlpWidth * kLdWidth];   // [in][out]
    u16 Ft[kMlpIn * kLdPts];                                   // features [feature][point]
    u16 H1t[kMlpWidth * kLdPts], H2t[kMlpWidth * kLdPts];       // activations [neuron][point]
    u16 dAt[kMlpWidth * kLdPts];                                // gradients [neuron][point]
    u16 dA[kTrBlockPts * kLdWidth];                             // gradients [point][neuron]
    float b[3 * kMlpWidth + 1];
    float red[kTrWaves][kMlpWidth + 2];
};

// Operand fragments of 16 points (hidden numbering) -> dst[neuron][point]
__device__ __forceinline__ void store_transposed(const Frag (&h)[2], u16 *dst, int point, int g)
{
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e)
            dst[(16 * (2 * ks + (e >> 2)) + 4 * g + (e & 3)) * kLdPts + point] = h[ks].h[e];
}

// ... and -> dst[point][neuron], four consecutive neurons per store
__device__ __forceinline__ void store_points(const Frag (&h)[2], u16 *dst, int point, int g)
{
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        uint2 *row = reinterpret_cast<uint2 *>(dst + point * kLdWidth + 32 * ks + 4 * g);
        row[0] = make_uint2(h[ks].q.x, h[ks].q.y);
        row[4] = make_uint2(h[ks].q.z, h[ks].q.w);
    }
}

// bf16(x [h > 0]) of a layer's accumulators, in the hidden numbering of h's fragments
template <int PT>
__device__ __forceinline__ void mask_to_operand(const f32x4 (&acc)[4][PT], const Frag (&h)[PT][2],
                                                Frag (&d)[PT][2])
{
#pragma unroll
    for (int pt = 0; pt < PT; ++pt)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                d[pt][ks].h[e] = h[pt][ks].h[e] != 0 ? f2bf(acc[2 * ks + (e >> 2)][pt][e & 3]) : (u16)0;
}

// dw[jt] (16 rows i0 .. of dW, columns j0 + 16 jt ..) += dAt[rows] Ht[columns]^T over the
// block's points; db += dAt[rows] 1
template <int NJ>
__device__ __forceinline__ void weight_grads(const u16 *dAt, const u16 *Ht, int i0, int j0, int lane,
                                             f32x4 (&dw)[NJ], f32x4 &db)
{
    const int r = lane & 15, g = lane >> 4;
    Frag ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones.h[e] = 0x3F80;
#pragma unroll
    for (int kk = 0; kk < kTrBlockPts / 32; ++kk) {
        Frag a;
        a.q = *reinterpret_cast<const uint4 *>(dAt + (i0 + r) * kLdPts + 32 * kk + 8 * g);
        db = mfma(a, ones, db);
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt) {
            Frag b;
            b.q = *reinterpret_cast<const uint4 *>(Ht + (j0 + 16 * jt + r) * kLdPts + 32 * kk + 8 * g);
            dw[jt] = mfma(a, b, dw[jt]);
        }
    }
}

__global__ __launch_bounds__(kTrThreads) void k_mlp_train(
    const float *__restrict__ w, const float *__restrict__ pts, const float *__restrict__ sun,
    int64_t M, const float *__restrict__ labels, const float *__restrict__ dlin, float scale,
    MlpNorm nz, float *__restrict__ part)
{
    __shared__ MlpTrainLds L;
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, col = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // this wave's share of the weight gradients: rows i0 .. i0 + 15, columns from half the width
    const int i0 = 16 * (wave & 3), half = wave >> 2;
    // unrolled, so that a thread's loads are in flight together
#pragma unroll
    for (int q = 0; q < kMlpW1 / kTrThreads; ++q) {
        const int i = q * kTrThreads + tid;
        L.W1[(i / kMlpIn) * kLdIn + i % kMlpIn] = f2bf(w[kOffW1 + i]);
    }
#pragma unroll
    for (int q = 0; q < kMlpW2 / kTrThreads; ++q) {
        const int i = q * kTrThreads + tid, o = i / kMlpWidth, k = i % kMlpWidth;
        const u16 w2 = f2bf(w[kOffW2 + i]), w3 = f2bf(w[kOffW3 + i]);
        const int p = o * kLdWidth + hidden_slot(k);
        L.W2[p] = w2;
        L.W3[p] = w3;
        L.W2t[k * kLdWidth + o] = w2;
        L.W3t[k * kLdWidth + o] = w3;
    }
    if (tid < kMlpWidth) {
        L.b[tid] = w[kOffB1 + tid];
        L.b[kMlpWidth + tid] = w[kOffB2 + tid];
        L.b[2 * kMlpWidth + tid] = w[kOffB3 + tid];
    }
    if (tid == 0) L.b[3 * kMlpWidth] = w[kOffB4];
    // rows of Ft past the 100 features stay zero
    for (int i = tid; i < (kMlpIn - 96) * kLdPts; i += kTrThreads) L.Ft[96 * kLdPts + i] = 0;
    // output weights (bf16) in the hidden numbering, for every row of a weight operand: each
    // lane group then finds its own point's logit in element 0
    Frag a4[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) a4[ks].h[e] = f2bf(w[kOffW4 + hidden_input(32 * ks + 8 * g + e)]);
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 dw1[4], dw2[2], dw3[2], db1 = zero, db2 = zero, db3 = zero;
#pragma unroll
    for (int j = 0; j < 4; ++j) dw1[j] = zero;
#pragma unroll
    for (int j = 0; j < 2; ++j) dw2[j] = dw3[j] = zero;
    float dw4[2][8], db4 = 0.f, loss = 0.f;
#pragma unroll
    for (int k = 0; k < 16; ++k) dw4[k >> 3][k & 7] = 0.f;
    __syncthreads();
    for (int64_t base = (int64_t)blockIdx.x * kTrBlockPts; base < M;
         base += (int64_t)gridDim.x * kTrBlockPts) {
        Frag fa[kTrPT][4], h1[kTrPT][2], h2[kTrPT][2], h[kTrPT][2], d[kTrPT][2];
        f32x4 acc[4][kTrPT];
        int slot[kTrPT];
#pragma unroll
        for (int pt = 0; pt < kTrPT; ++pt) {
            slot[pt] = (wave * kTrPT + pt) * 16 + col;
            const int64_t i = min(base + slot[pt], M - 1);
            const float ph[3] = {__fmul_rn(__fsub_rn(pts[3 * i], nz.cx), nz.inv_half),
                                 __fmul_rn(__fsub_rn(pts[3 * i + 1], nz.cy), nz.inv_half),
                                 __fmul_rn(__fsub_rn(pts[3 * i + 2], nz.cz), nz.inv_half)};
#pragma unroll
            for (int ks = 0; ks < 3; ++ks) {
                feature_chunk(ph[ks], g, fa[pt][ks]);
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    L.Ft[(32 * ks + 8 * g + e) * kLdPts + slot[pt]] = fa[pt][ks].h[e];
            }
            sun_chunk(sun[2 * i], sun[2 * i + 1], g, fa[pt][3]);
            if (g == 0) {
#pragma unroll
                for (int e = 0; e < 4; ++e) L.Ft[(96 + e) * kLdPts + slot[pt]] = fa[pt][3].h[e];
            }
        }
        layer_t<4>(L.W1, kLdIn, L.b, fa, lane, acc);
        relu_to_operand(acc, h1);
        layer_t<2>(L.W2, kLdWidth, L.b + kMlpWidth, h1, lane, acc);
        relu_to_operand(acc, h2);
        layer_t<2>(L.W3, kLdWidth, L.b + 2 * kMlpWidth, h2, lane, acc);
        relu_to_operand(acc, h);
#pragma unroll
        for (int pt = 0; pt < kTrPT; ++pt) {
            store_transposed(h1[pt], L.H1t, slot[pt], g);
            store_transposed(h2[pt], L.H2t, slot[pt], g);
            f32x4 o = mfma(a4[0], h[pt][0], zero);
            o = mfma(a4[1], h[pt][1], o);
            const float lg = o[0] + L.b[3 * kMlpWidth];
            const int64_t i = base + slot[pt];
            float dl = 0.f;
            if (i < M) {
                if (labels) {
                    const float y = labels[i];
                    dl = (1.f / (1.f + expf(-lg)) - y) * scale;
                    if (g == 0) loss += (fmaxf(lg, 0.f) - lg * y + log1pf(expf(-fabsf(lg)))) * scale;
                } else {
                    dl = dlin[i] * scale;
                }
                if (g == 0) db4 += dl;
            }
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const u16 hj = h[pt][ks].h[e];
                    if (i < M) dw4[ks][e] += dl * bf2f(hj);
                    d[pt][ks].h[e] = hj != 0 && i < M ? f2bf(dl * bf2f(a4[ks].h[e])) : (u16)0;
                }
            store_transposed(d[pt], L.dAt, slot[pt], g);
            store_points(d[pt], L.dA, slot[pt], g);
        }
        __syncthreads();
        weight_grads(L.dAt, L.H2t, i0, 32 * half, lane, dw3, db3);
#pragma unroll
        for (int layer = 2; layer > 0; --layer) {
            // gradients of the layer below from this wave's own points
            Frag x[kTrPT][2];
#pragma unroll
            for (int pt = 0; pt < kTrPT; ++pt)
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
                    x[pt][ks].q = *reinterpret_cast<const uint4 *>(L.dA + slot[pt] * kLdWidth + 32 * ks + 8 * g);
            layer_t<2>(layer == 2 ? L.W3t : L.W2t, kLdWidth, nullptr, x, lane, acc);
            mask_to_operand(acc, layer == 2 ? h2 : h1, d);
            __syncthreads();   // every wave has read the gradients above
#pragma unroll
            for (int pt = 0; pt < kTrPT; ++pt) {
                store_transposed(d[pt], L.dAt, slot[pt], g);
                if (layer == 2) store_points(d[pt], L.dA, slot[pt], g);
            }
            __syncthreads();
            if (layer == 2) weight_grads(L.dAt, L.H1t, i0, 32 * half, lane, dw2, db2);
            else weight_grads(L.dAt, L.Ft, i0, 64 * half, lane, dw1, db1);
        }
        __syncthreads();   // features and activations are rewritten by the next step
    }
    // the block's partial gradient, in the order of the parameter vector, then its loss
    float *out = part + (int64_t)blockIdx.x * kTrStride;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = i0 + 4 * g + r;
#pragma unroll
        for (int jt = 0; jt < 4; ++jt)
            out[kOffW1 + i * kMlpIn + 64 * half + 16 * jt + col] = dw1[jt][r];
#pragma unroll
        for (int jt = 0; jt < 2; ++jt) {
            out[kOffW2 + i * kMlpWidth + 32 * half + 16 * jt + col] = dw2[jt][r];
            out[kOffW3 + i * kMlpWidth + 32 * half + 16 * jt + col] = dw3[jt][r];
        }
        if (col == 0 && half == 0) {
            out[kOffB1 + i] = db1[r];
            out[kOffB2 + i] = db2[r];
            out[kOffB3 + i] = db3[r];
        }
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        float x = dw4[k >> 3][k & 7];
        for (int s = 8; s > 0; s >>= 1) x += __shfl_xor(x, s, 64);
        if (col == 0) L.red[wave][hidden_input(32 * (k >> 3) + 8 * g + (k & 7))] = x;
    }
    for (int s = 8; s > 0; s >>= 1) {
        db4 += __shfl_xor(db4, s, 64);
        loss += __shfl_xor(loss, s, 64);
    }
    if (lane == 0) {
        L.red[wave][kMlpWidth] = db4;
        L.red[wave][kMlpWidth + 1] = loss;
    }
    __syncthreads();
    if (tid < kMlpWidth + 2) {
        float x = 0.f;
        for (int k = 0; k < kTrWaves; ++k) x += L.red[k][tid];
        out[kOffW4 + tid] = x;      // dw4, db4, loss
    }
}

// grad[c] = sum over blocks of part[block][c]; the column after the parameters is the loss.
// 64 columns per block, a quarter of the rows per wave.
__global__ __launch_bounds__(256) void k_mlp_train_reduce(const float *__restrict__ part, int nblocks,
                                                          float *__restrict__ d_w, float *__restrict__ loss)
{
    __shared__ float red[4][64];
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int c = blockIdx.x * 64 + lane;
    float s = 0.f;
    if (c <= kMlpParams) {
#pragma unroll 8
        for (int b = q; b < nblocks; b += 4) s += part[(int64_t)b * kTrStride + c];
    }
    red[q][lane] = s;
    __syncthreads();
    if (q != 0 || c > kMlpParams) return;
    s = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
    if (c < kMlpParams) d_w[c] = s;
    else if (loss) *loss = s;
}

__global__ void k_mlp_adam(float *__restrict__ w, float *__restrict__ m, float *__restrict__ v,
                           const float *__restrict__ g, int64_t n, float lr, float b1, float b2,
                           float eps, float bc1, float bc2)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    w[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

// ------------------------------------------------------------------ launchers
hipError_t launch_mlp_prep(const float *w, uint16_t *wb, float *wf, hipStream_t st)
{
    hipLaunchKernelGGL(k_mlp_prep, dim3((kMlpBf16 + 255) / 256), dim3(256), 0, st, w, wb, wf);
    return hipGetLastError();
}

hipError_t launch_mlp_forward(const uint16_t *wb, const float *wf, const float *pts,
                              const float *sun, int64_t M, int64_t G, MlpNorm nz, bool prob,
                              float *out, hipStream_t st)
{
    if (M <= 0) return hipSuccess;
    int64_t tiles = (M + kFwdPts - 1) / kFwdPts;
    int64_t blocks = (tiles + kMlpWaves - 1) / kMlpWaves;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)blocks), dim3(kMlpThreads), 0, st, wb, wf,
                       pts, sun, M, G, nz, prob ? 1 : 0, out);
    return hipGetLastError();
}

hipError_t launch_mlp_train(const float *w, const float *pts, const float *sun, int64_t M,
                            const float *labels, const float *d_logits, float scale, MlpNorm nz,
                            float *part, float *d_w, float *loss, hipStream_t st)
{
    if (M <= 0) return hipSuccess;
    const int blocks = mlp_train_blocks(M);
    hipLaunchKernelGGL(k_mlp_train, dim3(blocks), dim3(kTrThreads), 0, st, w, pts, sun, M, labels,
                       d_logits, scale, nz, part);
    hipLaunchKernelGGL(k_mlp_train_reduce, dim3((kMlpParams + 1 + 63) / 64), dim3(256), 0, st, part,
                       blocks, d_w, loss);
    return hipGetLastError();
}

hipError_t launch_mlp_adam(float *w, float *m, float *v, const float *g, int64_t n, float lr,
                           float b1, float b2, float eps, int step, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const float bc1 = 1.f - powf(b1, (float)step), bc2 = 1.f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_mlp_adam, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, w, m, v, g, n,
                       lr, b1, b2, eps, bc1, bc2);
    return hipGetLastError();
}

}  // namespace ss
