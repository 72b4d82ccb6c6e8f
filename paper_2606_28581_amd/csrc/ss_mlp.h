// Internal declarations of the surrogate MLP kernels (layout constants, launchers).
#pragma once
#include "ss_internal.h"

namespace ss {

constexpr int kMlpIn = 128, kMlpWidth = 64;
constexpr int kMlpW1 = kMlpWidth * kMlpIn, kMlpW2 = kMlpWidth * kMlpWidth, kMlpW3 = kMlpW2;
// offsets in the FP32 master parameter vector [W1, b1, W2, b2, W3, b3, w4, b4]
constexpr int kOffW1 = 0, kOffB1 = kOffW1 + kMlpW1, kOffW2 = kOffB1 + kMlpWidth;
constexpr int kOffB2 = kOffW2 + kMlpW2, kOffW3 = kOffB2 + kMlpWidth;
constexpr int kOffB3 = kOffW3 + kMlpW3, kOffW4 = kOffB3 + kMlpWidth, kOffB4 = kOffW4 + kMlpWidth;
constexpr int kMlpParams = kOffB4 + 1;   // 16641
constexpr int kMlpBf16 = kMlpW1 + kMlpW2 + kMlpW3 + kMlpWidth;
constexpr int kMlpF32 = 3 * kMlpWidth + 1;
// training: points per block step, blocks (one per CU of the 256), floats per partial row
// (the gradient and the loss, padded to 16 bytes)
constexpr int kTrBlockPts = 128, kTrMaxBlocks = 256;
constexpr int kTrStride = (kMlpParams + 1 + 3) & ~3;
constexpr int mlp_train_blocks(int64_t M)
{
    const int64_t b = (M + kTrBlockPts - 1) / kTrBlockPts;
    return (int)(b < kTrMaxBlocks ? b : kTrMaxBlocks);
}

struct MlpNorm {
    float cx, cy, cz, inv_half;
};

hipError_t launch_mlp_prep(const float *w, uint16_t *wb, float *wf, hipStream_t st);
// logits[i] (or sigmoid(logit) when `prob`) for points i < M; G > 0: position i % G,
// sun i / G; G == 0: position i, sun i.
hipError_t launch_mlp_forward(const uint16_t *wb, const float *wf, const float *pts,
                              const float *sun, int64_t M, int64_t G, MlpNorm nz, bool prob,
                              float *out, hipStream_t st);
// d_w [kMlpParams] and loss (or NULL) of M paired points; dlogit = labels ?
// (sigmoid(logit) - y) * scale : d_logits * scale.  part: mlp_train_blocks(M) rows of
// kTrStride floats.
hipError_t launch_mlp_train(const float *w, const float *pts, const float *sun, int64_t M,
                            const float *labels, const float *d_logits, float scale, MlpNorm nz,
                            float *part, float *d_w, float *loss, hipStream_t st);
hipError_t launch_mlp_adam(float *w, float *m, float *v, const float *g, int64_t n, float lr,
                           float b1, float b2, float eps, int step, hipStream_t st);

}  // namespace ss
