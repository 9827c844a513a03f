// Host-visible argument blocks and launchers of the learned-demapper kernels.
#pragma once
#include <hip/hip_runtime.h>

#include "device_common.hpp"
#include <stdint.h>

namespace dm {

// Forward and backward of a batch; matrices over the batch ("f") are written in MFMA operand
// order, [32-row tile][16-sample step][hi, lo][64 lanes][8] (Xf: no low words); see
// mlp_kernels.hip.  A tile of 32 rows takes 64 B elements.
struct TrainPassArgs {
    const float* y;        // B x D
    const float* sigma2;   // B
    const float* target;   // B x m exact LLRs (nats)
    // weights in operand order: [256 x 32], [256 x 256] and its transpose, [32 x 256] and its transpose
    const __bf16 *W1t, *W2t, *W2, *W3t, *W3;
    const float *b1, *b2, *b3;
    __bf16 *Xf, *A1f, *A2f, *dOf, *dH2f, *dH1f;  // inputs, activations, deltas
    float* loss_tiles;     // B / 32 loss sums
    float scale;           // 1 / (B m)
    int B, D, m;
};

// Weight and bias gradients of a batch: K-split partials and the bias sums.
struct WeightGradArgs {
    const __bf16 *Xf, *A1f, *A2f, *dOf, *dH2f, *dH1f;
    float *part1, *part2, *part3;  // [splits][rows x cols] of W1t, W2t, W3t
    float* sums;                   // mlp_sum_floats(): bias partial sums, [dH1 | dH2 | dO 32-row tile][t][row]
    int B, splits2, splits13;      // splits of dW2 (16), and of dW1 and dW3 (16, 32 or 64)
};

struct AdamArgs {
    float* w;
    float* m;
    float* v;
    float* grad;        // written by the reduction
    const float* part;  // splits > 0: [splits][rows x cols]; splits == 0 (a bias): its partial sums
    int splits;
    __bf16* copy;   // BF16 copies in operand order, may be null
    __bf16* copyT;  // may be null
    int rows, cols, mask_rows, mask_cols;
    float lr, beta1, beta2, eps, bc1, bc2;
};

// Inference: all BF16 weights staged in LDS; see mlp_infer.hip for the fragment layout.
// One received block at its SNR.
struct MlpInferPoint {
    const float* y;           // N x D received symbols
    float* llr;               // N x m or null
    unsigned long long* acc;  // [kAccSlots][2] fixed-point GMI sum, or null
    float snr_feature;        // (s - 7.5) / 7.5, s = -10 log10(2 sigma2)
};
struct MlpInferArgs {
    MlpInferPoint pt[kMaxSnrPerLaunch];
    int n_pts;
    const uint4* frag;      // [W1 | W2 | W3] operand fragments
    const float* bias;      // b1 (256, unused: packed into the fragments) | b2 (256) | b3 (32, zero past m)
    const uint16_t* tx;     // N transmitted rows or null
    const uint16_t* row2label;
    int64_t N;              // symbols per block
    int D, m, M;
    uint32_t* bad_tx;
};

hipError_t launch_train_pass(const TrainPassArgs& a, hipStream_t st);
size_t mlp_sum_floats();
hipError_t launch_weight_grad(const WeightGradArgs& a, hipStream_t st);
// Several parameter tensors in one launch.
constexpr int kAdamMaxTensors = 8;
struct AdamBatch {
    AdamArgs t[kAdamMaxTensors];
    int first_block[kAdamMaxTensors];  // set by the launcher
    int count;
    int reduce, update;  // form the gradients from the splits; take the Adam step and rewrite the copies
};
hipError_t launch_adam_batch(AdamBatch b, hipStream_t st);

// Number of 16-byte fragments of the inference weight table (H = 256 hidden units).
size_t mlp_frag_count();
// Build the inference fragment table from the BF16 values of the row-major (out x in) FP32 masters
// W1t [256 x 32] (D + 1 <= 14 inputs), W2t [256 x 256], W3t [32 x 256] and the FP32 bias b1.
hipError_t launch_mlp_pack(const float* W1t, const float* W2t, const float* W3t, const float* b1, uint4* frag,
                           hipStream_t st);
hipError_t launch_mlp_infer(const MlpInferArgs& a, int grid, hipStream_t st);
hipError_t prepare_mlp_infer();

}  // namespace dm
