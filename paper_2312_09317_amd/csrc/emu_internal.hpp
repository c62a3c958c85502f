// Internal layout of the summary-statistics emulator (libcpm's emu_* calls).
#pragma once

#include <cstddef>
#include <cstdint>

#include <hip/hip_runtime.h>

namespace cpm {
namespace emu {

constexpr int kIn = 6;        // inputs per point
constexpr int kHidden = 256;  // width of the three hidden layers
constexpr int kOut = 8;       // outputs per point
constexpr int kTile = 16;     // edge of an MFMA tile (16 x 16 x 32)
constexpr int kStep = 32;     // its k extent
constexpr int kInPad = 32;    // K of the first layer, padded to one k-step
constexpr int kOutPad = 32;   // K of the last layer's backward product, likewise
constexpr int kRows = 64;     // batch rows are padded to a multiple of this
constexpr int kLayers = 4;
constexpr int kSplitK = 1024; // batch rows per workgroup in the weight-gradient products

// Packed fp32 parameter vector: W1 (256 x 6), b1, W2 (256 x 256), b2,
// W3 (256 x 256), b3, W4 (8 x 256), b4; W[l] is (out x in), row-major.
constexpr int64_t kW1 = 0, kB1 = kW1 + kHidden * kIn;
constexpr int64_t kW2 = kB1 + kHidden, kB2 = kW2 + kHidden * kHidden;
constexpr int64_t kW3 = kB2 + kHidden, kB3 = kW3 + kHidden * kHidden;
constexpr int64_t kW4 = kB3 + kHidden, kB4 = kW4 + kOut * kHidden;
constexpr int64_t kParams = kB4 + kOut;  // 135,432

// Operands of the matrix products are kept in the order the matrix cores take
// them: element (row, k) of an operand of `steps` k-steps lies in the 1 KiB
// fragment of its 16-row tile and 32-wide k-step, at lane 16 ((k mod 32) / 8)
// + row mod 16, eight consecutive k per lane, so that a wave loads a fragment
// with one contiguous 16-byte load per lane.
__host__ __device__ constexpr size_t frag_at(int row, int k, int steps)
{
    return ((size_t)(row / kTile) * steps + k / kStep) * (kTile * kStep) +
           (size_t)((k % kStep / 8) * kTile + row % kTile) * 8 + k % 8;
}

// bf16 copies of the weights as operands: w[l] rows = outputs, k = inputs
// (forward); wt[l] rows = inputs, k = outputs (backward; layers 2..4).
// Rows beyond the layer's outputs and k beyond its inputs are zero.
struct Copies {
    uint16_t *w[kLayers];
    uint16_t *wt[kLayers];
};

// One pass over a batch, forward only (y set) or forward and backward.
struct RowArgs {
    const float *x;        // n x 6
    const float *norm;
    const float *params;
    Copies c;
    int32_t n, n_pad;
    float *y;              // n x 8, the targets' units (forward)
    const float *targets;  // n x 8 (training)
    // operands of the weight gradients (rows = units, k = batch rows): inputs
    // and activations, and dL/dz of the four layers; and the loss partials
    uint16_t *in_t[kLayers];
    uint16_t *dz_t[kLayers];
    float *loss_part;
};

struct AdamArgs {
    float *param, *m, *v;
    // 1 - beta is passed separately: 1 - 0.999f in fp32 is 1.3e-5 off 0.001
    float lr, beta1, beta2, one_minus_beta1, one_minus_beta2, eps, c1, c2;  // c1, c2: bias corrections 1 - beta^t
    Copies c;
};

struct GradArgs {
    const uint16_t *in_t[kLayers];
    const uint16_t *dz_t[kLayers];
    int32_t n, n_pad;
    int32_t splits;          // workgroups along the batch; > 1: partial sums to part
    float *part;             // splits x kParams
    float *grad;             // kParams
    const float *loss_part;
    int32_t loss_parts;
    float *loss;
    float *grad_out, *loss_out;  // the caller's copies (nullable)
    bool update;             // Adam with the gradient just computed
    AdamArgs adam;
};

// Forward pass (train: and backward, up to dL/dz of every layer) of n rows.
// *loss_parts: loss partials written.
hipError_t launch_rows(const RowArgs &a, bool train, int *loss_parts, hipStream_t st);
// Weight and bias gradients, the loss, and (update) the Adam step.
hipError_t launch_grads(const GradArgs &a, hipStream_t st);
hipError_t launch_adam(const AdamArgs &a, const float *grad, hipStream_t st);
// The bf16 copies of all weights from the fp32 parameters.
hipError_t launch_copies(const Copies &c, const float *params, hipStream_t st);
hipError_t launch_fit_norm(const float *x, const float *t, int n, int log_mask, float *norm, hipStream_t st);
hipError_t launch_fill_f32(float *p, float v, int64_t n, hipStream_t st);

}  // namespace emu
}  // namespace cpm
