// Internal declarations of the per-point warm-start MLP (lskum_mlp.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

#include "lskum_internal.h"

namespace lskum {
namespace mlp {

constexpr int kIn = 5, kWidth = 128, kOut = 4;
// flat parameter layout: W1[128][5] b1 W2[128][128] b2 W3[128][128] b3 W4[4][128] b4
constexpr int kOffW1 = 0;
constexpr int kOffB1 = kOffW1 + kWidth * kIn;
constexpr int kOffW2 = kOffB1 + kWidth;
constexpr int kOffB2 = kOffW2 + kWidth * kWidth;
constexpr int kOffW3 = kOffB2 + kWidth;
constexpr int kOffB3 = kOffW3 + kWidth * kWidth;
constexpr int kOffW4 = kOffB3 + kWidth;
constexpr int kOffB4 = kOffW4 + kOut * kWidth;
constexpr int kParams = kOffB4 + kOut;
static_assert(kParams == 34308, "parameter count");
constexpr int kMaxParts = 256;  // blocks (and partial gradients) of a training pass
constexpr int kW1Rows = kWidth * 8;  // W1 as [unit][8]: five weights, the bias, two unused
constexpr int kW4Frag = 4 * 64 * 8;  // bf16 of W4 (four outputs padded to 16)

// Rounded copies of the weights: W1 as fp32 rows with the bias, the others as
// matrix-core operand fragments, W2f, W3f as the forward pass multiplies by them,
// W2t, W3t transposed for the backward pass.  The padding of W4f is zero.
struct WeightCopies {
    float* W1f;
    __bf16 *W2f, *W3f, *W4f, *W2t, *W3t;
};

struct Net {
    int device = 0;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    int64_t capacity = 0;  // workspace rows
    int64_t step = 0;      // Adam steps taken
    float* theta = nullptr;  // fp32 master weights
    float* m = nullptr;
    float* v = nullptr;
    WeightCopies copies{};
    // workspace, capacity rows
    float* Xin = nullptr;   // [cap][5] staged features (warm start)
    float* Yout = nullptr;  // [cap][4] predictions
    float* part = nullptr;  // gradient partials of a training pass, part_count(cap) x kParams
    double* loss_part = nullptr;  // kMaxParts
    double* d_loss = nullptr;
    int32_t* d_bad = nullptr;      // per component: 1 if the prediction is unusable
    double* d_res_fs = nullptr;    // per component free-stream residual (residual check)
    int64_t ncomp_cap = 0;
    hipEvent_t ev[2] = {};
};

// Once per process and device, before the first launch: the training kernel
// uses more LDS than a launch may by default.
hipError_t prepare_kernels();
// Predictions Y [m][4] of features X [m][5].
hipError_t forward(Net& net, const float* X, int m, float* Y);
// Partial gradients of a training pass over so many rows.
int part_count(int64_t rows);
// Loss (sum of squared errors, device) and gradient (device, may be NULL) of m
// rows; with lr also one Adam step.
hipError_t gradient(Net& net, const float* X, const float* T, int m, float* grad, double* loss,
                    const float* lr);
// One Adam step on B rows drawn from a data set of n: row r is
// floor(h(seed, step, r) * n / 2^64).
hipError_t minibatch_step(Net& net, int64_t n, const float* X, const float* T, int B, uint64_t seed,
                          int64_t step, double* loss, float lr);
hipError_t refresh_weights(Net& net);
// Features of points [p0, p0 + m) of a state (into Xin) and, optionally,
// targets from its U (into Tout, [m][4]).
hipError_t features(const State& s, int64_t p0, int64_t m, float* Xout, float* Tout);
// U of points [p0, p0 + m) from the predictions Y; marks d_bad[comp] for
// non-finite or non-physical predictions.
hipError_t pred_to_U(Net& net, const State& s, int64_t p0, int64_t m, const float* Y);
// Residual check: components whose residual res[k] is not finite or not below the
// free-stream residual are flagged in d_bad and reset to the free stream.
hipError_t vet_and_fallback(Net& net, const State& s, const double* res);

}  // namespace mlp
}  // namespace lskum
