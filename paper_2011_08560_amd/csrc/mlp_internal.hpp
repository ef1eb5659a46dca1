// Shapes, parameter layout and buffers of the weight-seeding network (shared by its kernels and
// its host API). Parameter vector (float, this order, weights row-major [in][out]):
//   W0 [96 x 128] (input rows 81..95 are padding and stay zero), b0 [128], W1 [128 x 128], b1 [128],
//   W2 [128 x 128], b2 [128], W3 [128 x 256], b3 [256].
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "philox.hpp"

namespace nfm {

constexpr int kMlpIn = 81, kMlpInPad = 96, kMlpHid = 128, kMlpOut = 256;
// Blocks of the sums over a batch's elements; their partial sums follow the loss in its buffer.
constexpr int kMlpLossBlocks = 64;

__host__ __device__ constexpr int mlp_in(int layer) { return layer == 0 ? kMlpInPad : kMlpHid; }
__host__ __device__ constexpr int mlp_out(int layer) { return layer == 3 ? kMlpOut : kMlpHid; }
// (In closed form: a recursive definition is called at run time in the kernels, and each call waits for all
// loads in flight.)
__host__ __device__ constexpr int mlp_w_off(int layer) {
  return layer == 0 ? 0 : (kMlpInPad + 1) * kMlpHid + (layer - 1) * (kMlpHid + 1) * kMlpHid;
}
__host__ __device__ constexpr int mlp_b_off(int layer) { return mlp_w_off(layer) + mlp_in(layer) * mlp_out(layer); }
constexpr int kMlpNParam = mlp_b_off(3) + kMlpOut;
static_assert(kMlpNParam == 78464, "parameter count");

// Operand order. A wave's products read, for 16 columns j of a [K x N] operand, B(k, j) in steps of four k
// (BF16: 16), lane 16 (k % 4) + j % 16 (BF16: 16 (k / 4 % 4) + j % 16, four consecutive k). Stored so
// that a lane's values for four (BF16: two) steps are 16 bytes and a wave's 1 KB in one piece: read
// from the row-major weights, the same operands took four to eight times as long to arrive (64 or 32
// bytes of each 128-byte line at a time).
__host__ __device__ constexpr int operand_index(int K, int k, int j) {
  return ((j / 16 * (K / 16) + k / 16) * 64 + k % 4 * 16 + j % 16) * 4 + k / 4 % 4;
}
__host__ __device__ constexpr int operand_index_bf16(int K, int k, int j) {
  return ((j / 16 * (K / 32) + k / 32) * 64 + k / 4 % 4 * 16 + j % 16) * 8 + k / 16 % 2 * 4 + k % 4;
}

struct MlpBuffers {
  float *params, *grads, *adam_m, *adam_v, *norm;  // norm: mean[81], sd[81]
  float *wf, *wb;                                 // the weights in operand order (operand_index): of
                                                  // W (products with activations), of W^T (gradients)
  uint16_t* wbf16;                                // BF16 weights in operand order
  float *Xn, *Z1, *A1, *Z2, *A2, *Z3, *A3, *Y, *dY, *dZ3, *dZ2, *dZ1, *loss;
};

hipError_t mlp_init(const MlpBuffers& m, uint64_t seed, hipStream_t s);
hipError_t mlp_forward_f32(const MlpBuffers& m, const float* X, int B, float* Y, hipStream_t s);
hipError_t mlp_loss_grad(const MlpBuffers& m, const float* X, const float* T, const float* Mk, int B, hipStream_t s);
// mlp_loss_grad and mlp_adam in one sequence
hipError_t mlp_train_step(const MlpBuffers& m, const float* X, const float* T, const float* Mk, int B, float lr,
                          float b1, float b2, float eps, float c1, float c2, hipStream_t s);
hipError_t mlp_adam(const MlpBuffers& m, float lr, float b1, float b2, float eps, float c1, float c2, hipStream_t s);
// wf and wb from params, after these were set from outside
hipError_t mlp_order_weights(const MlpBuffers& m, hipStream_t s);
hipError_t mlp_to_bf16(const MlpBuffers& m, hipStream_t s);
hipError_t mlp_infer_bf16(const MlpBuffers& m, const float* X, int B, float* Y, hipStream_t s);

}  // namespace nfm
