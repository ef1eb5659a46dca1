// Kernels of the weight-seeding network (a learned start for the weight iteration of Sec. II):
// 81 inputs -> 3 x 128 GELU -> 256 outputs. FP32 training (forward, backward, Adam) and BF16
// inference, with the dense products on the matrix cores.
//
// Products: one 64-lane wave computes a 16 x 16 tile of C = op(A) op(B) with
// v_mfma_f32_16x16x4_f32 (FP32) or v_mfma_f32_16x16x16_bf16 (BF16, FP32 accumulation). Operand
// lanes: lane l holds A(i0 + l%16, k0 + l/16) and B(k0 + l/16, j0 + l%16) (FP32; BF16: four
// consecutive k per lane, k0 + 4(l/16) + 0..3); the result tile has C(i0 + 4(l/16) + r, j0 + l%16)
// in accumulator r. Dimensions are padded (16 rows per tile, K a multiple of 4 / 16), so every
// access is in bounds without masks.
// FP32 sums have one order everywhere: a product's K range in four contiguous quarters, each summed
// in steps of four, the quarters then added in order.
//
// Launches bound the network (a layer's product at a batch of 256 is 0.01 GFLOP): a workgroup of eight waves
// takes 16 rows through all layers, activations in LDS, each wave's 16 columns of every layer's
// weights in registers, all requested before the first product. A training step is three launches:
// forward (and the sum of the mask), backward to the layers' inputs (and the sum of the errors), all
// gradients with Adam. Batch 256: 22 launches a step before; eight steps and
// their readback 797 us before, 405 us so. BF16 inference of 1000 rows: five launches and a copy,
// 21.5 us, before, 6.8 us so.
#include "mlp_internal.hpp"

namespace nfm {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float gelu_f(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }

__device__ __forceinline__ float gelu_grad_f(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

constexpr int kRowWaves = 8;   // waves of a workgroup that takes 16 rows through the layers
static_assert(kMlpHid == 16 * kRowWaves && kMlpOut == 2 * kMlpHid, "one hidden tile, two output tiles a wave");
// floats of a row in LDS: the 16 rows x 4 columns that a product's step reads lie in 64 banks
constexpr int row_stride(int K) { return K + 4; }

// The B operands of column tile j0 / 16 from weights in operand order.
template <int K>
__device__ __forceinline__ void load_operand(const float* __restrict__ W, int tile, int l, float (&f)[K / 4]) {
#pragma unroll
  for (int q = 0; q < K / 16; ++q) {
    const v4f v = *reinterpret_cast<const v4f*>(W + ((tile * (K / 16) + q) * 64 + l) * 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) f[4 * q + e] = v[e];
  }
}

// Loads above stay above: left to itself the compiler moves each layer's loads to their first use, a
// memory latency per layer.
__device__ __forceinline__ void loads_issued() { asm volatile("" ::: "memory"); }

// Barrier for values in LDS alone: global loads in flight stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A tile's product: 16 rows of A in LDS, B operands in registers.
template <int K>
__device__ __forceinline__ v4f tile_product(const float* A, int li, int lk, const float (&f)[K / 4]) {
  v4f acc[4] = {};
#pragma unroll
  for (int i = 0; i < K / 16; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int step = q * (K / 16) + i;
      acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[li * row_stride(K) + 4 * step + lk], f[step], acc[q], 0, 0, 0);
    }
  return ((acc[0] + acc[1]) + acc[2]) + acc[3];
}

// Sums over the n = B * 256 elements of a batch, in a fixed order: block b of kMlpLossBlocks sums its
// contiguous share (per thread of 256 in order, then a tree), and whoever needs the total adds the
// blocks' sums in a tree. Called by all threads of a block of at least 256.
template <class F>
__device__ __forceinline__ void partial_sum(int n, int block, float* s, float* out, F value) {
  const int chunk = (n + kMlpLossBlocks - 1) / kMlpLossBlocks;
  const int e0 = block * chunk, e1 = min(n, e0 + chunk);
  float v = 0.f;
  if (threadIdx.x < 256) {
    for (int e = e0 + (int)threadIdx.x; e < e1; e += 256) v += value(e);
    s[threadIdx.x] = v;
  }
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) s[threadIdx.x] += s[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[block] = s[0];
}

__device__ __forceinline__ float total_sum(const float* __restrict__ part, float* s) {
  static_assert(kMlpLossBlocks <= 256 && (kMlpLossBlocks & (kMlpLossBlocks - 1)) == 0, "loss partials");
  if ((int)threadIdx.x < kMlpLossBlocks) s[threadIdx.x] = part[threadIdx.x];
  lds_barrier();
  for (int h = kMlpLossBlocks / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) s[threadIdx.x] += s[threadIdx.x + h];
    lds_barrier();
  }
  const float t = s[0];
  lds_barrier();
  return t;
}

// The 16 input rows of a tile, (X - mean) / sd on the 81 inputs of the first B rows, zero elsewhere: a
// thread's elements, loaded ahead of their use.
struct InputRows {
  static constexpr int kEach = 16 * kMlpInPad / (64 * kRowWaves);
  static_assert(kEach * 64 * kRowWaves == 16 * kMlpInPad, "whole elements a thread");
  float x[kEach], mean[kEach], sd[kEach];
  __device__ __forceinline__ void load(const float* __restrict__ X, int row0, int B) {
#pragma unroll
    for (int u = 0; u < kEach; ++u) {
      const int e = threadIdx.x + u * 64 * kRowWaves, i = e / kMlpInPad, k = e % kMlpInPad;
      x[u] = row0 + i < B && k < kMlpIn ? X[(size_t)(row0 + i) * kMlpIn + k] : 0.f;
    }
  }
  __device__ __forceinline__ void load_norm(const float* __restrict__ norm) {
#pragma unroll
    for (int u = 0; u < kEach; ++u) {
      const int k = (threadIdx.x + u * 64 * kRowWaves) % kMlpInPad;
      mean[u] = k < kMlpIn ? norm[k] : 0.f;
      sd[u] = k < kMlpIn ? norm[kMlpIn + k] : 1.f;
    }
  }
  template <class F>
  __device__ __forceinline__ void each(int row0, int B, F f) const {
#pragma unroll
    for (int u = 0; u < kEach; ++u) {
      const int e = threadIdx.x + u * 64 * kRowWaves, i = e / kMlpInPad, k = e % kMlpInPad;
      f(i, k, row0 + i < B && k < kMlpIn ? (x[u] - mean[u]) / sd[u] : 0.f);
    }
  }
};

// Forward: input (X - mean) / sd on the 81 inputs of the first B rows, zero elsewhere; Y [rows_y x 256].
// TRAIN keeps the normalized input, pre-activations and activations of all padded rows, and its last
// kMlpLossBlocks workgroups sum the mask.
template <bool TRAIN>
__global__ void __launch_bounds__(64 * kRowWaves) k_forward(MlpBuffers m, const float* __restrict__ X,
                                                            const float* __restrict__ Mk, int B, int tiles, int row_blocks,
                                                            float* __restrict__ Y, int rows_y) {
  constexpr int IS = row_stride(kMlpInPad), HS = row_stride(kMlpHid);
  __shared__ float s_x[16 * IS], s_a[16 * HS], s_b[16 * HS];
  if (TRAIN && (int)blockIdx.x >= row_blocks) {
    partial_sum(B * kMlpOut, (int)blockIdx.x - row_blocks, s_a, m.loss + 1, [&](int e) { return Mk[e]; });
    return;
  }
  const int wv = threadIdx.x >> 6, l = threadIdx.x & 63, li = l & 15, lk = l >> 4, j = wv * 16 + li;
  const float* __restrict__ P = m.params;
  float w0[kMlpInPad / 4], w1[kMlpHid / 4], w2[kMlpHid / 4], w3[2][kMlpHid / 4];
  InputRows in;
  load_operand<kMlpInPad>(m.wf + mlp_w_off(0), wv, l, w0);
  in.load(X, blockIdx.x * 16, B);
  in.load_norm(m.norm);
  const float bias[5] = {P[mlp_b_off(0) + j], P[mlp_b_off(1) + j], P[mlp_b_off(2) + j], P[mlp_b_off(3) + j],
                         P[mlp_b_off(3) + j + kMlpHid]};
  load_operand<kMlpHid>(m.wf + mlp_w_off(1), wv, l, w1);
  load_operand<kMlpHid>(m.wf + mlp_w_off(2), wv, l, w2);
  load_operand<kMlpHid>(m.wf + mlp_w_off(3), wv, l, w3[0]);
  load_operand<kMlpHid>(m.wf + mlp_w_off(3), wv + kRowWaves, l, w3[1]);
  loads_issued();
  auto stage = [&](int row0) __attribute__((always_inline)) {
    in.each(row0, B, [&](int i, int k, float v) {
      s_x[i * IS + k] = v;
      if (TRAIN) m.Xn[(size_t)(row0 + i) * kMlpInPad + k] = v;
    });
  };
  stage(blockIdx.x * 16);   // (here, where what is in flight behind the inputs is known, not in the loop)
  for (int tile = blockIdx.x; tile < tiles; tile += row_blocks) {
    const int row0 = tile * 16;
    lds_barrier();
    auto hidden = [&](v4f acc, float b, float* s_out, float* Z, float* A) __attribute__((always_inline)) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float z = acc[r] + b, a = gelu_f(z);
        s_out[(4 * lk + r) * HS + j] = a;
        if (TRAIN) {
          const size_t o = (size_t)(row0 + 4 * lk + r) * kMlpHid + j;
          Z[o] = z;
          A[o] = a;
        }
      }
      lds_barrier();
    };
    hidden(tile_product<kMlpInPad>(s_x, li, lk, w0), bias[0], s_a, m.Z1, m.A1);
    hidden(tile_product<kMlpHid>(s_a, li, lk, w1), bias[1], s_b, m.Z2, m.A2);
    hidden(tile_product<kMlpHid>(s_b, li, lk, w2), bias[2], s_a, m.Z3, m.A3);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const v4f acc = tile_product<kMlpHid>(s_a, li, lk, w3[h]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = row0 + 4 * lk + r;
        if (row < rows_y) Y[(size_t)row * kMlpOut + j + h * kMlpHid] = acc[r] + bias[3 + h];
      }
    }
    if (tile + row_blocks < tiles) {
      in.load(X, row0 + 16 * row_blocks, B);
      stage(row0 + 16 * row_blocks);
    }
  }
}

// Masked mean squared error L = sum m (y - t)^2 / sum m over the first B rows: its gradient dY =
// 2 m (y - t) / sum m (zero on padded rows), then dZ = (dY W^T) gelu'(Z) layer by layer. The last
// kMlpLossBlocks workgroups sum m (y - t)^2.
__global__ void __launch_bounds__(64 * kRowWaves) k_backward(MlpBuffers m, const float* __restrict__ T,
                                                             const float* __restrict__ Mk, int B, int tiles) {
  constexpr int OS = row_stride(kMlpOut), HS = row_stride(kMlpHid);
  __shared__ float s_y[16 * OS], s_a[16 * HS], s_b[16 * HS];
  if ((int)blockIdx.x >= tiles) {
    partial_sum(B * kMlpOut, (int)blockIdx.x - tiles, s_a, m.loss + 1 + kMlpLossBlocks, [&](int e) {
      const float mk = Mk[e], d = m.Y[e] - T[e];
      return mk * d * d;
    });
    return;
  }
  const int wv = threadIdx.x >> 6, l = threadIdx.x & 63, li = l & 15, lk = l >> 4, j = wv * 16 + li;
  const int row0 = blockIdx.x * 16, n = B * kMlpOut;
  // the elements of dY and of the pre-activations, then the operands: all in flight at once
  constexpr int kEach = 16 * kMlpOut / (64 * kRowWaves);
  float mk[kEach], y[kEach], t[kEach], z[3][4];
#pragma unroll
  for (int u = 0; u < kEach; ++u) {
    const int e = row0 * kMlpOut + (int)threadIdx.x + u * 64 * kRowWaves;
    mk[u] = e < n ? Mk[e] : 0.f;
    y[u] = e < n ? m.Y[e] : 0.f;
    t[u] = e < n ? T[e] : 0.f;
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const size_t o = (size_t)(row0 + 4 * lk + r) * kMlpHid + j;
    z[0][r] = m.Z3[o];
    z[1][r] = m.Z2[o];
    z[2][r] = m.Z1[o];
  }
  float w3[kMlpOut / 4], w2[kMlpHid / 4], w1[kMlpHid / 4];
  load_operand<kMlpOut>(m.wb + mlp_w_off(3), wv, l, w3);
  load_operand<kMlpHid>(m.wb + mlp_w_off(2), wv, l, w2);
  load_operand<kMlpHid>(m.wb + mlp_w_off(1), wv, l, w1);
  loads_issued();
  const float msum = total_sum(m.loss + 1, s_a);
  const float inv = msum > 0.f ? 1.0f / msum : 0.f;
#pragma unroll
  for (int u = 0; u < kEach; ++u) {
    const int i = threadIdx.x + u * 64 * kRowWaves, e = row0 * kMlpOut + i;
    const float d = e < n ? 2.0f * mk[u] * (y[u] - t[u]) * inv : 0.f;
    s_y[i / kMlpOut * OS + i % kMlpOut] = d;
    m.dY[e] = d;
  }
  lds_barrier();
  auto layer = [&](v4f acc, const float (&Z)[4], float* dZ, float* s_out) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const size_t o = (size_t)(row0 + 4 * lk + r) * kMlpHid + j;
      const float d = acc[r] * gelu_grad_f(Z[r]);
      dZ[o] = d;
      if (s_out) s_out[(4 * lk + r) * HS + j] = d;
    }
    lds_barrier();
  };
  layer(tile_product<kMlpOut>(s_y, li, lk, w3), z[0], m.dZ3, s_a);
  layer(tile_product<kMlpHid>(s_a, li, lk, w2), z[1], m.dZ2, s_b);
  layer(tile_product<kMlpHid>(s_b, li, lk, w1), z[2], m.dZ1, nullptr);
}

// Adam with bias correction: c1 = 1 / (1 - beta1^t), c2 = 1 / (1 - beta2^t).
struct AdamArgs {
  float lr, b1, b2, eps, c1, c2;
};
// A parameter with its moments, loaded ahead of its gradient; step() returns its next value (whose
// copies in operand order are the caller's).
struct AdamState {
  float p, m, v;
  __device__ __forceinline__ void load(const MlpBuffers& b, int e) {
    p = b.params[e];
    m = b.adam_m[e];
    v = b.adam_v[e];
  }
  __device__ __forceinline__ float step(const MlpBuffers& b, int e, float gi, const AdamArgs& a) {
    const float mi = a.b1 * m + (1.0f - a.b1) * gi;
    const float vi = a.b2 * v + (1.0f - a.b2) * gi * gi;
    b.adam_m[e] = mi;
    b.adam_v[e] = vi;
    p -= a.lr * (mi * a.c1) / (sqrtf(vi * a.c2) + a.eps);
    b.params[e] = p;
    return p;
  }
};

// Weight (k, j) of a layer in both operand orders (the gradient never goes to the first layer's input).
__device__ __forceinline__ void store_ordered(const MlpBuffers& m, int layer, int k, int j, float w) {
  m.wf[mlp_w_off(layer) + operand_index(mlp_in(layer), k, j)] = w;
  if (layer > 0) m.wb[mlp_w_off(layer) + operand_index(mlp_out(layer), j, k)] = w;
}
__device__ __forceinline__ void store_ordered(const MlpBuffers& m, int e, float w) {
  for (int layer = 0; layer < 4; ++layer) {
    const int q = e - mlp_w_off(layer);
    if (q >= 0 && q < mlp_in(layer) * mlp_out(layer)) store_ordered(m, layer, q / mlp_out(layer), q % mlp_out(layer), w);
  }
}

__global__ void k_adam(MlpBuffers m, AdamArgs a) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= kMlpNParam) return;
  AdamState st;
  st.load(m, e);
  store_ordered(m, e, st.step(m, e, m.grads[e], a));
}

__global__ void k_order_weights(MlpBuffers m) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < kMlpNParam) store_ordered(m, e, m.params[e]);
}

// All gradients: dW = A^T dZ by 16 x 16 tiles (four waves, a quarter of the rows each; the first adds
// the quarters in order), db = column sums of dZ (a thread per 16th row and column, then the 16 in
// order), one workgroup for the loss. ADAM applies the step to each parameter where its gradient
// is formed (no other workgroup reads the parameters).
constexpr int weight_tiles(int layer) { return mlp_in(layer) / 16 * (mlp_out(layer) / 16); }
constexpr int kWeightTiles = weight_tiles(0) + weight_tiles(1) + weight_tiles(2) + weight_tiles(3);
constexpr int kBiasTiles = (3 * kMlpHid + kMlpOut) / 16;

template <bool ADAM>
__global__ void __launch_bounds__(256) k_grads(MlpBuffers m, int Bp, AdamArgs adam) {
  __shared__ __attribute__((aligned(16))) float s[16 * 17 * 4];
  static_assert(__alignof__(s) >= sizeof(v4f), "read and written as v4f below");
  const int wv = threadIdx.x >> 6, l = threadIdx.x & 63, li = l & 15, lk = l >> 4;
  int id = blockIdx.x;
  if (id == kWeightTiles + kBiasTiles) {
    const float msum = total_sum(m.loss + 1, s), esum = total_sum(m.loss + 1 + kMlpLossBlocks, s);
    if (threadIdx.x == 0) m.loss[0] = esum * (msum > 0.f ? 1.0f / msum : 0.f);
    return;
  }
  auto input = [&](int layer) -> const float* { return layer == 0 ? m.Xn : layer == 1 ? m.A1 : layer == 2 ? m.A2 : m.A3; };
  auto delta = [&](int layer) -> const float* { return layer == 0 ? m.dZ1 : layer == 1 ? m.dZ2 : layer == 2 ? m.dZ3 : m.dY; };
  if (id < kWeightTiles) {
    int layer = 3;   // the widest first
    while (id >= weight_tiles(layer)) id -= weight_tiles(layer--);
    const int lda = mlp_in(layer), ldb = mlp_out(layer), tj = id % (ldb / 16), ti = id / (ldb / 16);
    const float* __restrict__ A = input(layer) + ti * 16 + li;
    const float* __restrict__ D = delta(layer) + tj * 16 + li;
    const int kper = Bp / 4, e0 = mlp_w_off(layer) + (ti * 16 + 4 * lk) * ldb + tj * 16 + li;
    AdamState st[4];
    if (ADAM && wv == 0)
      for (int r = 0; r < 4; ++r) st[r].load(m, e0 + r * ldb);
    v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 16
    for (int k0 = wv * kper; k0 < (wv + 1) * kper; k0 += 4)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(A[(size_t)(k0 + lk) * lda], D[(size_t)(k0 + lk) * ldb], acc, 0, 0, 0);
    v4f* part = reinterpret_cast<v4f*>(s);
    static_assert(sizeof(s) >= 3 * 64 * sizeof(v4f), "three partial tiles");
    if (wv > 0) part[(wv - 1) * 64 + l] = acc;
    __syncthreads();
    if (wv > 0) return;
#pragma unroll
    for (int q = 0; q < 3; ++q) acc += part[q * 64 + l];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      m.grads[e0 + r * ldb] = acc[r];
      if (ADAM) store_ordered(m, layer, ti * 16 + 4 * lk + r, tj * 16 + li, st[r].step(m, e0 + r * ldb, acc[r], adam));
    }
    return;
  }
  id -= kWeightTiles;
  int layer = 3;
  while (id >= mlp_out(layer) / 16) id -= mlp_out(layer--) / 16;
  const int col = threadIdx.x & 15, slice = threadIdx.x >> 4, ld = mlp_out(layer);
  const float* __restrict__ D = delta(layer) + id * 16 + col;
  float v = 0.f;
  for (int i = slice; i < Bp; i += 16) v += D[(size_t)i * ld];
  s[slice * 17 + col] = v;
  __syncthreads();
  if (slice == 0) {
    float t = 0.f;
#pragma unroll
    for (int k = 0; k < 16; ++k) t += s[k * 17 + col];
    const int e = mlp_b_off(layer) + id * 16 + col;
    m.grads[e] = t;
    if (ADAM) {
      AdamState st;
      st.load(m, e);
      st.step(m, e, t, adam);
    }
  }
}

// Glorot-uniform weights from the Philox stream (counter (e >> 2, layer, 0, 6) under the seed),
// zero biases and zero padding rows of the first layer.
__global__ void k_mlp_init(float* __restrict__ p, uint32_t key0, uint32_t key1) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= kMlpNParam) return;
  float v = 0.f;
  for (int layer = 0; layer < 4; ++layer) {
    const int o = mlp_w_off(layer), nin = mlp_in(layer), nout = mlp_out(layer);
    if (e >= o && e < o + nin * nout) {
      const int row = (e - o) / nout;
      const int fan_in = layer == 0 ? kMlpIn : nin;
      if (row < fan_in) {
        const int q = e - o;
        const u32x4 r = philox4x32_10((uint32_t)(q >> 2), (uint32_t)layer, 0u, 6u, key0, key1);
        const uint32_t w = r.v[q & 3];
        const float a = sqrtf(6.0f / (float)(fan_in + nout));
        v = a * (2.0f * ((float)(w >> 8) + 0.5f) * (1.0f / 16777216.0f) - 1.0f);
      }
    }
  }
  p[e] = v;
}

// ------------------------------------------------------------------ BF16 inference

__device__ __forceinline__ uint16_t bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// BF16 copy of the weights, in operand order.
__global__ void k_to_bf16(const float* __restrict__ p, uint16_t* __restrict__ wt) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  for (int layer = 0; layer < 4; ++layer) {
    const int o = mlp_w_off(layer), nin = mlp_in(layer), nout = mlp_out(layer);
    if (e < nin * nout) wt[o + operand_index_bf16(nin, e / nout, e % nout)] = bf16_rne(p[o + e]);
  }
}

// A tile's product, 16 rows of A in LDS (BF16), B operands in registers, k in steps of 16 in order.
template <int K>
__device__ __forceinline__ v4f tile_product_bf16(const uint16_t* A, int li, int lk, const v4s (&f)[K / 16]) {
  v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < K / 16; ++i) {
    const v4s a = *reinterpret_cast<const v4s*>(A + li * (K + 16) + 16 * i + 4 * lk);
    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, f[i], acc, 0, 0, 0);
  }
  return acc;
}

template <int K>
__device__ __forceinline__ void load_operand_bf16(const uint16_t* __restrict__ Wt, int tile, int l, v4s (&f)[K / 16]) {
#pragma unroll
  for (int q = 0; q < K / 32; ++q) {
    const v8s v = *reinterpret_cast<const v8s*>(Wt + ((tile * (K / 32) + q) * 64 + l) * 8);
    f[2 * q] = __builtin_shufflevector(v, v, 0, 1, 2, 3);
    f[2 * q + 1] = __builtin_shufflevector(v, v, 4, 5, 6, 7);
  }
}

// Hidden activations are rounded to BF16, the output row stays FP32. MANY: workgroups take several row
// tiles each. Without it a layer's weights give their registers back when it is done: 105 in all (140 with
// the loop), so that the eight waves find room beside sampling waves that hold up to half of each SIMD's
// (256 rows beside 700 waves of L = 8, 7 ms: 0.025 ms, with 140 registers after the launch's end). Alone
// 6.8 us for 256 or 1000 rows (6.6 with the loop), 8192 rows 10.1 (12.5).
template <bool MANY>
__global__ void __launch_bounds__(64 * kRowWaves, MANY ? 1 : 4) k_infer_bf16(MlpBuffers m, const float* __restrict__ X,
                                                                             int B, float* __restrict__ Y) {
  constexpr int IS = kMlpInPad + 16, HS = kMlpHid + 16;
  __shared__ __attribute__((aligned(16))) uint16_t s_x[16 * IS], s_a[16 * HS], s_b[16 * HS];
  const int wv = threadIdx.x >> 6, l = threadIdx.x & 63, li = l & 15, lk = l >> 4, j = wv * 16 + li;
  const uint16_t* __restrict__ W = m.wbf16;
  const float* __restrict__ P = m.params;
  v4s w0[kMlpInPad / 16], w1[kMlpHid / 16], w2[kMlpHid / 16], w3[2][kMlpHid / 16];
  InputRows in;
  load_operand_bf16<kMlpInPad>(W + mlp_w_off(0), wv, l, w0);
  in.load(X, blockIdx.x * 16, B);
  in.load_norm(m.norm);
  const float bias[5] = {P[mlp_b_off(0) + j], P[mlp_b_off(1) + j], P[mlp_b_off(2) + j], P[mlp_b_off(3) + j],
                         P[mlp_b_off(3) + j + kMlpHid]};
  load_operand_bf16<kMlpHid>(W + mlp_w_off(1), wv, l, w1);
  load_operand_bf16<kMlpHid>(W + mlp_w_off(2), wv, l, w2);
  load_operand_bf16<kMlpHid>(W + mlp_w_off(3), wv, l, w3[0]);
  load_operand_bf16<kMlpHid>(W + mlp_w_off(3), wv + kRowWaves, l, w3[1]);
  loads_issued();
  auto stage = [&](int row0) __attribute__((always_inline)) {
    in.each(row0, B, [&](int i, int k, float v) { s_x[i * IS + k] = bf16_rne(v); });
  };
  stage(blockIdx.x * 16);
  const int step = gridDim.x * 16;
  for (int row0 = blockIdx.x * 16; row0 < B; row0 += step) {
    lds_barrier();
    auto hidden = [&](v4f acc, float b, uint16_t* s_out) __attribute__((always_inline)) {
#pragma unroll
      for (int r = 0; r < 4; ++r) s_out[(4 * lk + r) * HS + j] = bf16_rne(gelu_f(acc[r] + b));
      lds_barrier();
    };
    hidden(tile_product_bf16<kMlpInPad>(s_x, li, lk, w0), bias[0], s_a);
    hidden(tile_product_bf16<kMlpHid>(s_a, li, lk, w1), bias[1], s_b);
    hidden(tile_product_bf16<kMlpHid>(s_b, li, lk, w2), bias[2], s_a);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const v4f acc = tile_product_bf16<kMlpHid>(s_a, li, lk, w3[h]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = row0 + 4 * lk + r;
        if (row < B) Y[(size_t)row * kMlpOut + j + h * kMlpHid] = acc[r] + bias[3 + h];
      }
    }
    if constexpr (!MANY) break;
    if (row0 + step < B) {
      in.load(X, row0 + step, B);
      stage(row0 + step);
    }
  }
}

// ------------------------------------------------------------------ sequences

// Workgroups for the row tiles of a call: beyond two per compute unit they take several tiles each,
// with their weights kept.
static int row_blocks(int tiles) { return tiles < 512 ? tiles : 512; }

hipError_t mlp_forward_f32(const MlpBuffers& m, const float* X, int B, float* Y, hipStream_t s) {
  const int tiles = (B + 15) / 16, nb = row_blocks(tiles);
  hipLaunchKernelGGL(k_forward<false>, dim3(nb), dim3(64 * kRowWaves), 0, s, m, X, nullptr, B, tiles, nb, Y, B);
  return hipGetLastError();
}

static hipError_t loss_grad(const MlpBuffers& m, const float* X, const float* T, const float* Mk, int B,
                            const AdamArgs* adam, hipStream_t s) {
  const int tiles = (B + 15) / 16, nb = row_blocks(tiles);
  hipLaunchKernelGGL(k_forward<true>, dim3(nb + kMlpLossBlocks), dim3(64 * kRowWaves), 0, s, m, X, Mk, B, tiles, nb, m.Y,
                     tiles * 16);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_backward, dim3(tiles + kMlpLossBlocks), dim3(64 * kRowWaves), 0, s, m, T, Mk, B, tiles);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const dim3 grid(kWeightTiles + kBiasTiles + 1);
  if (adam)
    hipLaunchKernelGGL(k_grads<true>, grid, dim3(256), 0, s, m, tiles * 16, *adam);
  else
    hipLaunchKernelGGL(k_grads<false>, grid, dim3(256), 0, s, m, tiles * 16, AdamArgs{});
  return hipGetLastError();
}

hipError_t mlp_loss_grad(const MlpBuffers& m, const float* X, const float* T, const float* Mk, int B, hipStream_t s) {
  return loss_grad(m, X, T, Mk, B, nullptr, s);
}

hipError_t mlp_train_step(const MlpBuffers& m, const float* X, const float* T, const float* Mk, int B, float lr,
                          float b1, float b2, float eps, float c1, float c2, hipStream_t s) {
  const AdamArgs a{lr, b1, b2, eps, c1, c2};
  return loss_grad(m, X, T, Mk, B, &a, s);
}

hipError_t mlp_adam(const MlpBuffers& m, float lr, float b1, float b2, float eps, float c1, float c2, hipStream_t s) {
  const AdamArgs a{lr, b1, b2, eps, c1, c2};
  hipLaunchKernelGGL(k_adam, dim3((kMlpNParam + 255) / 256), dim3(256), 0, s, m, a);
  return hipGetLastError();
}

hipError_t mlp_order_weights(const MlpBuffers& m, hipStream_t s) {
  hipLaunchKernelGGL(k_order_weights, dim3((kMlpNParam + 255) / 256), dim3(256), 0, s, m);
  return hipGetLastError();
}

hipError_t mlp_init(const MlpBuffers& m, uint64_t seed, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_init, dim3((kMlpNParam + 255) / 256), dim3(256), 0, s, m.params, (uint32_t)seed,
                     (uint32_t)(seed >> 32));
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : mlp_order_weights(m, s);
}

hipError_t mlp_to_bf16(const MlpBuffers& m, hipStream_t s) {
  hipLaunchKernelGGL(k_to_bf16, dim3((kMlpHid * kMlpOut + 255) / 256), dim3(256), 0, s, m.params, m.wbf16);
  return hipGetLastError();
}

hipError_t mlp_infer_bf16(const MlpBuffers& m, const float* X, int B, float* Y, hipStream_t s) {
  const int tiles = (B + 15) / 16, nb = row_blocks(tiles);
  if (nb < tiles)
    hipLaunchKernelGGL(k_infer_bf16<true>, dim3(nb), dim3(64 * kRowWaves), 0, s, m, X, B, Y);
  else
    hipLaunchKernelGGL(k_infer_bf16<false>, dim3(nb), dim3(64 * kRowWaves), 0, s, m, X, B, Y);
  return hipGetLastError();
}

}  // namespace nfm
