// Inputs of the weight-seeding model: canonical tables for a short high-temperature run, and a
// per-realization feature vector from the couplings and that run's energy histogram.
//
// Feature vector (81 floats per realization):
//   x[0]       L / 12
//   x[1..3]    frustrated fraction of (x,y), (y,z), (z,x) plaquettes; x[4] of all plaquettes
//              (a plaquette (i; d1, d2) has bonds J_d1(i), J_d2(i+e_d1), J_d1(i+e_d2), J_d2(i) and
//              is frustrated when their product is -1)
//   x[5..7]    negative-bond fraction along x, y, z; x[8] of all bonds; x[9] = n_minus mod 2
//   x[10..13]  fraction of elementary cubes with 0, 2, 4, 6 frustrated faces
//   x[14..16]  mean / 6, variance / 6, fourth central moment / 96 of the site sums sum_j J_ij
//   x[17..80]  histogram of E/N in 64 bins over [-2, 0): bin floor((E/N + 2) 32) clipped to
//              [0, 63], as fractions of all entries of the realization's level histogram
// Counts are exact integers; the moments are formed in FP64 from the 7-bin histogram of site sums.
#include "kernels.hpp"
#include "table_builder.hpp"

namespace nfm {

// Canonical Metropolis at temperature T: lnW(k) = -E_k / T given on the two top levels; the table
// builder continues the lowest step below them, which is the same constant step -4/T.
__global__ void k_canonical_lnw(const RealInfo* __restrict__ reals, int n_real, double T, double* __restrict__ lnw,
                                int32_t* __restrict__ k_lo, int32_t* __restrict__ k_top) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n_real) return;
  const RealInfo ri = reals[r];
  const int K = ri.K;
  k_lo[r] = K - 2;
  k_top[r] = K - 1;
  lnw[ri.level_off + K - 2] = -(double)(ri.e_base + 4 * (K - 2)) / T;
  lnw[ri.level_off + K - 1] = -(double)(ri.e_base + 4 * (K - 1)) / T;
}

hipError_t launch_canonical_tables(RealInfo* reals, int n_real, double T, double* lnw, int32_t* k_lo, int32_t* k_top,
                                   uint32_t* tables, hipStream_t s) {
  hipLaunchKernelGGL(k_canonical_lnw, dim3((n_real + 255) / 256), dim3(256), 0, s, reals, n_real, T, lnw, k_lo, k_top);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_build_tables(reals, n_real, lnw, k_lo, k_top, tables, s);
}

// A row (y, z) of a direction's couplings as L bits (1 <=> J = -1), from words in LDS.
__device__ __forceinline__ uint32_t j_row(const uint32_t* jw, int JW, int L, int d, int y, int z) {
  const int off = L * (y + L * z);
  const uint32_t* q = jw + d * JW + (off >> 5);
  return __builtin_amdgcn_alignbit(q[1], q[0], off & 31) & ((1u << L) - 1u);
}
// Of a row: bits of the sites x + 1, x - 1 (periodic).
__device__ __forceinline__ uint32_t x_next(uint32_t v, int L) { return (v >> 1) | ((v & 1u) << (L - 1)); }
__device__ __forceinline__ uint32_t x_prev(uint32_t v, int L) { return ((v << 1) & ((1u << L) - 1u)) | (v >> (L - 1)); }

// Bit planes of the number of set bits among six.
struct Count6 {
  uint32_t c0, c1, c2;
};
__device__ __forceinline__ Count6 count6(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t e, uint32_t f) {
  const uint32_t s1 = a ^ b ^ c, k1 = (a & b) | (c & (a ^ b)), s2 = d ^ e ^ f, k2 = (d & e) | (f & (d ^ e));
  const uint32_t t = s1 & s2;
  return {s1 ^ s2, k1 ^ k2 ^ t, (k1 & k2) | (t & (k1 ^ k2))};
}

// Adds the wave's sums of three counts (each at most L per lane, so ten bits hold a sum) to a, b, c.
// (As single LDS additions, 17 in all, they were most of the kernel: the lanes of a wave one by one.)
__device__ __forceinline__ void add_counts(int n0, int n1, int n2, int* a, int* b, int* c) {
  static_assert(kWave * kMaxL < 1024, "ten bits a count");
  uint32_t v = (uint32_t)n0 | (uint32_t)n1 << 10 | (uint32_t)n2 << 20;
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if ((threadIdx.x & 63) == 0) {
    atomicAdd(a, (int)(v & 1023u));
    atomicAdd(b, (int)(v >> 10 & 1023u));
    atomicAdd(c, (int)(v >> 20));
  }
}

// A thread per row (y, z): plaquettes, cubes and site sums of its L sites at once, with exclusive ors
// of rows, bit-sliced counts and bit counts (site by site with divisions for each neighbour: 71 us for
// 1024 realizations of L = 10; 9 us so).
__global__ void k_features(const RealInfo* __restrict__ reals, const uint32_t* __restrict__ jabi,
                           const unsigned long long* __restrict__ hist, float* __restrict__ x) {
  const RealInfo ri = reals[blockIdx.x];
  const int L = ri.L, N = ri.N, JW = abi_plane_words(N);
  const uint32_t* jw = jabi + ri.jabi_off;
  __shared__ int s_cnt[17];  // fr[3], neg[3], cubes[4], site-sum histogram[7]
  __shared__ unsigned long long s_bin[64];
  __shared__ uint32_t s_j[3 * abi_plane_words(kMaxL * kMaxL * kMaxL) + 1];   // (a row's second word)
  __shared__ uint16_t s_p[3][kMaxL * kMaxL];                                // frustrated plaquettes of each row
  for (int k = threadIdx.x; k < 17; k += blockDim.x) s_cnt[k] = 0;
  for (int k = threadIdx.x; k < 64; k += blockDim.x) s_bin[k] = 0ull;
  for (int k = threadIdx.x; k < 3 * JW + 1; k += blockDim.x) s_j[k] = k < 3 * JW ? jw[k] : 0u;
  __syncthreads();
  const int row = threadIdx.x, y = row % L, z = row / L;
  const int yn = y + 1 < L ? y + 1 : 0, yp = y ? y - 1 : L - 1, zn = z + 1 < L ? z + 1 : 0, zp = z ? z - 1 : L - 1;
  auto J = [&](int d, int yy, int zz) { return j_row(s_j, JW, L, d, yy, zz); };
  const bool mine = row < L * L;
  const uint32_t all = mine ? (1u << L) - 1u : 0u;
  uint32_t p[3] = {0, 0, 0}, jr[3] = {0, 0, 0};
  Count6 n{0, 0, 0};
  if (mine) {
    for (int d = 0; d < 3; ++d) jr[d] = J(d, y, z);
    // J_d1(i) J_d2(i + e_d1) J_d1(i + e_d2) J_d2(i) for (x, y), (y, z), (z, x)
    p[0] = jr[0] ^ x_next(jr[1], L) ^ J(0, yn, z) ^ jr[1];
    p[1] = jr[1] ^ J(2, yn, z) ^ J(1, y, zn) ^ jr[2];
    p[2] = jr[2] ^ J(0, y, zn) ^ x_next(jr[2], L) ^ jr[0];
    for (int o = 0; o < 3; ++o) s_p[o][row] = (uint16_t)p[o];
    n = count6(jr[0], jr[1], jr[2], x_prev(jr[0], L), J(1, yp, z), J(2, y, zp));
  }
  auto with = [&](int m) { return __popc((m & 1 ? n.c0 : ~n.c0) & (m & 2 ? n.c1 : ~n.c1) & (m & 4 ? n.c2 : ~n.c2) & all); };
  add_counts(__popc(p[0]), __popc(p[1]), __popc(p[2]), s_cnt, s_cnt + 1, s_cnt + 2);
  add_counts(__popc(jr[0]), __popc(jr[1]), __popc(jr[2]), s_cnt + 3, s_cnt + 4, s_cnt + 5);
  // site sum 2 v - 6: 6 - v negative bonds
  add_counts(with(6), with(5), with(4), s_cnt + 10, s_cnt + 11, s_cnt + 12);
  add_counts(with(3), with(2), with(1), s_cnt + 13, s_cnt + 14, s_cnt + 15);
  const int none = with(0);
  __syncthreads();
  // an elementary cube: its three faces at i and the opposite ones; an even number is frustrated
  if (mine) n = count6(p[0], s_p[0][y + L * zn], p[1], x_next(p[1], L), p[2], s_p[2][yn + L * z]);
  add_counts(with(0), with(2), with(4), s_cnt + 6, s_cnt + 7, s_cnt + 8);
  add_counts(with(6), none, 0, s_cnt + 9, s_cnt + 16, s_cnt + 16);
  const int cap = level_capacity(N);
  const unsigned long long* H = hist + ri.level_off;
  for (int k = threadIdx.x; k < ri.K && k < cap; k += blockDim.x) {
    const unsigned long long h = H[k];
    if (h == 0ull) continue;
    const double e = (double)(ri.e_base + 4 * k) / (double)N;
    int j = (int)floor((e + 2.0) * 32.0);
    j = j < 0 ? 0 : (j > 63 ? 63 : j);
    atomicAdd(&s_bin[j], h);
  }
  __syncthreads();
  float* out = x + (int64_t)blockIdx.x * 81;
  // one quotient per lane, the moments on the second wave, the bins on the third
  const int k = threadIdx.x;
  if (k < 14) {
    const int nneg = s_cnt[3] + s_cnt[4] + s_cnt[5];
    const int num = k == 0 ? L : k < 4 ? s_cnt[k - 1] : k == 4 ? s_cnt[0] + s_cnt[1] + s_cnt[2] : k < 8 ? s_cnt[k - 2]
                  : k == 8 ? nneg : k == 9 ? nneg % 2 : s_cnt[k - 4];
    const double den = k == 0 ? 12.0 : k == 9 ? 1.0 : k == 4 || k == 8 ? 3.0 * (double)N : (double)N;
    out[k] = (float)((double)num / den);
  }
  if (k == 64) {
    const double n = (double)N;
    double sum = 0.0;
    for (int v = 0; v < 7; ++v) sum += (double)s_cnt[10 + v] * (double)(2 * v - 6);
    const double mean = sum / n;
    double m2 = 0.0, m4 = 0.0;
    for (int v = 0; v < 7; ++v) {
      const double dv = (double)(2 * v - 6) - mean;
      m2 += (double)s_cnt[10 + v] * dv * dv;
      m4 += (double)s_cnt[10 + v] * dv * dv * dv * dv;
    }
    out[14] = (float)(mean / 6.0);
    out[15] = (float)(m2 / n / 6.0);
    out[16] = (float)(m4 / n / 96.0);
  }
  if (k >= 128 && k < 192) {
    const int bin = k - 128;
    unsigned long long tot = 0ull;
    for (int j = 0; j < 64; ++j) tot += s_bin[j];
    out[17 + bin] = tot ? (float)((double)s_bin[bin] / (double)tot) : 0.0f;
  }
}

hipError_t launch_features(const RealInfo* reals, int n_real, const uint32_t* jabi, const unsigned long long* hist,
                           float* x, hipStream_t s) {
  static_assert(kMaxL * kMaxL <= 256, "a thread per row");
  hipLaunchKernelGGL(k_features, dim3(n_real), dim3(256), 0, s, reals, jabi, hist, x);
  return hipGetLastError();
}

}  // namespace nfm
