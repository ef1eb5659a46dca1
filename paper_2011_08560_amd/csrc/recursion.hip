// Weight iteration on the device (Sec. II): the density-of-states estimate is refined from the
// histograms of the last sampling round, re-anchored at new minima, and turned into the next
// log-weights and threshold table, all without leaving the GPU.
//
// Estimate: DOS steps b(k) = S(k+1) - S(k), S = ln Omega up to a constant, S(k_top) = 0.
// Profiles (ln P): flat 0; power law alpha ln((E - E_g + dE)/(dE - E_g)), Eq. (5) with E_g the
// lowest energy found; 1/k: S(k) - ln sum_{j=k_lo..k} exp S(j), Eq. (7). Weights lnW = -S + ln P
// (Eqs. (3), (4)). Update (accumulated statistics, Berg's multicanonical recursion written for a
// target profile): for consecutive visited levels k < k',
//   est = [ln H(k') - lnW(k')] - [ln H(k) - lnW(k)],  g0 = H(k) H(k') / (H(k) + H(k')),
//   p(k) += g0,  b(k) += (g0 / p(k)) (est - (b(k) + ... + b(k'-1))).
//
// One block per realization. What is a chain keeps the oracle's operation order on one thread: the
// prefix S, the flatness sum and the 1/k normalization, each over values staged in LDS (a step is one
// dependent FP64 addition beside reads that run ahead). Everything else is a level or a table entry
// per thread: the logarithms and exponentials, and the step updates, since consecutive visited levels
// k < k' touch only b(k), ..., b(k' - 1) and p(k). L = 8 x 1024 realizations: 610 us on one thread per
// realization from device memory, 34 us so.
#include "kernels.hpp"
#include "table_builder.hpp"

namespace nfm {

__device__ __forceinline__ double rec_lnP_power(double E, double E_g, double dE, double alpha) {
  return alpha * log(E / (dE - E_g) + 1.0);
}

// The chains are staged kChunk levels at a time (all of a lattice's up to L = 10 at once; L = 12 has
// about 730 on [k_lo, k_top]). 12 KB for both arrays leaves the block count per compute unit to the
// waves.
constexpr int kChunk = 768;
struct RecShared {
  alignas(16) double s[kChunk], v[kChunk];
};

// acc <- acc + sign x(i) for i = 0 ... n - 1 in order, in 16-byte reads eight elements ahead of the
// additions; KEEP stores the running value in the element's place. Elements up to the next multiple
// of eight must hold 0 (adding it changes nothing).
template <bool SUB, bool KEEP>
__device__ __forceinline__ double rec_chain(double* x, int n, double acc) {
  static_assert(kChunk % 8 == 0, "chunks of whole batches");
  double2* q = reinterpret_cast<double2*>(x);
  double2 cur[4], nxt[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) cur[i] = q[i];
  for (int j = 0; j < n; j += 8, q += 4) {
    const int ahead = j + 8 < n ? 4 : 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) nxt[i] = q[ahead + i];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      acc = SUB ? acc - cur[i].x : acc + cur[i].x;
      cur[i].x = acc;
      acc = SUB ? acc - cur[i].y : acc + cur[i].y;
      cur[i].y = acc;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (KEEP) q[i] = cur[i];
      cur[i] = nxt[i];
    }
  }
  return acc;
}

// Stages b's steps of the c-th chunk of [low, k_top] counted from above, one place per level from
// k_top down; place 0 of the first chunk is S(k_top) = 0. Returns the number of levels.
__device__ __forceinline__ int rec_stage_steps(RecShared& sh, const double* b, int low, int k_top, int c) {
  const int n = min(k_top - low + 1 - c * kChunk, kChunk);
  for (int i = threadIdx.x; i < ((n + 7) & ~7); i += blockDim.x) {
    const int k = k_top - c * kChunk - i;
    sh.s[i] = i < n && k < k_top ? b[k] : 0.0;
  }
  return n;
}

// ln P and lnW on [low, k_top] from S (all threads; S visible to them). With a seeded prior also on
// [k_seed, k_lo), where S continues with the seeded steps under the frozen profile lnP(k_lo).
__device__ void rec_profile_block(RecShared& sh, const RecInfo& ri, int e_base, const double* S, double* lnP,
                                  double* lnW) {
  const int k_lo = ri.k_lo, k_top = ri.k_top, low = rec_low(ri);
  const double E_g = (double)(e_base + 4 * k_lo);
  auto power = [&](int k) { return rec_lnP_power((double)(e_base + 4 * k), E_g, ri.pl_dE, ri.pl_alpha); };
  double lp_lo = 0.0;   // lnP(k_lo)
  if (ri.profile == 1) {
    lp_lo = power(k_lo);
  } else if (ri.profile != 0) {
    double acc = 0.0;
    for (int c0 = k_lo; c0 <= k_top; c0 += kChunk) {
      const int n = min(k_top - c0 + 1, kChunk);
      __syncthreads();
      for (int i = threadIdx.x; i < n; i += blockDim.x) sh.v[i] = S[c0 + i];
      __syncthreads();
      if (threadIdx.x == 0) {
        for (int i = 0; i < n; ++i) {
          const double Sk = sh.v[i];
          if (c0 + i == k_lo) {
            acc = Sk;
          } else {
            const double m = acc > Sk ? acc : Sk;
            acc = m + log1p(exp(-fabs(acc - Sk)));
          }
          sh.v[i] = Sk - acc;
        }
      }
      __syncthreads();
      for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const double lp = sh.v[i];
        lnP[c0 + i] = lp;
        lnW[c0 + i] = -S[c0 + i] + lp;
      }
    }
    lp_lo = S[k_lo] - S[k_lo];
  }
  for (int k = low + (int)threadIdx.x; k <= k_top; k += blockDim.x) {
    if (k >= k_lo && ri.profile != 0 && ri.profile != 1) break;
    const double lp = k > k_lo && ri.profile == 1 ? power(k) : lp_lo;
    lnP[k] = lp;
    lnW[k] = -S[k] + lp;
  }
}

// S, ln P and lnW from b (all threads; b visible to them).
__device__ void rec_weights_block(RecShared& sh, const RecInfo& ri, int e_base, const double* b, double* S,
                                  double* lnP, double* lnW) {
  const int k_top = ri.k_top, low = rec_low(ri);
  double acc = 0.0;   // thread 0's
  for (int c = 0; c * kChunk <= k_top - low; ++c) {
    const int n = rec_stage_steps(sh, b, low, k_top, c);
    __syncthreads();
    if (threadIdx.x == 0) acc = rec_chain<true, true>(sh.s, n, acc);
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) S[k_top - c * kChunk - i] = sh.s[i];
    __syncthreads();
  }
  rec_profile_block(sh, ri, e_base, S, lnP, lnW);
}

// One realization per block: weights from the current estimate, table, round-trip bounds.
__global__ void k_rec_weights(RealInfo* __restrict__ reals, RecInfo* __restrict__ recs, RecArrays A,
                              uint32_t* __restrict__ tables, int set_bounds) {
  RealInfo* rp = reals + blockIdx.x;
  RecInfo* rc = recs + blockIdx.x;
  const int64_t off = rp->level_off;
  __shared__ RecShared sh;
  const RecInfo ri = *rc;
  const int e_base = rp->e_base;
  rec_weights_block(sh, ri, e_base, A.b + off, A.S + off, A.lnP + off, A.lnW + off);
  if (threadIdx.x == 0 && set_bounds) {
    rp->e_bot = e_base + 4 * ri.k_lo;
    rp->e_top = 0;
  }
  __syncthreads();
  build_table_block(rp, A.lnW + off, rec_low(ri), ri.k_top, tables);
}

// Initial state: b = p = 0, nothing visited, k_lo = lowest level of any walker's minimum.
__global__ void k_rec_init(RealInfo* __restrict__ reals, RecInfo* __restrict__ recs, RecArrays A, WalkerState ws,
                           int profile, double pl_dE, double pl_alpha) {
  RealInfo* rp = reals + blockIdx.x;
  RecInfo* rc = recs + blockIdx.x;
  const int64_t off = rp->level_off;
  const int cap = level_capacity(rp->N);
  for (int k = threadIdx.x; k < cap; k += blockDim.x) {
    A.b[off + k] = 0.0;
    A.p[off + k] = 0.0;
    A.S[off + k] = 0.0;
    A.lnP[off + k] = 0.0;
    A.lnW[off + k] = 0.0;
    A.visited[off + k] = 0;
  }
  __shared__ int s_min;
  if (threadIdx.x == 0) s_min = 0x7fffffff;
  __syncthreads();
  int m = 0x7fffffff;
  for (int w = threadIdx.x; w < rp->walkers; w += blockDim.x) m = min(m, ws.E_min[rp->walker_off + w]);
  atomicMin(&s_min, m);
  __syncthreads();
  if (threadIdx.x == 0) {
    const int k_top = (-rp->e_base + 3) / 4;  // lowest level with E >= 0
    int k_lo = (s_min - rp->e_base) / 4;
    if (k_lo > k_top) k_lo = k_top;
    rc->k_lo = k_lo;
    rc->k_top = k_top;
    rc->profile = profile;
    rc->pl_dE = pl_dE;
    rc->pl_alpha = pl_alpha;
    rc->flatness = 0.0;
    rc->converged = 0;
    rc->iterations = 0;
    rc->k_lo_changed = 0;
    rc->k_seed = -1;
    rc->pad = 0;
  }
}

// One update from the histogram of the last sampling round, then the next weights and table.
// Bound by memory latency (about ten dependent round trips) and the two chains, the prefix S on the
// first wave's first lane beside the flatness sum on the second's.
__global__ void __launch_bounds__(256) k_rec_update(RealInfo* __restrict__ reals, RecInfo* __restrict__ recs,
                                                    RecArrays A, WalkerState ws, unsigned long long* __restrict__ hist,
                                                    uint32_t* __restrict__ tables, double f_tol) {
  RealInfo* rp = reals + blockIdx.x;
  RecInfo* rc = recs + blockIdx.x;
  const int64_t off = rp->level_off;
  const RecInfo ri = *rc;
  const int e_base = rp->e_base, tid = threadIdx.x;
  unsigned long long* H = hist + off;
  double* b = A.b + off;
  double* p = A.p + off;
  const double* lnW = A.lnW + off;
  const double* lnP = A.lnP + off;
  unsigned char* visited = A.visited + off;
  const int k_lo_used = ri.k_lo, k_top = ri.k_top;
  __shared__ RecShared sh;
  constexpr int kCap = level_capacity(kMaxL * kMaxL * kMaxL);
  __shared__ unsigned long long s_hit[(kCap + 63) / 64];   // levels with counts
  __shared__ int s_min, s_n;
  __shared__ unsigned long long s_vmin;                    // (not negative: ordered as integers)
  if (tid == 0) {
    s_min = 0x7fffffff;
    s_n = 0;
    s_vmin = 0x7ff0000000000000ull;
  }
  __syncthreads();
  int mn = 0x7fffffff;
  for (int w = tid; w < rp->walkers; w += blockDim.x) mn = min(mn, ws.E_min[rp->walker_off + w]);
  for (int o = 32; o > 0; o >>= 1) mn = min(mn, __shfl_xor(mn, o));
  if ((tid & 63) == 0) atomicMin(&s_min, mn);
  for (int k0 = tid & ~63; k0 <= k_top; k0 += blockDim.x) {
    const int k = k0 + (tid & 63);
    const unsigned long long hit = __ballot(k <= k_top && H[k] != 0);
    if ((tid & 63) == 0) s_hit[k0 / 64] = hit;
  }
  __syncthreads();
  const int k_lo = min((s_min - e_base) / 4, k_lo_used);
  // new levels: the lowest known step (plain) or their seeded steps, no accumulated weight
  if (k_lo < k_lo_used) {
    for (int k = k_lo + tid; k < k_lo_used; k += blockDim.x) {
      if (ri.k_seed < 0) b[k] = b[k_lo_used];
      p[k] = 0.0;
    }
    __syncthreads();
  }
  // weights used while sampling: stored on [low, k_top], continued with the lowest step below
  const int low = rec_low(ri);
  const double d_lo = (low < k_top) ? lnW[low + 1] - lnW[low] : 0.0;
  auto lnw_at = [&](int k) {
    return k >= low ? lnW[k] : lnW[low] - (double)(low - k) * d_lo;
  };
  for (int k = k_lo + tid; k <= k_top; k += blockDim.x) {
    if (!(s_hit[k >> 6] >> (k & 63) & 1ull)) continue;
    int q = (k + 1) >> 6;   // the next level with counts
    if (q > k_top >> 6) continue;
    unsigned long long rest = s_hit[q] >> ((k + 1) & 63) << ((k + 1) & 63);
    while (rest == 0ull && q < k_top >> 6) rest = s_hit[++q];
    if (rest == 0ull) continue;
    const int kn = q * 64 + __builtin_ctzll(rest);
    const double Hk = (double)H[k], Hk1 = (double)H[kn];
    const double est = (log(Hk1) - lnw_at(kn)) - (log(Hk) - lnw_at(k));
    double span = 0.0;
    for (int j = k; j < kn; ++j) span += b[j];
    const double g0 = Hk * Hk1 / (Hk + Hk1);
    const double pk = p[k] + g0;
    p[k] = pk;
    b[k] += (g0 / pk) * (est - span);
  }
  __syncthreads();
  // flatness of H / P over the levels ever visited; S from the new steps
  RecInfo rn = ri;
  rn.k_lo = k_lo;
  const int low_new = rec_low(rn);
  const double lp_lo = lnP[k_lo_used];
  double sum = 0.0, acc = 0.0;   // the second and the first wave's first lane
  double vmin = __builtin_inf();
  int nvis = 0;
  for (int c = 0; c * kChunk <= k_top - low_new; ++c) {
    const int nv = min(k_top - k_lo + 1 - c * kChunk, kChunk);   // (below the other range: none, or negative)
    for (int i = tid; i < ((nv + 7) & ~7); i += blockDim.x) {
      const int k = k_lo + c * kChunk + i;
      double v = 0.0;
      if (i < nv) {
        const unsigned long long h = H[k];
        if (h > 0) visited[k] = 1;
        if (h > 0 || visited[k]) {
          v = (double)h / exp(k >= k_lo_used ? lnP[k] : lp_lo);
          vmin = v < vmin ? v : vmin;
          ++nvis;
        }
      }
      sh.v[i] = v;
    }
    const int n = rec_stage_steps(sh, b, low_new, k_top, c);
    __syncthreads();
    if (tid == 0) acc = rec_chain<true, true>(sh.s, n, acc);
    if (tid == 64) sum = rec_chain<false, false>(sh.v, nv, sum);
    __syncthreads();
    for (int i = tid; i < n; i += blockDim.x) A.S[off + k_top - c * kChunk - i] = sh.s[i];
    __syncthreads();
  }
  for (int o = 32; o > 0; o >>= 1) {
    const double other = __shfl_xor(vmin, o);
    vmin = other < vmin ? other : vmin;
    nvis += __shfl_xor(nvis, o);
  }
  if ((tid & 63) == 0) {
    atomicMin(&s_vmin, (unsigned long long)__double_as_longlong(vmin));
    atomicAdd(&s_n, nvis);
  }
  __syncthreads();
  if (tid == 64) {
    const double flat = (s_n > 0 && sum > 0.0) ? __longlong_as_double((long long)s_vmin) / (sum / (double)s_n) : 0.0;
    rc->k_lo_changed = (k_lo != k_lo_used);
    rc->k_lo = k_lo;
    rc->flatness = flat;
    rc->converged = (flat >= f_tol && k_lo == k_lo_used) ? 1 : 0;
    rc->iterations = ri.iterations + 1;
    // bounds for the next round
    rp->e_bot = e_base + 4 * k_lo;
    rp->e_top = 0;
  }
  // next weights (re-anchored profile)
  rec_profile_block(sh, rn, e_base, A.S + off, A.lnP + off, A.lnW + off);
  __syncthreads();
  build_table_block(rp, A.lnW + off, low_new, k_top, tables);
  const int cap = level_capacity(rp->N);
  for (int k = tid; k < cap; k += blockDim.x) H[k] = 0ull;
}

// Production weights from the final estimate (Sec. II: the DOS is determined once and reused by
// every ensemble): flat lnW = -S, power law -S + ln P_SH, 1/k -S + (S - ln sum exp S).
__global__ void k_rec_production(RealInfo* __restrict__ reals, RecInfo* __restrict__ recs, RecArrays A,
                                 uint32_t* __restrict__ tables, int profile, double pl_dE, double pl_alpha) {
  RealInfo* rp = reals + blockIdx.x;
  RecInfo* rc = recs + blockIdx.x;
  const int64_t off = rp->level_off;
  __shared__ RecShared sh;
  RecInfo ri = *rc;
  ri.profile = profile;
  ri.pl_dE = pl_dE;
  ri.pl_alpha = pl_alpha;
  const int e_base = rp->e_base;
  rec_weights_block(sh, ri, e_base, A.b + off, A.S + off, A.lnP + off, A.lnW + off);
  __syncthreads();   // all threads have read the record
  if (threadIdx.x == 0) {
    rc->profile = profile;
    rc->pl_dE = pl_dE;
    rc->pl_alpha = pl_alpha;
    rp->e_bot = e_base + 4 * ri.k_lo;
    rp->e_top = 0;
  }
  build_table_block(rp, A.lnW + off, rec_low(ri), ri.k_top, tables);
}

// Seeded prior from caller-given steps: b(k) = src(k) on [k_seed, k_top) for realizations with
// k_seed >= 0, accumulated weights cleared; others untouched.
__global__ void k_rec_seed_copy(RealInfo* __restrict__ reals, RecInfo* __restrict__ recs, RecArrays A,
                                const double* __restrict__ src, const int32_t* __restrict__ k_seed) {
  RealInfo* rp = reals + blockIdx.x;
  RecInfo* rc = recs + blockIdx.x;
  const int ks = k_seed[blockIdx.x];
  if (ks < 0) return;
  const int64_t off = rp->level_off;
  const int cap = level_capacity(rp->N);
  for (int k = threadIdx.x; k < cap; k += blockDim.x) {
    if (k >= ks && k < rc->k_top) A.b[off + k] = src[off + k];
    A.p[off + k] = 0.0;
  }
  if (threadIdx.x == 0) rc->k_seed = ks;
}

// Seeded prior from a curve y_j = [S(E) - S(E_top)]/N on the grid e_j = -2 + 2j/255 (256 floats
// per realization): S(k) = N y(E_k/N), linear between grid points, y_255 above; b(k) =
// max(S(k+1) - S(k), 0) on [k_s, k_top), k_s = the lowest level with E >= -2N. A curve with a
// step that is not finite, or without a positive step, is rejected (plain start kept;
// k_seed_out = -1).
__device__ __forceinline__ double seed_curve(const float* y, double e) {
  const double t = (e + 2.0) * 127.5;
  if (t <= 0.0) return (double)y[0];
  if (t >= 255.0) return (double)y[255];
  const int j = (int)floor(t);
  const double f = t - (double)j;
  return (double)y[j] + f * ((double)y[j + 1] - (double)y[j]);
}

__device__ __forceinline__ double seed_step(int N, int e_base, const float* y, int k) {
  const double s0 = (double)N * seed_curve(y, (double)(e_base + 4 * k) / (double)N);
  const double s1 = (double)N * seed_curve(y, (double)(e_base + 4 * (k + 1)) / (double)N);
  return s1 - s0;
}

__global__ void k_rec_seed_grid(RealInfo* __restrict__ reals, RecInfo* __restrict__ recs, RecArrays A,
                                const float* __restrict__ curves, int32_t* __restrict__ k_seed_out) {
  RealInfo* rp = reals + blockIdx.x;
  RecInfo* rc = recs + blockIdx.x;
  const float* y = curves + (int64_t)blockIdx.x * 256;
  const int N = rp->N, e_base = rp->e_base, k_top = rc->k_top;
  int k_s = (-2 * N - e_base + 3) / 4;
  if (k_s < 0) k_s = 0;
  __shared__ int s_bad;
  __shared__ double s_pos[256];
  if (threadIdx.x == 0) s_bad = 0;
  __syncthreads();
  double pos = 0.0;
  for (int k = k_s + (int)threadIdx.x; k < k_top; k += blockDim.x) {
    const double d = seed_step(N, e_base, y, k);
    if (!isfinite(d)) atomicOr(&s_bad, 1);
    if (d > 0.0) pos += d;
  }
  s_pos[threadIdx.x] = pos;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) s_pos[threadIdx.x] += s_pos[threadIdx.x + h];
    __syncthreads();
  }
  if (s_bad || !(s_pos[0] > 0.0)) {
    if (threadIdx.x == 0) k_seed_out[blockIdx.x] = -1;
    return;
  }
  const int64_t off = rp->level_off;
  for (int k = k_s + (int)threadIdx.x; k < k_top; k += blockDim.x) {
    const double d = seed_step(N, e_base, y, k);
    A.b[off + k] = d > 0.0 ? d : 0.0;
  }
  const int cap = level_capacity(N);
  for (int k = threadIdx.x; k < cap; k += blockDim.x) A.p[off + k] = 0.0;
  if (threadIdx.x == 0) {
    rc->k_seed = k_s;
    k_seed_out[blockIdx.x] = k_s;
  }
}

// Training targets from the current estimate: on the grid e_j = -2 + 2j/255, y_j = S(e_j N) / N
// with S linear between levels (S(k_top) = 0), mask 1 where e_j N >= E(k_lo) (the estimate is
// defined there), 0 and y = 0 below.
__global__ void k_rec_targets(const RealInfo* __restrict__ reals, const RecInfo* __restrict__ recs, RecArrays A,
                              float* __restrict__ y, float* __restrict__ mask) {
  const RealInfo ri = reals[blockIdx.x];
  const RecInfo rc = recs[blockIdx.x];
  const double* S = A.S + ri.level_off;
  const int j = threadIdx.x;  // 256 threads
  const double N = (double)ri.N;
  const double E = (-2.0 + 2.0 * (double)j / 255.0) * N;
  const double E_lo = (double)(ri.e_base + 4 * rc.k_lo), E_top = (double)(ri.e_base + 4 * rc.k_top);
  float yv = 0.f, mv = 0.f;
  if (E >= E_lo) {
    double v;
    if (E >= E_top) {
      v = S[rc.k_top];
    } else {
      const double t = (E - (double)ri.e_base) / 4.0;
      int k = (int)floor(t);
      if (k < rc.k_lo) k = rc.k_lo;
      if (k > rc.k_top - 1) k = rc.k_top - 1;
      const double f = t - (double)k;
      v = S[k] + f * (S[k + 1] - S[k]);
    }
    yv = (float)(v / N);
    mv = 1.f;
  }
  y[(int64_t)blockIdx.x * 256 + j] = yv;
  mask[(int64_t)blockIdx.x * 256 + j] = mv;
}

hipError_t launch_rec_targets(const RealInfo* reals, const RecInfo* recs, int n_real, RecArrays A, float* y, float* mask,
                              hipStream_t s) {
  hipLaunchKernelGGL(k_rec_targets, dim3(n_real), dim3(256), 0, s, reals, recs, A, y, mask);
  return hipGetLastError();
}

hipError_t launch_rec_seed_copy(RealInfo* reals, RecInfo* recs, int n_real, RecArrays A, const double* src,
                                const int32_t* k_seed, hipStream_t s) {
  hipLaunchKernelGGL(k_rec_seed_copy, dim3(n_real), dim3(256), 0, s, reals, recs, A, src, k_seed);
  return hipGetLastError();
}

hipError_t launch_rec_seed_grid(RealInfo* reals, RecInfo* recs, int n_real, RecArrays A, const float* curves,
                                int32_t* k_seed_out, hipStream_t s) {
  hipLaunchKernelGGL(k_rec_seed_grid, dim3(n_real), dim3(256), 0, s, reals, recs, A, curves, k_seed_out);
  return hipGetLastError();
}

hipError_t launch_rec_init(RealInfo* reals, RecInfo* recs, int n_real, RecArrays A, WalkerState ws, int profile,
                           double pl_dE, double pl_alpha, uint32_t* tables, hipStream_t s) {
  hipLaunchKernelGGL(k_rec_init, dim3(n_real), dim3(256), 0, s, reals, recs, A, ws, profile, pl_dE, pl_alpha);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_rec_weights, dim3(n_real), dim3(256), 0, s, reals, recs, A, tables, 1);
  return hipGetLastError();
}

hipError_t launch_rec_weights(RealInfo* reals, RecInfo* recs, int n_real, RecArrays A, uint32_t* tables,
                              int set_bounds, hipStream_t s) {
  hipLaunchKernelGGL(k_rec_weights, dim3(n_real), dim3(256), 0, s, reals, recs, A, tables, set_bounds);
  return hipGetLastError();
}

hipError_t launch_rec_update(RealInfo* reals, RecInfo* recs, int n_real, RecArrays A, WalkerState ws,
                             unsigned long long* hist, uint32_t* tables, double f_tol, hipStream_t s) {
  hipLaunchKernelGGL(k_rec_update, dim3(n_real), dim3(256), 0, s, reals, recs, A, ws, hist, tables, f_tol);
  return hipGetLastError();
}

hipError_t launch_rec_production(RealInfo* reals, RecInfo* recs, int n_real, RecArrays A, uint32_t* tables,
                                 int profile, double pl_dE, double pl_alpha, hipStream_t s) {
  hipLaunchKernelGGL(k_rec_production, dim3(n_real), dim3(256), 0, s, reals, recs, A, tables, profile, pl_dE,
                     pl_alpha);
  return hipGetLastError();
}

}  // namespace nfm
