// Lattice, coupling and spin kernels of libnfm: disorder draw (Sec. II), the
// ABI <-> kernel layout conversions, initial spins, the energy of Eq. (1) and
// the per-realization reduction of walker statistics (Sec. III).
#include <type_traits>

#include "kernels.hpp"
#include "philox.hpp"

namespace nfm {

// ---------------------------------------------------------------------------------------------
// Kernel-layout position of site (x, y, z): colour c = (x+y+z)&1, plane z, field y, bit j = x>>1.
__device__ __forceinline__ void site_pos(int L, int x, int y, int z, int* word, int* bit) {
  const int F = field_bits(L), NWP = plane_words(L);
  const int c = (x + y + z) & 1;
  const int p = y * F + (x >> 1);
  *word = (c * L + z) * NWP + (p >> 5);
  *bit = p & 31;
}

// f(L as a constant) for the lattice sizes the kernels take; one switch per wave, so that row, field
// and word positions inside are constants.
template <class F>
__device__ __forceinline__ void for_size(int L, F f) {
  switch (L) {
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 10: f(std::integral_constant<int, 10>{}); break;
    case 12: f(std::integral_constant<int, 12>{}); break;
    default: break;
  }
}

// The even-numbered bits of v, closed up to the low half.
__device__ __forceinline__ uint32_t even_bits(uint32_t v) {
  v &= 0x55555555u;
  v = (v | (v >> 1)) & 0x33333333u;
  v = (v | (v >> 2)) & 0x0F0F0F0Fu;
  v = (v | (v >> 4)) & 0x00FF00FFu;
  return (v | (v >> 8)) & 0x0000FFFFu;
}

// Sec. II: 3V couplings, each -1 with probability 1/2. Stream bit c = d*N + i is bit c%32 of
// output[m & 3] of Philox counter (m >> 2, id, 0, TAG_J), m = c/32, key = disorder seed.
// A word of a direction covers 32 consecutive stream bits, so it is cut from two stream words (one
// generator call per bit took 24 us for 1024 realizations of L = 10).
__global__ void k_gen_couplings(const RealInfo* __restrict__ reals, uint32_t* __restrict__ jabi_all,
                                uint32_t key0, uint32_t key1) {
  const RealInfo ri = reals[blockIdx.x];
  const int JW = abi_plane_words(ri.N);
  uint32_t* jabi = jabi_all + ri.jabi_off;
  for (int t = threadIdx.x; t < 3 * JW; t += blockDim.x) {
    const int d = t / JW, w = t % JW;
    const uint32_t c = (uint32_t)(d * ri.N + w * 32), m = c >> 5;
    const u32x4 r = philox4x32_10(m >> 2, ri.real_id, 0u, kTagJ, key0, key1);
    uint32_t lo = r.v[0], hi = r.v[1];
    if ((m & 3) == 1) lo = r.v[1], hi = r.v[2];
    if ((m & 3) == 2) lo = r.v[2], hi = r.v[3];
    if ((m & 3) == 3) {
      lo = r.v[3];
      hi = philox4x32_10((m >> 2) + 1u, ri.real_id, 0u, kTagJ, key0, key1).v[0];
    }
    uint32_t word = __builtin_amdgcn_alignbit(hi, lo, c & 31u);
    const int valid = ri.N - w * 32;
    if (valid < 32) word &= (1u << valid) - 1u;
    jabi[t] = word;
  }
}

// ABI couplings -> kernel layout, plus n_minus, e_base and K of the realization.
// Kernel layout of (c, z), field y, bit j (site x = 2j + phi, phi = (c+y+z)&1):
//   0 Jz(x,y,z)  1 Jz(x,y,z-1)  2 Jy(x,y,z)  3 Jy(x,y-1,z)
//   4 Jx of the partner bond (phi=0: bond x--x+1 owned by x; phi=1: bond x-1--x owned by x-1)
//   5 Jx of the other bond   (phi=0: bond x-1--x owned by x-1; phi=1: bond x--x+1 owned by x)
// A row of L bits of the ABI layout gives a row of the kernel layout by taking its even or its odd
// bits, so a word is put together row by row from words in LDS (bit by bit from device memory: 38 us
// for 1024 realizations of L = 10).
__global__ void k_pack_couplings(RealInfo* __restrict__ reals, const uint32_t* __restrict__ jabi_all,
                                 uint32_t* __restrict__ jk_all) {
  RealInfo* rp = reals + blockIdx.x;
  const int N = rp->N;
  const int JW = abi_plane_words(N);
  const uint32_t* jabi = jabi_all + rp->jabi_off;
  uint32_t* jk = jk_all + rp->jk_off;
  constexpr int kWords = abi_plane_words(kMaxL * kMaxL * kMaxL);
  __shared__ uint32_t s_j[3 * kWords + 1];   // (a row's second word may lie past the last direction)
  for (int t = threadIdx.x; t < 3 * JW + 1; t += blockDim.x) s_j[t] = t < 3 * JW ? jabi[t] : 0u;
  __syncthreads();
  for_size(rp->L, [&](auto Lc) {
    constexpr int L = decltype(Lc)::value, F = field_bits(L), NWP = plane_words(L), H = L / 2;
    constexpr uint32_t RM = (1u << H) - 1u;
    for (int t = threadIdx.x; t < 2 * L * 6 * NWP; t += blockDim.x) {
      const int w = t % NWP;
      const int kind = (t / NWP) % 6;
      const int cz = t / (6 * NWP);
      const int c = cz / L, z = cz % L;
      const int d = kind < 2 ? 2 : kind < 4 ? 1 : 0;
      const int zs = kind == 1 ? (z ? z - 1 : L - 1) : z;
      uint32_t word = 0;
      for (int y = w * 32 / F; y < L && y < (w + 1) * 32 / F; ++y) {
        const int phi = (c + y + z) & 1;
        const int ys = kind == 3 ? (y ? y - 1 : L - 1) : y;
        const int off = L * (ys + L * zs);
        const uint32_t* q = s_j + d * JW + (off >> 5);
        const uint32_t row = __builtin_amdgcn_alignbit(q[1], q[0], off & 31);
        // bonds along x: the partner's is owned by the even site, the other's by the odd one (of the
        // pair before for phi = 0)
        const int odd = kind < 4 ? phi : kind - 4;
        uint32_t f = even_bits(row >> odd) & RM;
        if (kind == 5 && phi == 0) f = ((f << 1) | (f >> (H - 1))) & RM;
        word |= f << (y * F - w * 32);
      }
      jk[t] = word;
    }
  });
  // n_minus over the 3N valid bits
  __shared__ int cnt;
  if (threadIdx.x == 0) cnt = 0;
  __syncthreads();
  int local = 0;
  for (int t = threadIdx.x; t < 3 * JW; t += blockDim.x) {
    const int w = t % JW;
    uint32_t v = s_j[t];
    const int valid = N - w * 32;
    if (valid < 32) v &= (1u << valid) - 1u;
    local += __popc(v);
  }
  atomicAdd(&cnt, local);
  __syncthreads();
  if (threadIdx.x == 0) {
    rp->n_minus = cnt;
    rp->e_base = -3 * N + 2 * (cnt & 1);
    rp->K = (3 * N - rp->e_base) / 4 + 1;
    rp->row0 = 0;   // no table: an earlier one referred to the old level set
    rp->rows = 0;
  }
}

// Initial spins: bit i of walker w is bit i%32 of output[m & 3] of counter
// (m >> 2, 0, id, (w << 8) | TAG_SPIN), m = i/32, key = walker seed; bit set <=> S = -1.
// Rows start at even bits, so the even and the odd bits of the stream hold the rows of either parity
// closed up, H = L / 2 bits each; a word of the layout takes its rows from them by position. Bound by
// the generator and the row moves, about 2000 vector instructions a walker at L = 10 (1024
// realizations x 64 walkers: 470 us bit by bit, with a generator call and a read-modify-write each;
// 8 us so).
__global__ void __launch_bounds__(64) k_gen_spins(const RealInfo* __restrict__ reals, int32_t r0, int32_t nr,
                                                  uint32_t* __restrict__ spins, uint32_t key0, uint32_t key1) {
  const int r = r0 + blockIdx.y;
  if (blockIdx.y >= (unsigned)nr) return;
  const RealInfo ri = reals[r];
  const int wl = blockIdx.x * blockDim.x + threadIdx.x;
  if (wl >= ri.walkers) return;
  uint32_t* base = spins + ri.spin_off;
  for_size(ri.L, [&](auto Lc) {
    constexpr int L = decltype(Lc)::value, N = L * L * L, F = field_bits(L), NWP = plane_words(L), H = L / 2;
    constexpr int M = abi_plane_words(N), SW = (M + 1) / 2;
    uint32_t par[2][SW];   // even and odd bits of the stream
#pragma unroll
    for (int m = 0; m < M; m += 4) {
      const u32x4 rr = philox4x32_10((uint32_t)(m / 4), 0u, ri.real_id, ((uint32_t)wl << 8) | kTagSpin, key0, key1);
#pragma unroll
      for (int i = 0; i < 4; i += 2) {
        if (m + i >= M) continue;
        par[0][(m + i) / 2] = even_bits(rr.v[i]) | even_bits(rr.v[i + 1]) << 16;
        par[1][(m + i) / 2] = even_bits(rr.v[i] >> 1) | even_bits(rr.v[i + 1] >> 1) << 16;
      }
    }
#pragma unroll
    for (int cz = 0; cz < 2 * L; ++cz) {
#pragma unroll
      for (int w = 0; w < NWP; ++w) {
        uint32_t word = 0;
#pragma unroll
        for (int y = w * 32 / F; y < L && y < (w + 1) * 32 / F; ++y) {
          const int z = cz % L, phi = (cz / L + y + z) & 1;
          const int off = H * (y + L * z), q = off >> 5, sh = off & 31;
          uint32_t row = par[phi][q] >> sh;
          if (sh + H > 32) row |= par[phi][q + 1 < SW ? q + 1 : q] << ((32 - sh) & 31);
          word |= (row & ((1u << H) - 1u)) << (y * F - w * 32);
        }
        base[(int64_t)(cz * NWP + w) * ri.walkers + wl] = word;
      }
    }
  });
}

// int8 spins (walker-major, N each) <-> kernel layout for walkers [wl0, wl0+count) of realization r.
__global__ void k_pack_spins(const RealInfo* __restrict__ reals, int32_t r, int32_t wl0, int32_t count,
                             const int8_t* __restrict__ src, uint32_t* __restrict__ spins) {
  const RealInfo ri = reals[r];
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= count) return;
  const int wl = wl0 + t, L = ri.L, WPW = walker_words(L);
  uint32_t* base = spins + ri.spin_off;
  for (int k = 0; k < WPW; ++k) base[(int64_t)k * ri.walkers + wl] = 0;
  for (int i = 0; i < ri.N; ++i) {
    int word, b;
    site_pos(L, i % L, (i / L) % L, i / (L * L), &word, &b);
    if (src[(int64_t)t * ri.N + i] < 0) base[(int64_t)word * ri.walkers + wl] |= 1u << b;
  }
}

__global__ void k_unpack_spins(const RealInfo* __restrict__ reals, int32_t r, int32_t wl0, int32_t count,
                               const uint32_t* __restrict__ spins, int8_t* __restrict__ dst) {
  const RealInfo ri = reals[r];
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= count) return;
  const int wl = wl0 + t, L = ri.L;
  const uint32_t* base = spins + ri.spin_off;
  for (int i = 0; i < ri.N; ++i) {
    int word, b;
    site_pos(L, i % L, (i / L) % L, i / (L * L), &word, &b);
    dst[(int64_t)t * ri.N + i] = ((base[(int64_t)word * ri.walkers + wl] >> b) & 1u) ? -1 : 1;
  }
}

// Field rows y + 1 (UP) or y - 1 of a plane-colour string (periodic).
template <int L, bool UP>
__device__ __forceinline__ void rows_beside(const uint32_t (&in)[plane_words(L)], uint32_t (&out)[plane_words(L)]) {
  constexpr int NWP = plane_words(L), BITS = L * field_bits(L), S = UP ? field_bits(L) : BITS - field_bits(L);
  // bit p of the result is bit (p + S) mod BITS
#pragma unroll
  for (int w = 0; w < NWP; ++w) {
    uint32_t v = 0;
#pragma unroll
    for (int k = 0; k < NWP; ++k) {
      // where input word k lands, taken once below and once above the string's end
#pragma unroll
      for (int turn = 0; turn < 2; ++turn) {
        const int at = 32 * k - S + turn * BITS - 32 * w;
        if (at > -32 && at < 32) v |= at >= 0 ? in[k] << (at & 31) : in[k] >> (-at & 31);
      }
    }
    const int valid = BITS - 32 * w;
    out[w] = valid < 32 ? v & ((1u << (valid & 31)) - 1u) : v;
  }
}

// Eq. (1): E = -sum over sites and forward directions of J S_i S_{i+e_d} = -3N + 2 (unsatisfied
// bonds). Every bond has one end of colour 0, so the six bonds of those sites are all bonds: per word
// of the colour's strings six exclusive ors and bit counts (bit by bit with divisions for each
// neighbour: 415 us for 65536 walkers of L = 10; 7 us so, bound by the latency of a wave's
// reads of the spins). Resets the walker's bookkeeping (E_min = E, no round trips, no new minimum).
__global__ void __launch_bounds__(64) k_energy(const RealInfo* __restrict__ reals, const uint32_t* __restrict__ jk_all,
                                               const uint32_t* __restrict__ spins, WalkerState ws) {
  const RealInfo ri = reals[blockIdx.y];
  const int wl = blockIdx.x * blockDim.x + threadIdx.x;
  if (wl >= ri.walkers) return;
  const uint32_t* jk = jk_all + ri.jk_off;
  const uint32_t* base = spins + ri.spin_off;
  int E = 0;
  for_size(ri.L, [&](auto Lc) {
    constexpr int L = decltype(Lc)::value, F = field_bits(L), NWP = plane_words(L), H = L / 2;
    constexpr uint32_t RM = (1u << H) - 1u;
    auto plane = [&](int c, int z, uint32_t (&v)[NWP]) {
#pragma unroll
      for (int w = 0; w < NWP; ++w) v[w] = base[(int64_t)((c * L + z) * NWP + w) * ri.walkers + wl];
    };
    int u = 0;
    uint32_t S[NWP], O[NWP], Ob[NWP], On[NWP];
    plane(1, L - 1, Ob);
    plane(1, 0, O);
#pragma unroll
    for (int z = 0; z < L; ++z) {
      plane(0, z, S);
      plane(1, (z + 1) % L, On);
      uint32_t up[NWP], dn[NWP];
      rows_beside<L, true>(O, up);
      rows_beside<L, false>(O, dn);
#pragma unroll
      for (int w = 0; w < NWP; ++w) {
        // rows of the word and those whose sites have phi = (y + z) & 1 = 0
        uint32_t all = 0, even = 0;
#pragma unroll
        for (int y = w * 32 / F; y < L && y < (w + 1) * 32 / F; ++y) {
          all |= RM << (y * F - w * 32);
          if (((y + z) & 1) == 0) even |= RM << (y * F - w * 32);
        }
        uint32_t first = 0;   // the first and the last site of each row
#pragma unroll
        for (int y = w * 32 / F; y < L && y < (w + 1) * 32 / F; ++y) first |= 1u << (y * F - w * 32);
        const uint32_t last = first << (H - 1);
        // the other neighbour along x: of the pair before (phi = 0), of the pair after (phi = 1)
        const uint32_t before = ((O[w] << 1) & all & ~first) | ((O[w] >> (H - 1)) & first);
        const uint32_t after = ((O[w] >> 1) & all & ~last) | ((O[w] << (H - 1)) & last);
        const uint32_t other = (before & even) | (after & ~even);
        const uint32_t* J = jk + z * 6 * NWP + w;
        u += __popc((S[w] ^ On[w] ^ J[0]) & all) + __popc((S[w] ^ Ob[w] ^ J[NWP]) & all) +
             __popc((S[w] ^ up[w] ^ J[2 * NWP]) & all) + __popc((S[w] ^ dn[w] ^ J[3 * NWP]) & all) +
             __popc((S[w] ^ O[w] ^ J[4 * NWP]) & all) + __popc((S[w] ^ other ^ J[5 * NWP]) & all);
      }
#pragma unroll
      for (int w = 0; w < NWP; ++w) {
        Ob[w] = O[w];
        O[w] = On[w];
      }
    }
    E = -3 * L * L * L + 2 * u;
  });
  const int64_t g = ri.walker_off + wl;
  ws.E[g] = E;
  ws.E_min[g] = E;
  ws.rt_state[g] = 0;
  ws.new_min[g] = 0;
  ws.rt_count[g] = 0;
  ws.t_first[g] = 0;
  ws.t_last[g] = 0;
}

// Per-realization integer sums over walkers (Sec. III bookkeeping): one block per realization.
__global__ void k_reduce_real(const RealInfo* __restrict__ reals, WalkerState ws, RealStatsDev* __restrict__ out) {
  const RealInfo ri = reals[blockIdx.x];
  uint64_t cnt = 0, time = 0;
  int emin = 0x7fffffff, nm = 0, with = 0;
  for (int wl = threadIdx.x; wl < ri.walkers; wl += blockDim.x) {
    const int64_t g = ri.walker_off + wl;
    const uint64_t c = ws.rt_count[g];
    cnt += c;
    if (c > 0) {
      time += ws.t_last[g] - ws.t_first[g];
      with += 1;
    }
    emin = min(emin, ws.E_min[g]);
    nm |= ws.new_min[g];
  }
  __shared__ uint64_t s_cnt[256], s_time[256];
  __shared__ int s_emin[256], s_nm[256], s_with[256];
  s_cnt[threadIdx.x] = cnt;
  s_time[threadIdx.x] = time;
  s_emin[threadIdx.x] = emin;
  s_nm[threadIdx.x] = nm;
  s_with[threadIdx.x] = with;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      s_cnt[threadIdx.x] += s_cnt[threadIdx.x + s];
      s_time[threadIdx.x] += s_time[threadIdx.x + s];
      s_emin[threadIdx.x] = min(s_emin[threadIdx.x], s_emin[threadIdx.x + s]);
      s_nm[threadIdx.x] |= s_nm[threadIdx.x + s];
      s_with[threadIdx.x] += s_with[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    RealStatsDev o;
    o.rt_count = s_cnt[0];
    o.rt_time = s_time[0];
    o.E_min = s_emin[0];
    o.new_min = s_nm[0];
    o.walkers_with_trips = s_with[0];
    o.pad = 0;
    o.reserved = 0;
    out[blockIdx.x] = o;
  }
}

// ---------------------------------------------------------------------------------------------
// Host launchers.
hipError_t launch_gen_couplings(const RealInfo* reals, int n_real, uint32_t* jabi, uint64_t seed, hipStream_t s) {
  hipLaunchKernelGGL(k_gen_couplings, dim3(n_real), dim3(64), 0, s, reals, jabi, (uint32_t)seed,
                     (uint32_t)(seed >> 32));
  return hipGetLastError();
}

hipError_t launch_pack_couplings(RealInfo* reals, int n_real, const uint32_t* jabi, uint32_t* jk, hipStream_t s) {
  hipLaunchKernelGGL(k_pack_couplings, dim3(n_real), dim3(256), 0, s, reals, jabi, jk);
  return hipGetLastError();
}

hipError_t launch_gen_spins(const RealInfo* reals, int r0, int nr, int max_walkers, uint32_t* spins, uint64_t seed,
                            hipStream_t s) {
  dim3 grid((max_walkers + 63) / 64, nr);
  hipLaunchKernelGGL(k_gen_spins, grid, dim3(64), 0, s, reals, r0, nr, spins, (uint32_t)seed, (uint32_t)(seed >> 32));
  return hipGetLastError();
}

hipError_t launch_pack_spins(const RealInfo* reals, int r, int wl0, int count, const int8_t* src, uint32_t* spins,
                             hipStream_t s) {
  hipLaunchKernelGGL(k_pack_spins, dim3((count + 63) / 64), dim3(64), 0, s, reals, r, wl0, count, src, spins);
  return hipGetLastError();
}

hipError_t launch_unpack_spins(const RealInfo* reals, int r, int wl0, int count, const uint32_t* spins, int8_t* dst,
                               hipStream_t s) {
  hipLaunchKernelGGL(k_unpack_spins, dim3((count + 63) / 64), dim3(64), 0, s, reals, r, wl0, count, spins, dst);
  return hipGetLastError();
}

hipError_t launch_energy(const RealInfo* reals, int n_real, int max_walkers, const uint32_t* jk,
                         const uint32_t* spins, WalkerState ws, hipStream_t s) {
  dim3 grid((max_walkers + 63) / 64, n_real);
  hipLaunchKernelGGL(k_energy, grid, dim3(64), 0, s, reals, jk, spins, ws);
  return hipGetLastError();
}

hipError_t launch_reduce_real(const RealInfo* reals, int n_real, WalkerState ws, RealStatsDev* out, hipStream_t s) {
  hipLaunchKernelGGL(k_reduce_real, dim3(n_real), dim3(256), 0, s, reals, ws, out);
  return hipGetLastError();
}

// Stuck-walker watch: a walker is flagged when its last completed round trip (without one: the
// clearing of its round-trip state, at sweep `since`) lies `window` or more sweeps before the
// sweep counter `now`. Stamps count attempts (sweep t, attempt a: t N + a + 1), so the age in
// whole sweeps is floor((now N - last) / N). One block per realization; flags (optional) per
// walker, the number flagged added to *count.
__global__ void k_stuck(const RealInfo* __restrict__ reals, WalkerState ws, uint64_t now, uint64_t since,
                        uint64_t window, uint8_t* __restrict__ flags, uint32_t* __restrict__ count) {
  const RealInfo ri = reals[blockIdx.x];
  const uint64_t N = (uint64_t)ri.N;
  const uint64_t end = now * N;
  uint32_t n = 0;
  for (int wl = threadIdx.x; wl < ri.walkers; wl += blockDim.x) {
    const int64_t g = ri.walker_off + wl;
    const uint64_t last = ws.rt_count[g] > 0 ? ws.t_last[g] : since * N;
    const uint64_t age = last < end ? (end - last) / N : 0;
    const bool stuck = age >= window;
    if (flags) flags[g] = stuck ? 1 : 0;
    n += stuck ? 1u : 0u;
  }
  if (n) atomicAdd(count, n);
}

hipError_t launch_stuck(const RealInfo* reals, int n_real, WalkerState ws, uint64_t now, uint64_t since,
                        uint64_t window, uint8_t* flags, uint32_t* count, hipStream_t s) {
  hipLaunchKernelGGL(k_stuck, dim3(n_real), dim3(256), 0, s, reals, ws, now, since, window, flags, count);
  return hipGetLastError();
}

// Round-trip times (Sec. III): tau_i = (sum of completed-trip time) / (number of trips) / N in
// sweeps, censored (NaN) below min_trips trips; tau_pop = mean of the uncensored tau_i. One block;
// the sum runs as a fixed-shape tree, so the result does not depend on scheduling.
__global__ void k_rt_stats(const RealInfo* __restrict__ reals, const RealStatsDev* __restrict__ st, int r0, int count,
                           uint64_t min_trips, double* __restrict__ tau, RtSummaryDev* __restrict__ out) {
  __shared__ double s_sum[256];
  __shared__ uint64_t s_trips[256];
  __shared__ int s_used[256];
  double sum = 0.0;
  uint64_t trips = 0;
  int used = 0;
  for (int i = threadIdx.x; i < count; i += blockDim.x) {
    const int r = r0 + i;
    const RealStatsDev d = st[r];
    trips += d.rt_count;
    double ti = __builtin_nan("");
    if (d.rt_count >= min_trips && d.rt_count > 0) {
      ti = (double)d.rt_time / (double)d.rt_count / (double)reals[r].N;
      sum += ti;
      used += 1;
    }
    tau[i] = ti;
  }
  s_sum[threadIdx.x] = sum;
  s_trips[threadIdx.x] = trips;
  s_used[threadIdx.x] = used;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      s_sum[threadIdx.x] += s_sum[threadIdx.x + s];
      s_trips[threadIdx.x] += s_trips[threadIdx.x + s];
      s_used[threadIdx.x] += s_used[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    RtSummaryDev o;
    o.tau_pop = s_used[0] > 0 ? s_sum[0] / (double)s_used[0] : __builtin_nan("");
    o.trips = s_trips[0];
    o.n_used = s_used[0];
    o.n_censored = count - s_used[0];
    *out = o;
  }
}

hipError_t launch_rt_stats(const RealInfo* reals, const RealStatsDev* stats, int r0, int count, uint64_t min_trips,
                           double* tau, RtSummaryDev* out, hipStream_t s) {
  hipLaunchKernelGGL(k_rt_stats, dim3(1), dim3(256), 0, s, reals, stats, r0, count, min_trips, tau, out);
  return hipGetLastError();
}

}  // namespace nfm
