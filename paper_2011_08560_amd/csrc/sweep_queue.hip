// Persistent sweep kernels over batches of mixed lattice size, without (NFM_SPEC = 0) or with
// (1) speculative table reads (one compilation each, in parallel).
#include "sweep_launch.hpp"
#include "sweep_wave.hpp"

namespace nfm {

// Persistent multicanonical launch over a batch of mixed lattice sizes: each workgroup takes
// work items (one wave of walkers for this launch's sweeps) from a global counter until the
// queue is empty. The queue lists waves longest-first (by N), so the last items to start are
// the cheapest ones. Results do not depend on which workgroup runs which item.
// MAXL: the largest lattice the launch's items have (a launch over small lattices only holds
// fewer registers per wave, so more waves stay resident). SOLO: the wave claims the whole
// register file of its SIMD (all 256 accumulation registers besides its own), so no other wave
// shares that SIMD's issue slots while it runs; for the largest lattices, whose serial chains
// bound the batch.
// The uniform rounds: a wave alone on its SIMD takes them on the vector unit, at L = 12 staged (89.5 us
// per sweep against 93.6 on the scalar unit); beside others, and where speculation's second reads need
// the registers, on the scalar unit.
// (L = 6 planes are unrolled in the form for waves alone, 13.1 us per sweep against 13.7; beside other
// sizes the code is too much for the instruction cache: five-size batch 92.8 us per sweep rolled, 94.4.)
template <bool SPEC, bool SOLO>
constexpr Gen queue_gen(int L) { return !SOLO || SPEC ? kGenScalar : L >= 12 ? kGenStaged : kGenVector; }

template <bool SPEC, int MAXL, bool SOLO = false>
__global__ void __launch_bounds__(64, MAXL <= 8 ? 3 : MAXL <= 10 ? 2 : 1) k_sweeps_queue(SweepArgs A, const int32_t* __restrict__ order, int n_items,
                                                     uint32_t* __restrict__ counter) {
  extern __shared__ uint32_t stab[];
  (void)stab;
  if constexpr (SOLO) asm volatile("" ::: "a255");
  for (;;) {
    __syncthreads();  // the previous item's table reads are done before the next table is loaded
    int item = 0;
    if (threadIdx.x == 0) item = (int)atomicAdd(counter, 1u);
    // the item is the same for the whole wave: in a scalar register, and with it the realization's
    // record and the uniform words of the random stream
    item = __builtin_amdgcn_readfirstlane(item);
    if (item >= n_items) break;
    const int wave = order[item];
    switch (A.reals[A.wave_real[wave]].L) {
      case 2: sweep_wave<2, SPEC, false, false, queue_gen<SPEC, SOLO>(2), true>(A, wave); break;
      case 4: if constexpr (MAXL >= 4) sweep_wave<4, SPEC, false, false, queue_gen<SPEC, SOLO>(4), true>(A, wave); break;
      case 6: if constexpr (MAXL >= 6) sweep_wave<6, SPEC, false, false, queue_gen<SPEC, SOLO>(6), !SOLO>(A, wave); break;
      case 8: if constexpr (MAXL >= 8) sweep_wave<8, SPEC, false, false, queue_gen<SPEC, SOLO>(8), true>(A, wave); break;
      case 10: if constexpr (MAXL >= 10) sweep_wave<10, SPEC, false, false, queue_gen<SPEC, SOLO>(10), true>(A, wave); break;
      case 12: if constexpr (MAXL >= 12) sweep_wave<12, SPEC, false, false, queue_gen<SPEC, SOLO>(12), true>(A, wave); break;
      default: break;
    }
  }
}

template <bool SPEC>
const void* queue_kernel_S(int maxl, bool solo) {
  if (solo) return reinterpret_cast<const void*>(&k_sweeps_queue<SPEC, kMaxL, true>);
  switch (queue_maxl(maxl)) {
    case 8: return reinterpret_cast<const void*>(&k_sweeps_queue<SPEC, 8>);
    case 10: return reinterpret_cast<const void*>(&k_sweeps_queue<SPEC, 10>);
    default: return reinterpret_cast<const void*>(&k_sweeps_queue<SPEC, kMaxL>);
  }
}

template <bool SPEC, int MAXL, bool SOLO>
static hipError_t launch_queue_S(const SweepArgs& a, const int32_t* order, int n_items, uint32_t* counter, int grid,
                                 size_t lds_bytes, hipStream_t s) {
  static int checked = 0;
  if (!checked) {
    hipFuncAttributes attr;
    hipError_t e = hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(&k_sweeps_queue<SPEC, MAXL, SOLO>));
    if (e != hipSuccess) return e;
    if (attr.sharedSizeBytes != 0) return hipErrorInvalidKernelFile;
    checked = 1;
  }
  hipError_t e = launch_fill_u32(counter, 1, 0u, s);
  if (e != hipSuccess) return e;
  note_kernel(SPEC ? "k_sweeps_queue_spec" : "k_sweeps_queue", MAXL, SOLO ? "exclusive" : "shared", grid, 64, lds_bytes);
  hipLaunchKernelGGL((k_sweeps_queue<SPEC, MAXL, SOLO>), dim3(grid), dim3(64), lds_bytes, s, a, order, n_items,
                     counter);
  return hipGetLastError();
}

template <bool SPEC>
hipError_t launch_queue_M(int maxl, bool solo, const SweepArgs& a, const int32_t* order, int n_items,
                                 uint32_t* counter, int grid, size_t lds_bytes, hipStream_t s) {
  if (solo) return launch_queue_S<SPEC, kMaxL, true>(a, order, n_items, counter, grid, lds_bytes, s);
  switch (queue_maxl(maxl)) {
    case 8: return launch_queue_S<SPEC, 8, false>(a, order, n_items, counter, grid, lds_bytes, s);
    case 10: return launch_queue_S<SPEC, 10, false>(a, order, n_items, counter, grid, lds_bytes, s);
    default: return launch_queue_S<SPEC, kMaxL, false>(a, order, n_items, counter, grid, lds_bytes, s);
  }
}

template const void* queue_kernel_S<NFM_SPEC != 0>(int, bool);
template hipError_t launch_queue_M<NFM_SPEC != 0>(int, bool, const SweepArgs&, const int32_t*, int, uint32_t*, int, size_t,
                                                  hipStream_t);

}  // namespace nfm
