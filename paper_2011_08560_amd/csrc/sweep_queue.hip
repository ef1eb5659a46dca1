// Persistent sweep kernels over batches of mixed lattice size: one compilation, in parallel, for each
// of the forms (NFM_FORM, a QueueForm) without (NFM_SPEC = 0) and with (1) speculative table reads.
#include "sweep_launch.hpp"
#include "sweep_wave.hpp"

namespace nfm {

// Persistent multicanonical launch over a batch of mixed lattice sizes: each workgroup takes
// work items (one wave of walkers for this launch's sweeps) from a global counter until the
// queue is empty. The queue lists waves longest-first (by N), so the last items to start are
// the cheapest ones. Results do not depend on which workgroup runs which item.
// MAXL: the largest lattice the launch's items have (a launch over small lattices only holds
// fewer registers per wave, so more waves stay resident).
// The uniform rounds: waves alone on their SIMDs take them on the vector unit (L = 12: 86 us per
// sweep, 91 staged, 92 on the scalar unit), in the SIMD-exclusive form staged at L = 12 (89.5 us per
// sweep against 93.6 on the scalar unit; 88.6 since the window checks come every 32 attempts); beside
// others, and where speculation's second reads need the registers, on the scalar unit.
// (L = 6 planes are unrolled in the forms for waves alone, 12.7 us per sweep against 13.7 and, with
// speculation, 15.5 against 16.6; beside other sizes the code is too much for the instruction cache:
// five-size batch 92.8 us per sweep rolled, 94.4.)
template <bool SPEC, QueueForm FORM>
constexpr Gen queue_gen(int L) {
  if (FORM == kQueueShared || SPEC) return kGenScalar;
  return FORM == kQueueExclusive && L >= 12 ? kGenStaged : kGenVector;
}

template <bool SPEC, int MAXL, QueueForm FORM>
__device__ __forceinline__ void queue_items(const SweepArgs& A, const int32_t* __restrict__ order, int n_items,
                                            uint32_t* __restrict__ counter) {
  for (;;) {
    __syncthreads();  // the previous item's table reads are done before the next table is loaded
    int item = 0;
    if (threadIdx.x == 0) item = (int)atomicAdd(counter, 1u);
    // the item is the same for the whole wave: in a scalar register, and with it the realization's
    // record and the uniform words of the random stream
    item = __builtin_amdgcn_readfirstlane(item);
    if (item >= n_items) break;
    const int wave = order[item];
    auto run = [&](auto Lc, auto roll) __attribute__((always_inline)) {
      constexpr int L = decltype(Lc)::value;
      if constexpr (L <= MAXL) sweep_wave<L, SPEC, false, false, queue_gen<SPEC, FORM>(L), decltype(roll)::value>(A, wave);
    };
    using std::integral_constant;
    switch (A.reals[A.wave_real[wave]].L) {
      case 2: run(integral_constant<int, 2>{}, std::true_type{}); break;
      case 4: run(integral_constant<int, 4>{}, std::true_type{}); break;
      case 6: run(integral_constant<int, 6>{}, std::bool_constant<FORM == kQueueShared>{}); break;
      case 8: run(integral_constant<int, 8>{}, std::true_type{}); break;
      case 10: run(integral_constant<int, 10>{}, std::true_type{}); break;
      case 12: run(integral_constant<int, 12>{}, std::true_type{}); break;
      default: break;
    }
  }
}

// SOLO: the wave claims the whole register file of its SIMD (all 256 accumulation registers besides
// its own), so no other wave shares that SIMD's issue slots while it runs; for the largest lattices,
// whose serial chains bound the batch, beside a queue over the others.
template <bool SPEC, int MAXL, bool SOLO = false>
__global__ void __launch_bounds__(64, MAXL <= 8 ? 3 : MAXL <= 10 ? 2 : 1)
    k_sweeps_queue(SweepArgs A, const int32_t* __restrict__ order, int n_items, uint32_t* __restrict__ counter) {
  extern __shared__ uint32_t stab[];
  (void)stab;
  if constexpr (SOLO) asm volatile("" ::: "a255");
  queue_items<SPEC, MAXL, SOLO ? kQueueExclusive : kQueueShared>(A, order, n_items, counter);
}

// For grids of at most one workgroup per SIMD: each wave has a SIMD to itself as long as nothing else
// runs, and leaves at least half of its registers to kernels of other streams (a small kernel beside a
// 10 ms launch ends after 0.03 ms; where the waves claimed their SIMDs, after the launch).
template <bool SPEC, int MAXL>
__global__ void __launch_bounds__(64, MAXL <= 8 ? 3 : 2)
    k_sweeps_queue_lone(SweepArgs A, const int32_t* __restrict__ order, int n_items, uint32_t* __restrict__ counter) {
  extern __shared__ uint32_t stab[];
  (void)stab;
  queue_items<SPEC, MAXL, kQueueLone>(A, order, n_items, counter);
}

template <bool SPEC, QueueForm FORM, int MAXL>
static constexpr auto queue_kernel_of() {
  if constexpr (FORM == kQueueLone) return &k_sweeps_queue_lone<SPEC, MAXL>;
  else return &k_sweeps_queue<SPEC, MAXL, FORM == kQueueExclusive>;
}

// f(MAXL as a constant) for the kernel that takes lattices up to maxl (SIMD-exclusive: one for all)
template <QueueForm FORM, class F>
static auto for_maxl(int maxl, F f) {
  if constexpr (FORM != kQueueExclusive) {
    if (queue_maxl(maxl) == 8) return f(std::integral_constant<int, 8>{});
    if (queue_maxl(maxl) == 10) return f(std::integral_constant<int, 10>{});
  }
  return f(std::integral_constant<int, kMaxL>{});
}

template <bool SPEC, QueueForm FORM>
const void* queue_kernel(int maxl) {
  return for_maxl<FORM>(maxl, [](auto M) { return reinterpret_cast<const void*>(queue_kernel_of<SPEC, FORM, M>()); });
}

template <bool SPEC, QueueForm FORM>
hipError_t launch_queue(int maxl, const SweepArgs& a, const int32_t* order, int n_items, uint32_t* counter, int grid,
                        size_t lds_bytes, hipStream_t s) {
  return for_maxl<FORM>(maxl, [&](auto M) {
    constexpr auto kernel = queue_kernel_of<SPEC, FORM, M>();
    static int checked = 0;
    if (!checked) {
      hipFuncAttributes attr;
      hipError_t e = hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(kernel));
      if (e != hipSuccess) return e;
      if (attr.sharedSizeBytes != 0) return hipErrorInvalidKernelFile;
      checked = 1;
    }
    hipError_t e = launch_fill_u32(counter, 1, 0u, s);
    if (e != hipSuccess) return e;
    note_kernel(SPEC ? "k_sweeps_queue_spec" : "k_sweeps_queue", M,
                FORM == kQueueExclusive ? "exclusive" : FORM == kQueueLone ? "lone" : "shared", grid, 64, lds_bytes);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(64), lds_bytes, s, a, order, n_items, counter);
    return hipGetLastError();
  });
}

template const void* queue_kernel<NFM_SPEC != 0, (QueueForm)NFM_FORM>(int);
template hipError_t launch_queue<NFM_SPEC != 0, (QueueForm)NFM_FORM>(int, const SweepArgs&, const int32_t*, int, uint32_t*,
                                                                     int, size_t, hipStream_t);

}  // namespace nfm
