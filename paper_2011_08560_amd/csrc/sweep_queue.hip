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
// sweep against 93.6 on the scalar unit); beside others, and where speculation's second reads need the
// registers, on the scalar unit.
// (L = 6 planes are unrolled in the forms for waves alone, 12.7 us per sweep against 13.7 and, with
// speculation, 15.5 against 16.6; beside other sizes the code is too much for the instruction cache:
// five-size batch 92.8 us per sweep rolled, 94.4.)
template <bool SPEC, QueueForm FORM>
constexpr Gen queue_gen(int L) {
  if (FORM == kQueueShared || SPEC) return kGenScalar;
  return FORM == kQueueExclusive && L >= 12 ? kGenStaged : kGenVector;
}

// The next item of the queue, the same for the whole wave: in a scalar register, and with it the
// realization's record and the uniform words of the random stream.
__device__ __forceinline__ int next_item(uint32_t* __restrict__ counter) {
  __syncthreads();  // the previous item's table reads are done before the next table is loaded
  int item = 0;
  if (threadIdx.x == 0) item = (int)atomicAdd(counter, 1u);
  return __builtin_amdgcn_readfirstlane(item);
}

// SOLO: the wave claims the whole register file of its SIMD (all 256 accumulation registers besides
// its own), so no other wave shares that SIMD's issue slots while it runs; for the largest lattices,
// whose serial chains bound the batch, beside a queue over the others.
// (The registers of the form up to L = 8 let three waves share a SIMD, not four: where four fit, 3000
// waves of L = 8 come to lie by fours and twos and take 42.8 us per sweep, by threes 34.0.)
template <bool SPEC, int MAXL, bool SOLO = false>
__global__ void __launch_bounds__(64, MAXL <= 8 ? 3 : MAXL <= 10 ? 2 : 1)
    k_sweeps_queue(SweepArgs A, const int32_t* __restrict__ order, int n_items, uint32_t* __restrict__ counter) {
  extern __shared__ uint32_t stab[];
  (void)stab;
  if constexpr (SOLO) asm volatile("" ::: "a255");
  constexpr QueueForm form = SOLO ? kQueueExclusive : kQueueShared;
  for (;;) {
    const int item = next_item(counter);
    if (item >= n_items) break;
    const int wave = order[item];
    switch (A.reals[A.wave_real[wave]].L) {
      case 2: sweep_wave<2, SPEC, false, false, queue_gen<SPEC, form>(2), true>(A, wave); break;
      case 4: if constexpr (MAXL >= 4) sweep_wave<4, SPEC, false, false, queue_gen<SPEC, form>(4), true>(A, wave); break;
      case 6: if constexpr (MAXL >= 6) sweep_wave<6, SPEC, false, false, queue_gen<SPEC, form>(6), !SOLO>(A, wave); break;
      case 8: if constexpr (MAXL >= 8) sweep_wave<8, SPEC, false, false, queue_gen<SPEC, form>(8), true>(A, wave); break;
      case 10: if constexpr (MAXL >= 10) sweep_wave<10, SPEC, false, false, queue_gen<SPEC, form>(10), true>(A, wave); break;
      case 12: if constexpr (MAXL >= 12) sweep_wave<12, SPEC, false, false, queue_gen<SPEC, form>(12), true>(A, wave); break;
      default: break;
    }
  }
}

// The item loop of the lone forms as a function, each size through a generic lambda: the compiler then
// simplifies them by themselves before they join the loop and keeps less in registers across sizes (130,
// 219 and 248 for sizes up to 8, 10 and 12; 146, 249 and 256 with the calls in place), at the same speed
// for waves alone. The forms that share SIMDs lose by it (4000 waves of L = 8: 41.0 us per sweep, 43.0
// through the lambda).
template <bool SPEC, int MAXL>
__device__ __forceinline__ void lone_items(const SweepArgs& A, const int32_t* __restrict__ order, int n_items,
                                           uint32_t* __restrict__ counter) {
  for (;;) {
    const int item = next_item(counter);
    if (item >= n_items) break;
    const int wave = order[item];
    auto run = [&](auto Lc) __attribute__((always_inline)) {
      constexpr int L = decltype(Lc)::value;
      if constexpr (L <= MAXL) sweep_wave<L, SPEC, false, false, queue_gen<SPEC, kQueueLone>(L), L != 6>(A, wave);
    };
    switch (A.reals[A.wave_real[wave]].L) {
      case 2: run(std::integral_constant<int, 2>{}); break;
      case 4: run(std::integral_constant<int, 4>{}); break;
      case 6: run(std::integral_constant<int, 6>{}); break;
      case 8: run(std::integral_constant<int, 8>{}); break;
      case 10: run(std::integral_constant<int, 10>{}); break;
      case 12: run(std::integral_constant<int, 12>{}); break;
      default: break;
    }
  }
}

// For grids of at most one workgroup per SIMD: each wave has a SIMD to itself as long as nothing else
// runs, and leaves at least half of its registers to kernels of other streams (a small kernel beside a
// 10 ms launch ends after 0.03 ms; where the waves claimed their SIMDs, after the launch).
template <bool SPEC, int MAXL>
__global__ void __launch_bounds__(64, MAXL <= 8 ? 3 : 2)
    k_sweeps_queue_lone(SweepArgs A, const int32_t* __restrict__ order, int n_items, uint32_t* __restrict__ counter) {
  extern __shared__ uint32_t stab[];
  (void)stab;
  lone_items<SPEC, MAXL>(A, order, n_items, counter);
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
