// Sweep kernels of one lattice size, L = NFM_SIZE (one compilation per size, in parallel).
#include <algorithm>

#include "sweep_launch.hpp"
#include "sweep_wave.hpp"

namespace nfm {

// The sampling wave beside a generator wave. Where each wave has a SIMD, its step is bound by the chain
// from one threshold read to the next (115-125 cycles at every size with one read per attempt), so it
// reads the thresholds of both outcomes ahead (the paired form): 95 (L = 12) to 107 cycles per step.
template <int L, bool PAIRED>
__global__ void __launch_bounds__(128) k_sweeps_ws(SweepArgs A) {
  extern __shared__ uint32_t stab[];  // addressed from LDS address 0
  (void)stab;
  // the role is uniform per wave: a scalar branch, so that each wave meets only its own barriers
  const int role = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (role == 0) {
    // the sampling wave's decisions form the critical chain: its instructions go first
    __builtin_amdgcn_s_setprio(3);
    sweep_wave<L, PAIRED, false, true, kGenWave>(A, (int)blockIdx.x);
  } else {
    generate_words<L>(A, (int)blockIdx.x);
  }
}

// The uniform rounds of a form: on the scalar unit for the compact and tempering forms (usually
// several waves per SIMD, which leave it idle), except tempering at L = 2 (a sweep is eight attempts
// and an exchange, bound by its chain), L = 6 (unrolled planes, scalar registers short) and L >= 10
// (whose scalar registers spill with them: L = 10 1024 waves 44.9 us per sweep, 42.6 on the vector unit,
// 2048 waves 64.5, 63.8; L = 12 69.6, 66.6 and 1500 waves 100.6, 98.6).
// The expanded table usually means a wave alone on its SIMD: on the vector unit
// (L = 8: 125 cycles per step against 130 staged), but staged at L = 12, where the sweep's start is
// a small part of it (118 against 124). The compact form of L = 12 comes on the vector unit and
// staged (launch_L chooses).
template <int L, bool SPEC, bool PT, bool XT>
constexpr Gen gen_of() {
  if (XT) return L >= 12 ? kGenStaged : kGenVector;
  if (L >= 12 && !SPEC && !PT) return kGenVector;
  return PT && (L == 2 || L == 6 || L >= 10) ? kGenVector : kGenScalar;
}

template <int L, bool SPEC, bool PT, bool XT, Gen GEN>
__global__ void __launch_bounds__(64) k_sweeps(SweepArgs A) {
  extern __shared__ uint32_t stab[];  // addressed from LDS address 0 by sweep_wave
  (void)stab;
  sweep_wave<L, SPEC, PT, XT, GEN>(A, (int)blockIdx.x);
}

template <int L, bool SPEC, bool PT, bool XT = false, Gen GEN = gen_of<L, SPEC, PT, XT>()>
static hipError_t launch_LS(const SweepArgs& a, int n_waves, size_t lds_bytes, hipStream_t s) {
  // The kernel addresses its dynamic LDS block from address 0, which is only valid
  // when the compiler placed nothing else in LDS.
  static int checked = 0;
  if (!checked) {
    hipFuncAttributes attr;
    hipError_t e = hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(&k_sweeps<L, SPEC, PT, XT, GEN>));
    if (e != hipSuccess) return e;
    if (attr.sharedSizeBytes != 0) return hipErrorInvalidKernelFile;
    checked = 1;
  }
  note_kernel(PT ? "k_sweeps_pt" : SPEC ? "k_sweeps_spec" : XT ? "k_sweeps_xt" : "k_sweeps", L,
              GEN == kGenStaged ? "staged" : GEN == kGenScalar ? "scalar" : "vector", n_waves, 64, lds_bytes);
  hipLaunchKernelGGL((k_sweeps<L, SPEC, PT, XT, GEN>), dim3(n_waves), dim3(64), lds_bytes, s, a);
  return hipGetLastError();
}

template <int L, bool PAIRED>
static hipError_t launch_ws(const SweepArgs& a, int n_waves, size_t lds_bytes, bool spec, hipStream_t s) {
  static int checked = 0;
  if (!checked) {
    hipFuncAttributes attr;
    hipError_t e = hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(&k_sweeps_ws<L, PAIRED>));
    if (e != hipSuccess) return e;
    if (attr.sharedSizeBytes != 0) return hipErrorInvalidKernelFile;
    checked = 1;
  }
  note_kernel(spec ? "k_sweeps_ws_spec" : "k_sweeps_ws", L, PAIRED ? "paired" : "single", n_waves, 128, lds_bytes);
  hipLaunchKernelGGL((k_sweeps_ws<L, PAIRED>), dim3(n_waves), dim3(128), lds_bytes, s, a);
  return hipGetLastError();
}

template <int L>
hipError_t launch_L(SweepArgs a, int n_waves, int lds_rows, int hist_levels, int n_cu, int hist_mode,
                           int ws_mode, bool spec, bool pt, hipStream_t s) {
  const size_t jb = (size_t)jk_words(L) * 4;
  if (pt) return launch_LS<L, false, true>(a, n_waves, (size_t)a.pt_M * 32 + 3 * 256 + jb, s);
  const void* f = spec ? reinterpret_cast<const void*>(&k_sweeps<L, true, false, false, gen_of<L, true, false, false>()>)
                       : reinterpret_cast<const void*>(&k_sweeps<L, false, false, false, gen_of<L, false, false, false>()>);
  const int want = (n_waves + n_cu - 1) / std::max(n_cu, 1);
  const HistPlan h = plan_hist(f, (size_t)lds_rows * 32 + jb, lds_rows, hist_levels, want, hist_mode);   // table, couplings
  if (hist_mode == 0) {
    // the expanded table (and every level of the histogram) when it costs no resident workgroups
    const void* fx = reinterpret_cast<const void*>(&k_sweeps<L, false, false, true, gen_of<L, false, false, true>()>);
    const size_t lds_x = staged_base((uint32_t)((size_t)hist_levels * 32 + jb), hist_levels) + (L >= 12 ? staged_bytes<L>() : 0);
    int occ_x = 0, occ = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ_x, fx, 64, lds_x) == hipSuccess &&
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, f, 64, h.lds) == hipSuccess && occ_x >= std::min(occ, want)) {
      if (ws_mode != 1) {
        const size_t lds_w = (size_t)ws_ring_base(hist_levels, jk_words(L), hist_levels) + 3 * (size_t)ws_slot_bytes<L>();
        const void* fw = reinterpret_cast<const void*>(&k_sweeps_ws<L, true>);
        int occ_w = 0;
        const bool fits = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ_w, fw, 128, lds_w) == hipSuccess &&
                          occ_w >= want;
        if (ws_mode == 2 ? occ_w >= 1 : (fits && n_waves <= 4 * n_cu)) {
          a.hist_margin = hist_levels;
          a.hist_n = hist_levels;
          // With more pairs of waves than half the SIMDs, waves share SIMDs, and the paired form's more
          // instructions (34.0 per step of a pair against 30.2) wait for each other: L = 6 then reads
          // once, at the 122 cycles per step of that form's chain with a SIMD of its own or shared
          // (1024 waves: 120, paired 124; paired alone 107). L = 4 (116 paired, 119 read once) and L = 8
          // (768 waves: 108 paired, 121 read once) stay paired; beyond L = 8 so many pairs do not fit in
          // LDS.
          if constexpr (L == 6)
            if (!spec && n_waves > 2 * n_cu) return launch_ws<L, false>(a, n_waves, lds_w, spec, s);
          return launch_ws<L, true>(a, n_waves, lds_w, spec, s);
        }
      }
      if (!spec) {
        a.hist_margin = hist_levels;
        a.hist_n = hist_levels;
        return launch_LS<L, false, false, true>(a, n_waves, lds_x, s);
      }
    }
  }
  if constexpr (L >= 12) {
    // Staged words take 6.9 KB of LDS: only where several waves share a SIMD (its issue slots, not a
    // wave's chain, bind) and no resident workgroup is lost. 1300 waves, tables of 400 rows: 127.4 us
    // per sweep staged, 133.4 on the vector unit; 600 rows (5 per compute unit staged, 6 not): 175.9,
    // 135.0. Waves alone: 512 waves, 677 rows 90.8 staged, 88.1 on the vector unit.
    if (!spec) {
      const void* fs = reinterpret_cast<const void*>(&k_sweeps<L, false, false, false, kGenStaged>);
      const size_t words = staged_bytes<L>() + 12;   // after the histogram, 16-byte aligned
      const HistPlan hs = plan_hist(fs, (size_t)lds_rows * 32 + jb + words, lds_rows, hist_levels, want, hist_mode);
      int occ_s = 0, occ = 0;
      if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ_s, fs, 64, hs.lds) == hipSuccess &&
          hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, f, 64, h.lds) == hipSuccess &&
          std::min(occ, want) > 4 && occ_s >= std::min(occ, want)) {
        a.hist_margin = hs.margin;
        a.hist_n = hs.n;
        return launch_LS<L, false, false, false, kGenStaged>(a, n_waves, hs.lds, s);
      }
    }
  }
  a.hist_margin = h.margin;
  a.hist_n = h.n;
  return spec ? launch_LS<L, true, false>(a, n_waves, h.lds, s) : launch_LS<L, false, false>(a, n_waves, h.lds, s);
}

template hipError_t launch_L<NFM_SIZE>(SweepArgs, int, int, int, int, int, int, bool, bool, hipStream_t);

}  // namespace nfm
