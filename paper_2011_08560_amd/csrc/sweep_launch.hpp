// Host side of the sweep kernels, shared by the files that instantiate them.
#pragma once
#include "kernels.hpp"

namespace nfm {

// The histogram's extent for a launch: every level of the realization when that leaves as many
// workgroups resident per CU as the window would (capped at the ones the launch needs), else the
// window [row0 - kHistMargin, row0 + rows + kHistMargin).
struct HistPlan {
  int margin, n;
  size_t lds;
};

HistPlan plan_hist(const void* f, size_t base_lds, int rows, int K, int want_blocks, int mode);

// Record a kernel of the calling host thread's last sweep launch (for reports): its name, lattice size
// (persistent kernels: the largest they are compiled for), compiled form, grid and dynamic LDS.
void note_kernel(const char* kernel, int L, const char* form, int grid, int threads, size_t lds_bytes);

// Kernels of one lattice size (sweep_size.hip, compiled once per size).
// ws_mode (expanded-table launches): 0 automatic -- the generator wave when the launch has at
// most one wave of walkers per SIMD (4 per CU) and all its workgroups stay resident -- 1 never,
// 2 always (when the expanded table is used).
template <int L>
hipError_t launch_L(SweepArgs a, int n_waves, int lds_rows, int hist_levels, int n_cu, int hist_mode, int ws_mode,
                    bool spec, bool pt, hipStream_t s);

// Persistent kernels (sweep_queue.hip, compiled once per form without and with speculation): for
// lattices up to 8, 10 or 12; the SIMD-exclusive form up to 12.
inline int queue_maxl(int maxl) { return maxl <= 8 ? 8 : maxl <= 10 ? 10 : kMaxL; }
template <bool SPEC, QueueForm FORM>
const void* queue_kernel(int maxl);
template <bool SPEC, QueueForm FORM>
hipError_t launch_queue(int maxl, const SweepArgs& a, const int32_t* order, int n_items, uint32_t* counter, int grid,
                        size_t lds_bytes, hipStream_t s);
hipError_t launch_fill_u32(uint32_t* p, int n, uint32_t v, hipStream_t s);

}  // namespace nfm
