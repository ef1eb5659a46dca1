// Launches of the sweep kernels: which form runs a launch, its on-chip histogram, the persistent
// grids, and small helper kernels. The kernels themselves: sweep_wave.hpp, sweep_size.hip,
// sweep_queue.hip.
#include <algorithm>
#include <cstdio>
#include <cstring>

#include "sweep_launch.hpp"
#include "sweep_wave.hpp"

namespace nfm {

// The exchange thresholds the sweep kernel uses for realization r, for inspection: [s][d - 1]
// for d = 1..D.
__global__ void k_pt_swap_table(const double* q, int r, int M, int D, uint32_t* swap) {
  const double* qr = q + (int64_t)r * kMaxReplicas;
  for (int f = blockIdx.x * blockDim.x + threadIdx.x; f < (M - 1) * D; f += gridDim.x * blockDim.x)
    swap[f] = pt_swap_threshold(qr[f / D], f % D + 1);
}

hipError_t launch_pt_swap_table(const double* q, int r, int M, int D, uint32_t* swap, hipStream_t s) {
  if (M < 2 || M > kMaxReplicas || D < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_pt_swap_table, dim3(64), dim3(256), 0, s, q, r, M, D, swap);
  return hipGetLastError();
}

__global__ void k_fill_u32(uint32_t* p, int n, uint32_t v) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

hipError_t launch_fill_u32(uint32_t* p, int n, uint32_t v, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_u32, dim3((n + 63) / 64), dim3(64), 0, s, p, n, v);
  return hipGetLastError();
}

// The sweep kernels the last launch on this host thread used (for reports): the last one's name, and
// every kernel of the launch with its compiled form, grid and LDS.
static thread_local char g_last_kernel[48] = "none";
static thread_local char g_last_launch[512] = "none";
const char* last_sweep_kernel() { return g_last_kernel; }
const char* last_sweep_launch() { return g_last_launch; }
void begin_launch() { g_last_launch[0] = '\0'; }
void note_kernel(const char* kernel, int L, const char* form, int grid, int threads, size_t lds_bytes) {
  const bool queue = strncmp(kernel, "k_sweeps_queue", 14) == 0;   // over several sizes: named without one
  snprintf(g_last_kernel, sizeof(g_last_kernel), queue ? "%s" : "%s<%d>", kernel, L);
  const size_t n = strlen(g_last_launch);
  snprintf(g_last_launch + n, sizeof(g_last_launch) - n, "%s%s<%d> %s %dx%d %zu", n ? "; " : "", kernel, L, form, grid,
           threads, lds_bytes);
}
void note_partitioned_launch(bool spec) {
  snprintf(g_last_kernel, sizeof(g_last_kernel), "%s", spec ? "k_sweeps_queue_spec_solo" : "k_sweeps_queue_solo");
}

// Levels kept on chip below the table rows and above them when the histogram is a window.
constexpr int kHistMargin = 64;

HistPlan plan_hist(const void* f, size_t base_lds, int rows, int K, int want_blocks, int mode) {
  const HistPlan full{K, K, base_lds + (size_t)K * 4};
  const int nw = std::min(K, rows + 2 * kHistMargin);
  const HistPlan win{kHistMargin, nw, base_lds + (size_t)nw * 4};
  if (mode == 1) return win;
  if (mode == 2) return full;
  if (mode == 3) return HistPlan{0, std::min(K, rows), base_lds + (size_t)std::min(K, rows) * 4};
  int occ_full = 0, occ_win = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ_full, f, 64, full.lds) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ_win, f, 64, win.lds) != hipSuccess)
    return win;
  return occ_full >= std::min(occ_win, want_blocks) ? full : win;
}

static hipError_t launch_any(int L, const SweepArgs& a, int n_waves, int lds_rows, int hist_levels, int n_cu,
                             int hist_mode, int ws_mode, bool spec, bool pt, hipStream_t s) {
  switch (L) {
    case 2: return launch_L<2>(a, n_waves, lds_rows, hist_levels, n_cu, hist_mode, ws_mode, spec, pt, s);
    case 4: return launch_L<4>(a, n_waves, lds_rows, hist_levels, n_cu, hist_mode, ws_mode, spec, pt, s);
    case 6: return launch_L<6>(a, n_waves, lds_rows, hist_levels, n_cu, hist_mode, ws_mode, spec, pt, s);
    case 8: return launch_L<8>(a, n_waves, lds_rows, hist_levels, n_cu, hist_mode, ws_mode, spec, pt, s);
    case 10: return launch_L<10>(a, n_waves, lds_rows, hist_levels, n_cu, hist_mode, ws_mode, spec, pt, s);
    case 12: return launch_L<12>(a, n_waves, lds_rows, hist_levels, n_cu, hist_mode, ws_mode, spec, pt, s);
    default: return hipErrorInvalidValue;
  }
}

bool sweep_supported(int L) { return L >= 2 && L <= kMaxL && (L % 2) == 0; }

hipError_t launch_muca_sweeps(int L, const SweepArgs& a, int n_waves, int lds_rows, int hist_levels, int n_cu,
                              int hist_mode, int ws_mode, bool spec, hipStream_t s) {
  return launch_any(L, a, n_waves, lds_rows, hist_levels, n_cu, hist_mode, ws_mode, spec, false, s);
}

static const void* queue_kernel_of(bool spec, int maxl, QueueForm form) {
  switch (form) {
    case kQueueExclusive: return spec ? queue_kernel<true, kQueueExclusive>(maxl) : queue_kernel<false, kQueueExclusive>(maxl);
    case kQueueLone: return spec ? queue_kernel<true, kQueueLone>(maxl) : queue_kernel<false, kQueueLone>(maxl);
    default: return spec ? queue_kernel<true, kQueueShared>(maxl) : queue_kernel<false, kQueueShared>(maxl);
  }
}

// LDS of the persistent kernel: the largest table, the couplings of the largest lattice and the
// histogram planned for the largest table and level count of the launch's items.
static HistPlan queue_plan(bool spec, int maxl, QueueForm form, int lds_rows, int hist_levels, int want_blocks, int mode) {
  const int jl = form == kQueueExclusive ? kMaxL : queue_maxl(maxl);
  // after the histogram, 16-byte aligned
  const size_t staged = form == kQueueExclusive && maxl >= 12 && !spec ? staged_bytes<kMaxL>() + 12 : 0;
  return plan_hist(queue_kernel_of(spec, maxl, form), (size_t)lds_rows * 32 + (size_t)jk_words(jl) * 4 + staged, lds_rows,
                   hist_levels, want_blocks, mode);
}

int queue_blocks_per_cu(bool spec, int lds_rows, int hist_levels, int hist_mode, int maxl, QueueForm form) {
  int n = 0;
  const HistPlan h = queue_plan(spec, maxl, form, lds_rows, hist_levels, 1 << 20, hist_mode);
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, queue_kernel_of(spec, maxl, form), 64, h.lds) != hipSuccess) return 0;
  return n;
}

// A grid of at most one workgroup per SIMD takes the form for waves alone where that keeps all of it
// resident (sizes 6 and 8, 1000 waves: 28.1 us per sweep, 30.7 in the shared form; sizes up to 6: 12.7
// and 14.5; with L = 12: 85.9 and 92.8).
QueueForm queue_form(bool spec, int lds_rows, int hist_levels, int hist_mode, int maxl, int64_t grid, int n_cu) {
  const bool lone = grid <= 4LL * n_cu && (int64_t)queue_blocks_per_cu(spec, lds_rows, hist_levels, hist_mode, maxl,
                                                                       kQueueLone) * n_cu >= grid;
  return lone ? kQueueLone : kQueueShared;
}

hipError_t launch_muca_queue(SweepArgs a, const int32_t* order, int n_items, uint32_t* counter, int grid, int n_cu,
                             int lds_rows, int hist_levels, int hist_mode, bool spec, hipStream_t s, int maxl,
                             QueueForm form) {
  if (grid < 1 || n_items < 0 || maxl < 2 || maxl > kMaxL) return hipErrorInvalidValue;
  const HistPlan h =
      queue_plan(spec, maxl, form, lds_rows, hist_levels, (grid + n_cu - 1) / std::max(n_cu, 1), hist_mode);
  a.hist_margin = h.margin;
  a.hist_n = h.n;
  auto launch = [&](auto* f) { return f(maxl, a, order, n_items, counter, grid, h.lds, s); };
  switch (form) {
    case kQueueExclusive: return launch(spec ? &launch_queue<true, kQueueExclusive> : &launch_queue<false, kQueueExclusive>);
    case kQueueLone: return launch(spec ? &launch_queue<true, kQueueLone> : &launch_queue<false, kQueueLone>);
    default: return launch(spec ? &launch_queue<true, kQueueShared> : &launch_queue<false, kQueueShared>);
  }
}

// A short bounded wait (six sleeps of about 8k cycles each) on one stream, so that a launch
// queued on another stream at the same moment is placed on the CUs first.
__global__ void k_hold() {
  for (int i = 0; i < 6; ++i) __builtin_amdgcn_s_sleep(127);
}

hipError_t launch_hold(hipStream_t s) {
  hipLaunchKernelGGL(k_hold, dim3(1), dim3(64), 0, s);
  return hipGetLastError();
}

hipError_t launch_pt_sweeps(int L, const SweepArgs& a, int n_waves, hipStream_t s) {
  if (a.pt_M < 2 || a.pt_M > kMaxReplicas || a.pt_spw != 64 / a.pt_M ||
      a.pt_minv != 0xFFFFFFFFu / (uint32_t)a.pt_M + 1u)
    return hipErrorInvalidValue;
  return launch_any(L, a, n_waves, 1, 0, 1, 0, 1, false, true, s);
}

}  // namespace nfm
