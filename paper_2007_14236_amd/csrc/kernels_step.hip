// kernels_step.hip -- step kernels of LIF networks, the choice of the step
// kernel, and the small kernels beside it.
#include <mutex>

#include "step_dev.h"

namespace snn {

namespace {

__global__ void k_advance(Ctrl* ctrl, uint32_t steps) {
  if (threadIdx.x == 0 && blockIdx.x == 0) ctrl->step_base += steps;
}

__global__ void __launch_bounds__(kB) k_poisson_counts(NetDev nd, uint64_t step, uint32_t first, uint32_t n,
                                                       uint32_t* out) {
  const uint32_t j = blockIdx.x * kB + threadIdx.x;
  if (j >= n) return;
  const uint32_t i = first + j;
  const PopDev& pp = nd.pops[find_pop(nd.pops, nd.npop, i)];
  out[j] = (pp.pois >= 0) ? poisson_draw(nd.pois_thr + (size_t)pp.pois * kPoisKmax, pp.seed, i - pp.gid_base, step) : 0u;
}

// Readback of the binned input pending in input buffer buf, on one port, for
// gids [first, first + n): block = one tile, entries decoded and added to
// out[gid - first] (which holds the tile's spill already).
__global__ void __launch_bounds__(kB) k_pending_input(NetDev nd, uint32_t buf, uint32_t first, uint32_t n,
                                                      uint32_t port, int64_t* out) {
  const uint32_t t = (first >> nd.tile_shift) + blockIdx.x;
  const uint32_t tfirst = t << nd.tile_shift;
  const size_t ti = (size_t)buf * nd.n_tiles + t;
  const uint32_t cnt = min(nd.bin_cnt[ti], nd.bin_cap[t]);
  const uint32_t* bin = nd.bins + (size_t)buf * nd.bins_total + nd.bin_off[t];
  for (uint32_t j = threadIdx.x; j < cnt; j += kB) {
    const uint32_t e = bin[j];
    const uint32_t cls = e & (uint32_t)(kMaxClasses - 1);
    const uint32_t gid = tfirst + (e >> kBinLocalShift);
    if (cls >= nd.n_classes || gid < first || gid - first >= n || nd.cls_port[cls] != port) continue;
    const int64_t v = nd.cls_wq[cls] * (int64_t)((e >> kBinMultShift) & kMaxMult);
    atomicAdd((unsigned long long*)&out[gid - first], (unsigned long long)v);
  }
}

}  // namespace

const char* step_kernel(const NetDev& nd) {
  if (nd.small_row) return "k_small";
  if (nd.n_pull) return "k_pull";
  if (nd.n_strips) return "k_step_strip";
  if (!nd.n_tiles) return "k_step";
  return nd.tile_runs ? "k_step_binned_runs" : "k_step_binned";
}

hipError_t launch_step(const NetDev& nd, uint32_t rel, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  const dim3 blk(kB), grid((nd.n_tiles ? nd.n_tiles : nd.nblk_upd) + nd.sel_grid);
  const bool lif = nd.pad0 & 1u, adex = nd.pad0 & 2u, beta = nd.pad0 & 4u;
  const bool plastic = nd.n_rules != 0;
  if (nd.n_pull) {
    launch_pull_step(nd, rel, s, start, stop);
    return hipGetLastError();
  }
  if (nd.n_strips) return launch_strip_step(nd, rel, s, start, stop);
  if (adex || (nd.n_tiles && !nd.tile_win)) {  // or a tile overlaps more populations than its LDS window holds
    auto f = beta ? (plastic ? launch_adex_beta_plastic : launch_adex_beta)
                  : (plastic ? launch_adex_exp_plastic : launch_adex_exp);
    f(nd, grid, s, start, stop, rel, lif);
  } else if (!nd.n_tiles) {
    launch(plastic ? k_step<true, 0, 1, true> : k_step<true, 0, 1, false>, grid, blk, s, start, stop, nd, rel);
  } else if (nd.tile_runs) {
    launch(k_step_binned_runs<true, 0, 1>, grid, blk, s, start, stop, nd, rel);
  } else {
    launch(plastic ? k_step_binned<true, 0, 1, true> : k_step_binned<true, 0, 1, false>, grid, blk, s, start, stop, nd,
           rel);
  }
  return hipGetLastError();
}

hipError_t launch_advance(Ctrl* ctrl, uint32_t steps, hipStream_t s) {
  hipLaunchKernelGGL(k_advance, dim3(1), dim3(64), 0, s, ctrl, steps);
  return hipGetLastError();
}

hipError_t launch_pending_input(const NetDev& nd, uint32_t buf, uint32_t first, uint32_t n, uint32_t port,
                                int64_t* out, hipStream_t s) {
  if (n == 0 || nd.n_tiles == 0 || nd.n_pull) return hipSuccess;  // pulled: no bins
  const uint32_t t0 = first >> nd.tile_shift, t1 = (first + n - 1) >> nd.tile_shift;
  hipLaunchKernelGGL(k_pending_input, dim3(t1 - t0 + 1), dim3(kB), 0, s, nd, buf, first, n, port, out);
  return hipGetLastError();
}

// Workspace of the allocation-free input readback: a file-scope device array.
// Host code must not pass its name to a kernel or a copy (on the host the name
// is only a stand-in); the device address comes from hipGetSymbolAddress, once
// per device with that device current, and is kept per device.
static __device__ __align__(256) int64_t scratch[kNoAllocInputMax];

namespace {
std::mutex g_ws_mu;
int64_t* g_ws_ptr[kMaxDevices] = {};
}  // namespace

hipError_t input_workspace(int device, bool resolve, int64_t** out) {
  *out = nullptr;
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_ws_mu);
  if (!g_ws_ptr[device] && resolve) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_ws_ptr[device] = static_cast<int64_t*>(p);
  }
  *out = g_ws_ptr[device];
  return hipSuccess;
}

hipError_t launch_poisson_counts(const NetDev& nd, uint64_t step, uint32_t first, uint32_t n, uint32_t* k,
                                 hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_poisson_counts, dim3((n + kB - 1) / kB), dim3(kB), 0, s, nd, step, first, n, k);
  return hipGetLastError();
}

}  // namespace snn
