// kernels.h -- host-callable launchers of the device kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "snn_types.h"

namespace snn {

// ---- connectivity build ----
// Weight levels of one projection (empty: its single weight): the class of
// level j onto a target of population k is cls[(k - pop0) * levels + j];
// drawn projections take j from thr (u32 draws), lists from lvl[synapse].
struct ProjW {
  const uint64_t* thr;
  const uint16_t* cls;
  const uint16_t* lvl;
  uint32_t levels, pop0;
};

// total_pairs = sum over projections of tgt_n * ceil(K / 2)
hipError_t launch_gen_count(const ProjDev* projs, uint32_t nproj, uint64_t total_pairs, uint32_t dmax_cfg,
                            uint32_t D1, uint32_t* cnt, hipStream_t s);
hipError_t launch_gen_scatter(const ProjDev* projs, uint32_t nproj, uint64_t total_pairs, uint32_t dmax_cfg,
                              uint32_t D1, uint64_t* cursor, uint32_t* payload, const uint16_t* cls_of,
                              const ProjW* pw, const uint32_t* pop_first, uint32_t npop, uint32_t cls_bits,
                              hipStream_t s);
// exclusive scan of n u32 (in32) or u64 (in64) values into out; *total_dev receives the sum.
// tmp must hold scan_tmp_words(n) u64 words.
size_t scan_tmp_words(uint64_t n);
hipError_t launch_scan_u32(const uint32_t* in, uint64_t n, uint64_t* out, uint64_t* tmp, hipStream_t s);
hipError_t launch_scan_u64(const uint64_t* in, uint64_t n, uint64_t* out, uint64_t* tmp, hipStream_t s);
hipError_t launch_masks(const uint32_t* cnt, uint32_t N, uint32_t D1, uint64_t* mask, uint64_t* ngroups,
                        uint32_t* longest, hipStream_t s);  // longest (or null): synapses of a source, at most
hipError_t launch_grp_off(const uint32_t* cnt, const uint64_t* off, const uint64_t* grp_ptr64, uint32_t N,
                          uint32_t D1, uint64_t* grp_off, uint32_t* grp_ptr32, hipStream_t s);
// Bins of consecutive sources that the synapses of a large network are drawn
// into: sources [first[b], first[b + 1]), places off[b] .. off[b] + cap[b] of
// rec (source in the bin << 6 | delay, payload), cnt[b] taken; *over is set when
// one was full.  words: most (source, delay) counters of a bin.
struct BinBuild {
  uint32_t nbin, words;
  const uint32_t* first;    // [nbin + 1]
  const uint16_t* of_src;   // [N]
  const uint64_t* off;      // [nbin]
  const uint32_t* cap;      // [nbin]
  uint32_t* cnt;            // [nbin], zeroed by the caller
  uint32_t* over;
  uint32_t* longest;        // longest row, from launch_masks
  uint2* rec;
};
hipError_t launch_bin_gen(const ProjDev* projs, uint32_t nproj, uint64_t total_pairs, uint32_t dmax_cfg,
                          const uint16_t* cls_of, const ProjW* pw, const uint32_t* pop_first, uint32_t npop,
                          uint32_t cls_bits, const BinBuild& bb, hipStream_t s);
hipError_t launch_bin_count(const BinBuild& bb, uint32_t D1, uint32_t* cnt, hipStream_t s);
hipError_t launch_bin_place(const BinBuild& bb, uint32_t D1, const uint64_t* off, uint32_t* payload, hipStream_t s);
// sort every group's payload ascending; longer: list of segsort_list entries
// for groups beyond a wave's (*n_longer zeroed by the caller); groups longer
// than 16384 are listed in big[] (count in *nbig)
// rows: the words are in place by source only (launch_bin_rows), their delays in
// del; otherwise (del null) by group.
struct RowSort {
  const uint8_t* del = nullptr;
  const uint64_t* off = nullptr;      // [N * D1 + 1] as for launch_bin_place
  const uint32_t* grp_ptr = nullptr;  // [N + 1]
  uint32_t D1 = 0, N = 0, longest = 0;
};
bool row_sort_fits(const BinBuild& bb, uint32_t D1, uint32_t longest, uint64_t mean);
hipError_t launch_bin_rows(const BinBuild& bb, uint32_t D1, const uint64_t* off, uint32_t* payload, uint8_t* del,
                           hipStream_t s);
size_t segsort_list(uint64_t n_syn, uint64_t n_groups);
hipError_t launch_segsort(const uint64_t* grp_off, uint64_t n_groups, uint32_t* payload, uint64_t* longer,
                          uint32_t* n_longer, uint64_t list_cap, uint64_t* big, uint32_t* nbig, uint32_t big_cap,
                          const RowSort& rows, hipStream_t s);
// Tile runs of every group (binned delivery with tile shift tsh): fill =
// false counts them into cnt[g] (and sets *too_long for a group of
// kRunMaxGroup synapses or more), fill = true writes them at run_desc[grp_run[g] ..].
hipError_t launch_runs(bool fill, const uint64_t* grp_off, uint64_t n_groups, const uint32_t* payload,
                       uint32_t cls_bits, uint32_t tsh, uint32_t* cnt, const uint64_t* grp_run, uint32_t* run_desc,
                       uint32_t* too_long, hipStream_t s);

// ---- per-step pipeline (step = ctrl->step_base + rel) ----
// One step: update, spike emission and delay-1/-2 delivery, and delivery of
// earlier steps' spikes.  With start/stop events the events are recorded on
// the kernel's own dispatch.
hipError_t launch_step(const NetDev& nd, uint32_t rel, hipStream_t s, hipEvent_t start = nullptr,
                       hipEvent_t stop = nullptr);
const char* step_kernel(const NetDev& nd);  // the one it launches (or "k_small")
// Pulled delivery (LIF networks with nd.n_pull): one step, the run index and the
// 16-bit synapses of one instance (sets *too_long for a group of kRunMaxGroup synapses or more),
// the waiting input into acc[buf], and what a restored snapshot needs: records by
// slice (clears what the counts hold).
void launch_pull_step(const NetDev& nd, uint32_t rel, hipStream_t s, hipEvent_t start, hipEvent_t stop);
hipError_t launch_pull_rows(const NetDev& nd, const PullInst& pi, uint64_t groups, uint32_t* row, uint32_t* too_long,
                            hipStream_t s);
hipError_t launch_pull_pay(const NetDev& nd, const PullInst& pi, uint64_t syn, uint16_t* pay, hipStream_t s);
hipError_t launch_pull_fold(const NetDev& nd, uint32_t buf, hipStream_t s);
hipError_t launch_pull_restore(const NetDev& nd, hipStream_t s);
// Small LIF networks (kernels_small.hip): steps in one launch (advances the
// step counter itself), what a readback needs, what a restored snapshot needs
// (ring cleared by the caller), the rows of the sources, the LDS of a block.
hipError_t launch_small_steps(const NetDev& nd, uint32_t steps, hipStream_t s, hipEvent_t start = nullptr,
                              hipEvent_t stop = nullptr);
hipError_t launch_small_fold(const NetDev& nd, hipStream_t s);
hipError_t launch_small_restore(const NetDev& nd, hipStream_t s);
hipError_t launch_small_rows(const NetDev& nd, uint32_t* row, uint32_t* pay, hipStream_t s);
size_t small_lds_bytes(const NetDev& nd);
// Strips (kernels_strip.hip): one step, what a readback needs, what a restored
// snapshot needs (spill cleared by the caller), the rows by (source, strip).
constexpr uint32_t kStripPops = 16, kStripPois = 8;  // populations and Poisson tables, at most
hipError_t launch_strip_step(const NetDev& nd, uint32_t rel, hipStream_t s, hipEvent_t start, hipEvent_t stop);
hipError_t launch_strip_fold(const NetDev& nd, hipStream_t s);
hipError_t launch_strip_restore(const NetDev& nd, hipStream_t s);
hipError_t launch_strip_rows(const NetDev& nd, uint32_t* row, uint32_t* pay, uint32_t* deg, hipStream_t s);
// The step kernels of networks with AdEx neurons: exponential ports only or
// with beta ports, without or with plastic synapses (launch_step picks one).
void launch_adex_exp(const NetDev& nd, dim3 grid, hipStream_t s, hipEvent_t start, hipEvent_t stop, uint32_t rel,
                     bool lif);
void launch_adex_beta(const NetDev& nd, dim3 grid, hipStream_t s, hipEvent_t start, hipEvent_t stop, uint32_t rel,
                      bool lif);
void launch_adex_exp_plastic(const NetDev& nd, dim3 grid, hipStream_t s, hipEvent_t start, hipEvent_t stop,
                             uint32_t rel, bool lif);
void launch_adex_beta_plastic(const NetDev& nd, dim3 grid, hipStream_t s, hipEvent_t start, hipEvent_t stop,
                              uint32_t rel, bool lif);
hipError_t launch_advance(Ctrl* ctrl, uint32_t steps, hipStream_t s);
// Binned delivery: add the pending bin entries of input buffer `buf` on `port`
// for gids [first, first+n) to out[0..n) (device int64).
hipError_t launch_pending_input(const NetDev& nd, uint32_t buf, uint32_t first, uint32_t n, uint32_t port,
                                int64_t* out, hipStream_t s);
// Multimeter: after the step ctrl->step_base + rel, copy *addr[c] for the nch
// channels into buf[(step % window) * nch + c].
hipError_t launch_sample(const float* const* addr, uint32_t nch, float* buf, uint32_t window, const Ctrl* ctrl,
                         uint32_t rel, hipStream_t s);
// Device address of this library's fixed readback workspace on `device`
// (kNoAllocInputMax int64 values, one copy per GPU, held until the process
// ends).  Resolved once per device; call with that device current first
// (resolve = true), later calls only look it up.  Null if never resolved.
hipError_t input_workspace(int device, bool resolve, int64_t** out);
// ---- nearest-neighbour STDP ----
// Plasticity of step ctrl->step_base + rel (after that step's kernel); no-op
// without plastic synapses.
hipError_t launch_stdp(const NetDev& nd, uint32_t rel, hipStream_t s);
// Set-up: pw[j] = the class weight and cleared arrivals for every synapse;
// cnt[t] += the plastic synapses onto t (cnt zeroed by the caller).
hipError_t launch_stdp_count(const NetDev& nd, uint32_t* cnt, hipStream_t s);
// tidx[cursor[t]++] = j for every plastic synapse j onto t (cursor = tptr copy).
hipError_t launch_stdp_scatter(const NetDev& nd, uint64_t* cursor, uint64_t* tidx, hipStream_t s);
hipError_t launch_poisson_counts(const NetDev& nd, uint64_t step, uint32_t first, uint32_t n, uint32_t* k,
                                 hipStream_t s);

}  // namespace snn
