// kernels_pull.hip -- steps of LIF networks whose delivery is pulled by the
// targets: large batches (and single networks) whose connection groups put
// many synapses on each target tile they reach.
//
// A tile is a range of up to 32,768 neurons of one instance.  The synapses of
// a connection group onto one tile are contiguous (groups are sorted by
// target), so with an index of where each (group, tile) run starts a block
// can take the tile's input from the runs alone: it goes over the in-flight
// spikes of the tile's instance, and for each whose delay expires now (Sec.
// 2.2, Fig. 1) counts the run's synapses per target in LDS.  No event is
// written to a bin and read back, none is counted first, none takes a device
// atomic.
//
// What is counted: a neuron receives at most four weight classes (host rule),
// so its input is sum over them of count x weight, and a step's count per
// (neuron, class) is below 2^16 (its in-degree times the largest
// multiplicity, host rule).  The sum is the same integer.  16-bit counts, two
// to a 32-bit word, let a tile be a whole instance of the sweep (int64 sums:
// an eighth of it): runs as long as the groups and few index reads.  A synapse
// is 16 bits here (target within the tile and which count), made from the
// 32-bit words at build.
//
// Step n is two kernels.  k_pull_update: block = slice of 512 to 4,096 neurons;
// input of step n from the counts, update, emission, the range of the slice's
// spikes in the step.  k_pull: every delay >= 1 into the counts of step n + 1
// (the records of step n are complete by then).  The work of k_pull follows
// the spikes, which differ by a factor of ten and more between the instances
// of a sweep and between a quiet step and a volley: a tile is split into parts by
// the step's events, about two parts to a block, which blocks take from a queue
// and whose counts the update adds up.  A part of fewer than 2,048 events costs
// more to clear, write and add up than it saves.
//
// Measured on 128 Brunel instances (3.0 10^6 neurons, 10^8 events a step):
// through bins 769 us a step; pulled with int64 sums of 4,096-neuron tiles
// 1,068 us; with 16-bit counts of 16,384-neuron tiles from the 32-bit words
// 350 us (245 in k_pull, 1.03 GB fetched at 4.2 TB/s, lines of 128 B of runs
// of ~54); with the 16-bit synapses and 32,768-neuron tiles 305 us (206 in
// k_pull, 0.57 GB fetched; bound by the latency of the runs, 16 waves a CU); with
// full batches of runs and parts by the step's events 257.
// With parts of 196,608 events and slices of 4,096 neurons whatever the network,
// few events left most CUs without any.  Us a step through bins, so, and now: 120,000
// neurons with 5,000 synapses and 240,000 events a step 52, 165, 29; ten networks of
// 25,000 and 2,500, 230,000 events 57, 99, 32; 60,000 and 10,000, 340,000 events 61,
// 152, 31; the 77,169-neuron microcircuit, 130,000 events 68, 129, 42.
#include "step_dev.h"

namespace snn {

namespace {

constexpr int kT = 1024;            // threads of a k_pull block
constexpr int kWaves = kT / 64;
constexpr int kUT = 512;            // threads of a k_pull_update block
constexpr int kUpdN = kPullSlice / kUT;
static_assert(kUT == kPullRow, "a row of a slice is a neuron a thread");
constexpr uint32_t kUnits = 2 * kPullGrid;  // parts of tiles, about, where there are many events
// ... of at least this many, in 1,024s: 2, 4 and 16 for the microcircuit 42, 41 and 48 us
// a step, at 0.37 of its size (5,700 events) 30, 32 and 36
constexpr uint32_t kUnitMin = 2;
constexpr int kBatch = 32;          // spikes of a wave's batch, at most: their runs are all in flight at once
constexpr int kRunLanes = 16;       // lanes that share a run
constexpr int kGroups = 64 / kRunLanes;
constexpr int kU = 8;
constexpr int kDelays = 16;         // spike counts of a tile's instance in flight at once

// Counts of neuron i (nw words) of its tile's parts, as the int64 input a[].
__device__ __forceinline__ void pull_input(const NetDev& nd, const PullPop& pw, uint32_t i, uint32_t parts, int64_t* a) {
  const uint32_t nw = nd.pull_words;
  const size_t stride = (size_t)nd.N * nw;
  uint32_t c0 = 0, c1 = 0;
  const uint32_t* c = nd.pull_cnt + (size_t)i * nw;
#pragma unroll 4
  for (uint32_t q = 0; q < parts; ++q) {
    c0 += c[q * stride];
    if (nw == 2) c1 += c[q * stride + 1];
  }
#pragma unroll
  for (int p = 0; p < kMaxPorts; ++p) a[p] = 0;
#pragma unroll
  for (int k = 0; k < kPullSlots; ++k) {
    const uint32_t v = ((k & 2) ? c1 : c0) >> ((k & 1) * 16) & 0xffffu;
#pragma unroll
    for (int p = 0; p < kMaxPorts; ++p)
      if ((int)pw.port[k] == p) a[p] += pw.wq[k] * (int64_t)v;
  }
}

struct PullUpdLds {
  PopDev spops[kTilePopLds];
  uint64_t sthr[kPoisLds * kPoisKmax];
  PullPop pw[kTilePopLds];
  uint32_t wcnt[kUpdN][kUT / 64];
  uint32_t emit;
};

// Step n of a slice.  Its spikes take consecutive positions in the step, in
// gid order, by one atomic; their range is left in slice_spk for k_pull.
__global__ void __launch_bounds__(kUT, 6) k_pull_update(NetDev nd, uint32_t rel) {
  __shared__ PullUpdLds sl;
  const uint64_t n = nd.ctrl->step_base + rel;
  const uint32_t slot = (uint32_t)(n % nd.R);
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) step_books(nd, n);
    const uint32_t next = (uint32_t)((n + 1) % nd.R);  // no block reads or adds to this slot during step n
    for (uint32_t i = threadIdx.x; i < nd.n_pull; i += kUT) nd.inst_spk[(size_t)next * nd.n_pull + i] = 0;
  }
  const PullSlice ps = nd.pull_slice[blockIdx.x];
  const uint32_t first = ps.first, nt = ps.n, PP = nd.P;
  const bool from_acc = *nd.pull_acc_step == n;  // after a restore
  const uint32_t parts = nd.pull_parts[ps.tile];
  const uint64_t pos_n = step_pos(nd, n);
  const uint32_t p0 = find_pop(nd.pops, nd.npop, first);
  const uint32_t npop = find_pop(nd.pops, nd.npop, first + nt - 1) - p0 + 1;
  load_tile_window<kUT>(nd, p0, npop, sl.spops, sl.sthr);
  if (threadIdx.x < npop) sl.pw[threadIdx.x] = nd.pull_pop[p0 + threadIdx.x];
  __syncthreads();
  const int64_t* acc = nd.acc + (size_t)inbuf(n) * nd.N * PP;
  uint64_t mq = 0;  // spikes of the thread's neurons, a byte each
  static_assert(kUpdN <= 8, "a byte of mq per neuron");
  bool mover = false;
#pragma unroll 1
  for (int q = 0; q * kUT < (int)nt; ++q) {
    const uint32_t loc = q * kUT + threadIdx.x;
    if (loc < nt) {
      const uint32_t i = first + loc;
      int64_t a[kMaxPorts];
      if (from_acc) {
#pragma unroll
        for (int p = 0; p < kMaxPorts; ++p) a[p] = (p < (int)PP) ? acc[(size_t)i * PP + p] : 0;
      } else {
        pull_input(nd, sl.pw[find_pop(sl.spops, npop, i)], i, parts, a);
      }
      uint32_t na = 0, nr = 0;
      bool capped = false;
      const uint32_t m = neuron_step<true, 0, 1>(nd, sl.spops, sl.sthr, n, i, a, na, nr, capped, mover, npop);
      mq |= (uint64_t)m << (8 * q);
    }
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint64_t bal[kUpdN];
#pragma unroll
  for (int q = 0; q < kUpdN; ++q) {
    bal[q] = __ballot((mq >> (8 * q)) & 0xff);
    if (lane == 0) sl.wcnt[q][wv] = __popcll(bal[q]);
  }
  __syncthreads();
  uint32_t before[kUpdN], spikes = 0;  // spikes of the (row, wave)s ahead of this wave's
#pragma unroll
  for (int q = 0; q < kUpdN; ++q)
    for (int w = 0; w < (kUT / 64) && q * kUT < (int)nt; ++w) {
      if (w == wv) before[q] = spikes;
      spikes += sl.wcnt[q][w];
    }
  if (threadIdx.x == 0) {
    uint32_t at = 0;
    if (spikes) {
      at = __hip_atomic_fetch_add(&nd.ring_cnt[slot], spikes, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_fetch_add(&nd.inst_spk[(size_t)slot * nd.n_pull + ps.inst], spikes, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_fetch_add(&nd.blk_stats[(size_t)kBlkStats * (first / kB) + 2], (uint64_t)spikes, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
    }
    nd.slice_spk[(size_t)slot * nd.n_slices + blockIdx.x] = SpkRange{at, at + spikes};
    sl.emit = at;
  }
  if (mover) atomicOr(&nd.ctrl->overflow, 1u);
  if (spikes == 0) return;  // block-uniform
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kUpdN; ++q) {
    const uint32_t m = (uint32_t)(mq >> (8 * q)) & 0xffu;
    if (!m) continue;
    const uint32_t i = first + q * kUT + threadIdx.x;
    emit_spike(nd, n, pos_n, sl.emit + before[q] + (uint32_t)__popcll(bal[q] & lanemask_lt()), i | (m << kMultShift),
               nd.grp_ptr[i], nd.src_mask[i]);
  }
}

// Block-wide exclusive scan of one value per thread (kT threads).
__device__ __forceinline__ uint32_t scan_excl(uint32_t v, uint32_t* lds, uint32_t* total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  __syncthreads();
  if (lane == 63) lds[wv] = x;
  __syncthreads();
  uint32_t before = 0, tot = 0;
  for (int w = 0; w < kWaves; ++w) {
    const uint32_t y = lds[w];
    if (w < wv) before += y;
    tot += y;
  }
  *total = tot;
  return before + x - v;
}

struct PullLds {
  uint32_t cnt[kPullWords];          // counts of the tile
  uint32_t unit0[kPullMaxTiles];     // first unit of each tile
  uint32_t item0[kT];                // first item of each segment of the unit
  uint32_t spk0[kT];                 // a segment's first spike
  uint32_t red[kWaves];
  uint32_t unit;                     // the block's unit, from the queue
};

// Input of step n + 1.  Units: part q of tile t, for the parts of each tile;
// blocks take them from the step's queue.  A unit's segments are the (delay, source
// slice) pairs whose number is q modulo the tile's parts; their spikes, segment
// after segment, are cut into batches of up to kBatch, one wave each: its lanes
// find the runs, then groups of kRunLanes lanes take them, kU runs in flight per
// group.
__global__ void __launch_bounds__(kT) k_pull(NetDev nd, uint32_t rel) {
  __shared__ PullLds sh;
  const uint64_t n = nd.ctrl->step_base + rel;
  const uint32_t ndel = (uint32_t)((n + 1 < nd.dmax) ? n + 1 : nd.dmax), slot0 = (uint32_t)((n + 1) % nd.R);
  const uint32_t nw = nd.pull_words, ntile = nd.n_ptiles;
  // parts of every tile, from the spikes in flight of its instance
  uint32_t units = 0, mine = 0;
  {
    uint32_t parts = 0, ev = 0, all, segs = 0;  // ev: the tile's events, in 1,024s
    if (threadIdx.x < ntile) {
      const PullTile tl = nd.pull_tile[threadIdx.x];
      uint64_t items = 0;
      for (uint32_t d0 = 1; d0 <= ndel; d0 += kDelays) {
        uint32_t c[kDelays];
#pragma unroll
        for (int q = 0; q < kDelays; ++q) {
          const uint32_t d = d0 + q, slot = slot0 >= d ? slot0 - d : slot0 + nd.R - d;
          c[q] = d <= ndel ? nd.inst_spk[(size_t)slot * nd.n_pull + tl.inst] : 0u;
        }
#pragma unroll
        for (int q = 0; q < kDelays; ++q) items += c[q];
      }
      ev = (uint32_t)fminf((float)items * tl.mean_run * (1.f / 1024.f), 4194304.f);
      segs = ndel * nd.pull_inst[tl.inst].ns;
    }
    (void)scan_excl(ev, sh.red, &all);
    if (threadIdx.x < ntile) {
      const uint32_t unit = max(all / kUnits, kUnitMin);
      parts = min(min((uint32_t)kPullParts, ev / unit + 1), segs);  // a segment a part at least
      if (blockIdx.x == 0) nd.pull_parts[threadIdx.x] = parts;
    }
    mine = scan_excl(parts, sh.red, &units);
    if (threadIdx.x < ntile) sh.unit0[threadIdx.x] = mine;
  }
  __syncthreads();
  const uint32_t lane = threadIdx.x & 63, sub = lane % kRunLanes, grp = lane / kRunLanes;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t lbits = 16 - nw, lmask = (1u << lbits) - 1u;
  uint64_t events = 0, pairs = 0;
  auto add = [&](uint32_t h, uint32_t mult) {  // one synapse: target within the tile, which count
    const uint32_t k = h >> lbits, loc = h & lmask;
    atomicAdd(&sh.cnt[nw == 1 ? loc : 2 * loc + (k >> 1)], mult << ((k & 1) * 16));
  };
  for (;;) {  // block-uniform
    if (threadIdx.x == 0)
      sh.unit = (uint32_t)__hip_atomic_fetch_add(&nd.ctrl->dlv_next[n & 3], (uint64_t)1, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const uint32_t u = sh.unit;
    if (u >= units) break;
    uint32_t lo = 0, hi = ntile;
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (sh.unit0[mid] <= u) lo = mid; else hi = mid;
    }
    const uint32_t t = __builtin_amdgcn_readfirstlane(lo);
    const uint32_t q = u - sh.unit0[t], parts = (t + 1 < ntile ? sh.unit0[t + 1] : units) - sh.unit0[t];
    const PullTile tl = nd.pull_tile[t];
    const PullInst pi = nd.pull_inst[tl.inst];
    for (uint32_t j = threadIdx.x; j < tl.n * nw; j += kT) sh.cnt[j] = 0;
    const uint32_t* pay = reinterpret_cast<const uint32_t*>(nd.pull_pay);  // two synapses to a word
    const uint32_t* row = nd.pull_row + pi.row0 + tl.k;
    const size_t w0 = pi.pay0 >> 1;
    const uint32_t nseg = ndel * pi.ns, first = tl.first;
    for (uint32_t s0 = q; s0 < nseg; s0 += parts * kT) {  // block-uniform: up to kT of the unit's segments
      const uint32_t s = s0 + threadIdx.x * parts;
      SpkRange r = {0u, 0u};
      if (s < nseg) {
        const uint32_t d = s / pi.ns + 1, slot = slot0 >= d ? slot0 - d : slot0 + nd.R - d;
        r = nd.slice_spk[(size_t)slot * nd.n_slices + pi.s0 + s % pi.ns];
      }
      uint32_t nitem;
      const uint32_t i0 = scan_excl(r.end - r.begin, sh.red, &nitem);
      sh.item0[threadIdx.x] = i0;
      sh.spk0[threadIdx.x] = r.begin;
      __syncthreads();
      // a wave's batch: few items go to all the waves
      const uint32_t bat = min((uint32_t)kBatch, max((uint32_t)kGroups, (nitem + kWaves - 1) / kWaves));
      for (uint32_t b = wv * bat; b < nitem; b += kWaves * bat) {  // wave-uniform
        const uint32_t x = b + lane;
        uint32_t off = 0, lm = 0;  // first synapse of the lane's run; length | multiplicity << kRunLenBits
        if (lane < bat && x < nitem) {
          uint32_t sl = 0, sr = kT;  // the last segment that starts at or before item x
          while (sr - sl > 1) {
            const uint32_t mid = (sl + sr) >> 1;
            if (sh.item0[mid] <= x) sl = mid; else sr = mid;
          }
          const uint32_t d = (s0 + sl * parts) / pi.ns + 1;
          const uint32_t slot = slot0 >= d ? slot0 - d : slot0 + nd.R - d;
          const SpikeRec rec = nd.recent[(size_t)slot * nd.N + sh.spk0[sl] + (x - sh.item0[sl])];
          if ((rec.mask >> d) & 1ull) {
            const uint32_t g = rec.grp_ptr + (uint32_t)__popcll(rec.mask & ((1ull << d) - 1ull)) - pi.g0;
            const uint32_t* e = row + (size_t)g * pi.nt;
            off = e[0];
            const uint32_t len = e[1] - off;
            lm = len | ((rec.entry >> kMultShift) << kRunLenBits);
            events += len;
            pairs += tl.k == 0 ? 1u : 0u;
          }
        }
        constexpr uint32_t kLen = (1u << kRunLenBits) - 1u;
#pragma unroll 1
        for (int r0 = 0; r0 < kBatch; r0 += kU * kGroups) {  // kU runs of a lane group in flight
          uint32_t at[kU], lmv[kU], longest = 0;
#pragma unroll
          for (int v = 0; v < kU; ++v) {
            at[v] = __shfl(off, r0 + v * kGroups + (int)grp, 64);
            lmv[v] = __shfl(lm, r0 + v * kGroups + (int)grp, 64);
            longest = max(longest, (lmv[v] & kLen) + (at[v] & 1u));
          }
          for (uint32_t z = 2 * sub; z - 2 * sub < longest; z += 2 * kRunLanes) {
            uint32_t w[kU];  // synapses z and z + 1 counted from the run's first whole word
#pragma unroll
            for (int v = 0; v < kU; ++v) {
              const uint32_t odd = at[v] & 1u;
              w[v] = z < (lmv[v] & kLen) + odd ? pay[w0 + ((at[v] + z) >> 1)] : 0u;
            }
#pragma unroll
            for (int v = 0; v < kU; ++v) {
              const uint32_t odd = at[v] & 1u, end = (lmv[v] & kLen) + odd, m = lmv[v] >> kRunLenBits;
              if (z >= odd && z < end) add(w[v] & 0xffffu, m);
              if (z + 1 < end) add(w[v] >> 16, m);
            }
          }
        }
      }
      __syncthreads();  // the segments are rewritten
    }
    __syncthreads();
    uint32_t* out = nd.pull_cnt + ((size_t)q * nd.N + first) * nw;
    for (uint32_t j = threadIdx.x; j < tl.n * nw; j += kT) out[j] = sh.cnt[j];
    __syncthreads();
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    events += __shfl_xor(events, o, 64);
    pairs += __shfl_xor(pairs, o, 64);
  }
  if (lane == 0 && (events || pairs)) {
    const size_t b = blockIdx.x % nd.sel_grid;
    if (pairs) __hip_atomic_fetch_add(&nd.sel_stats[2 * b], pairs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_add(&nd.sel_stats[2 * b + 1], events, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// The input waiting in the counts as int64 sums in acc[buf], for the readback.
__global__ void __launch_bounds__(kB) k_pull_fold(NetDev nd, uint32_t buf) {
  const PullSlice ps = nd.pull_slice[blockIdx.x];
  const uint32_t parts = nd.pull_parts[ps.tile];
  for (uint32_t j = threadIdx.x; j < ps.n; j += kB) {
    const uint32_t i = ps.first + j;
    int64_t a[kMaxPorts];
    pull_input(nd, nd.pull_pop[find_pop(nd.pops, nd.npop, i)], i, parts, a);
    for (uint32_t p = 0; p < nd.P; ++p) nd.acc[((size_t)buf * nd.N + i) * nd.P + p] = a[p];
  }
}

// ---- set-up ----
// Run index of one instance: row k of its group g = the first synapse of g at
// or beyond the instance's k-th tile, counted from the instance's first
// synapse; the entry after a group's last row is the next group's first, so a
// run ends where the following entry says.  One thread per entry (threads of
// one group search the same synapses).
__global__ void __launch_bounds__(kB) k_pull_rows(NetDev nd, PullInst pi, uint64_t groups, uint32_t* row,
                                                  uint32_t* too_long) {
  const uint64_t total = groups * pi.nt;
  for (uint64_t x = (uint64_t)blockIdx.x * kB + threadIdx.x; x <= total; x += (uint64_t)gridDim.x * kB) {
    uint64_t lo;
    if (x == total) {
      lo = nd.grp_off[pi.g0 + groups];
    } else {
      const uint64_t g = x / pi.nt;
      const uint32_t k = (uint32_t)(x - g * pi.nt);
      lo = nd.grp_off[pi.g0 + g];
      uint64_t hi = nd.grp_off[pi.g0 + g + 1];
      if (hi - lo >= kRunMaxGroup) atomicOr(too_long, 1u);
      if (k > 0) {  // first synapse whose target lies at or beyond the tile's first neuron
        const uint32_t bound = nd.pull_tile[pi.t0 + k].first;
        while (lo < hi) {
          const uint64_t mid = (lo + hi) >> 1;
          if ((nd.payload[mid] >> nd.cls_bits) < bound) lo = mid + 1; else hi = mid;
        }
      }
    }
    row[x] = (uint32_t)(lo - pi.syn0);
  }
}

// The 16-bit synapses of one instance: target within its tile | count << bits.
__global__ void __launch_bounds__(kB) k_pull_pay(NetDev nd, PullInst pi, uint64_t syn, uint16_t* pay) {
  const uint32_t lbits = 16 - nd.pull_words, cls_mask = (1u << nd.cls_bits) - 1u;
  for (uint64_t x = (uint64_t)blockIdx.x * kB + threadIdx.x; x < syn; x += (uint64_t)gridDim.x * kB) {
    const uint32_t w = nd.payload[pi.syn0 + x], tgt = w >> nd.cls_bits;
    uint32_t k = 0;
    while (k + 1 < pi.nt && nd.pull_tile[pi.t0 + k + 1].first <= tgt) ++k;
    pay[pi.pay0 + x] = (uint16_t)((tgt - nd.pull_tile[pi.t0 + k].first) | ((uint32_t)nd.pull_slot[w & cls_mask] << lbits));
  }
}

// After a restore: the records of one step slot put in the order of the
// slices (any order within a step delivers the same), with the slices' ranges
// and the instances' counts.  tmp: the slot's records as they were.
__global__ void __launch_bounds__(kT) k_pull_sort_slot(NetDev nd, uint32_t slot, const SpikeRec* tmp) {
  __shared__ uint32_t cur[kPullMaxSlices];
  const uint32_t cnt = min(nd.ring_cnt[slot], nd.N);
  for (uint32_t s = threadIdx.x; s < nd.n_slices; s += kT) cur[s] = 0;
  __syncthreads();
  auto slice_of = [&](const SpikeRec& r) {
    uint32_t lo = 0, hi = nd.n_slices;
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (nd.pull_slice[mid].first <= (r.entry & kGidMask)) lo = mid; else hi = mid;
    }
    return lo;
  };
  for (uint32_t j = threadIdx.x; j < cnt; j += kT) atomicAdd(&cur[slice_of(tmp[j])], 1u);
  __syncthreads();
  if (threadIdx.x == 0) {
    for (uint32_t i = 0; i < nd.n_pull; ++i) nd.inst_spk[(size_t)slot * nd.n_pull + i] = 0;
    uint32_t at = 0;
    for (uint32_t s = 0; s < nd.n_slices; ++s) {
      const uint32_t c = cur[s];
      nd.slice_spk[(size_t)slot * nd.n_slices + s] = SpkRange{at, at + c};
      nd.inst_spk[(size_t)slot * nd.n_pull + nd.pull_slice[s].inst] += c;
      cur[s] = at;
      at += c;
    }
  }
  __syncthreads();
  for (uint32_t j = threadIdx.x; j < cnt; j += kT) {
    const SpikeRec r = tmp[j];
    nd.recent[(size_t)slot * nd.N + atomicAdd(&cur[slice_of(r)], 1u)] = r;
  }
}

}  // namespace

void launch_pull_step(const NetDev& nd, uint32_t rel, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  const dim3 upd(nd.n_slices), pull(kPullGrid), ublk(kUT), blk(kT);
  if (start) {
    hipExtLaunchKernelGGL(k_pull_update, upd, ublk, 0, s, start, nullptr, 0, nd, rel);
    hipExtLaunchKernelGGL(k_pull, pull, blk, 0, s, nullptr, stop, 0, nd, rel);
  } else {
    hipLaunchKernelGGL(k_pull_update, upd, ublk, 0, s, nd, rel);
    hipLaunchKernelGGL(k_pull, pull, blk, 0, s, nd, rel);
  }
}

hipError_t launch_pull_fold(const NetDev& nd, uint32_t buf, hipStream_t s) {
  hipLaunchKernelGGL(k_pull_fold, dim3(nd.n_slices), dim3(kB), 0, s, nd, buf);
  return hipGetLastError();
}

hipError_t launch_pull_rows(const NetDev& nd, const PullInst& pi, uint64_t groups, uint32_t* row, uint32_t* too_long,
                            hipStream_t s) {
  const uint64_t blocks = (groups * pi.nt + kB) / kB;
  hipLaunchKernelGGL(k_pull_rows, dim3((uint32_t)(blocks < 65536 ? blocks : 65536)), dim3(kB), 0, s, nd, pi, groups,
                     row, too_long);
  return hipGetLastError();
}

hipError_t launch_pull_pay(const NetDev& nd, const PullInst& pi, uint64_t syn, uint16_t* pay, hipStream_t s) {
  if (!syn) return hipSuccess;
  const uint64_t blocks = (syn + kB - 1) / kB;
  hipLaunchKernelGGL(k_pull_pay, dim3((uint32_t)(blocks < 65536 ? blocks : 65536)), dim3(kB), 0, s, nd, pi, syn, pay);
  return hipGetLastError();
}

// The records of a slot are put by in the counts, which the next step does not
// read (its input lies in acc) and then writes.
static_assert(kPullParts * sizeof(uint32_t) >= sizeof(SpikeRec), "N records fit the counts");
hipError_t launch_pull_restore(const NetDev& nd, hipStream_t s) {
  SpikeRec* tmp = reinterpret_cast<SpikeRec*>(nd.pull_cnt);
  for (uint32_t slot = 0; slot < nd.R; ++slot) {
    const hipError_t e = hipMemcpyAsync(tmp, nd.recent + (size_t)slot * nd.N, (size_t)nd.N * sizeof(SpikeRec),
                                        hipMemcpyDeviceToDevice, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_pull_sort_slot, dim3(1), dim3(kT), 0, s, nd, slot, tmp);
  }
  return hipGetLastError();
}

}  // namespace snn
