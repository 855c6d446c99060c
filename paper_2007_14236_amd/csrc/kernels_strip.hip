// kernels_strip.hip -- LIF networks with direct delivery: every strip of
// neurons takes its own input.
//
// The network is cut into strips of 32 .. 1024 consecutive neurons, a block
// each.  In step n a block reads the spikes of step n - 1 and, from rows by
// (source, strip), their synapses onto its neurons: those of delay 1 go into the
// strip's input in LDS, the others into the strip's own lists of events by
// arrival step, through cursors in LDS and with plain stores; the list of step n
// is added to the input; then the neurons are advanced and their spikes
// emitted.  Each event is stored and read once, and no input crosses a block, so
// a step needs no device atomics but those of its spike counts.
//
// What bounds it: the chain of dependent reads of one step (step counter and
// spikes; row index; synapses; the emission's atomic) after the launch, 2 + 1 +
// 1.5 + 1.2 + 1.2 us.  With the events as device atomics on a target's input a
// step of 234,000 events (the 77,169-neuron microcircuit) is bound by them: 2.3
// 10^10 a second here, whatever their scope, width and footprint, against 1.2
// 10^11 scattered stores and 3 10^11 loads, and every other block's reads wait
// behind them.  Per step, with device atomics and so: that network at 126,000
// events 13.8 -> 9.3 us; LIF networks with delta PSCs of 2,100 neurons and 1,900
// events 7.9 -> 6.1 us, 10,000 and 45,000 10.0 -> 7.1, 150,000 and 680,000 46.9
// -> 24.7, 450,000 and 2.0 10^6 143 -> 54.
//
// The spike books and, once folded, input and counters are those of the other
// step kernels, so readback and snapshots are the same.
#include "step_dev.h"

namespace snn {

namespace {

constexpr int kT = 1024;
constexpr int kWaves = kT / 64;
constexpr int kRows = 4;  // rows in flight per lane

// LDS of a block: the head, then the strip's input [strip_n][P].
struct StripHead {
  PopDev spops[kPopLds];
  uint64_t sthr[kPoisLds * kPoisKmax];
  int64_t wq[kMaxClasses];
  uint64_t red[kWaves];
  uint64_t ovf;       // arrival slots whose list was full
  uint32_t cur[64];   // events in the list of each arrival slot
  uint8_t port[kMaxClasses];
};
static_assert(kStripPops <= kPopLds && kStripPois <= kPoisLds && kStripPois * kPoisKmax <= kT, "tables of the head");
static_assert(sizeof(StripHead) % 8 == 0 && kStripN <= kT && kStripN <= 1u << (32 - kStripLocalShift) &&
                  kStripN <= 1u << (32 - kBinLocalShift),
              "what follows is read in 64-bit words; a neuron a thread; bits of a synapse word and of an event");

// What the step kernel uses of a NetDev, in the order of use: the whole (twelve
// cache lines of it, read as they are needed) keeps a block waiting longer at its
// start.
struct StripNet {
  uint32_t N, P, R, n_strips, strip_n, strip_lanes, strip_cap, npop;
  uint32_t npois, pois_len, n_classes, nblk_upd;
  Ctrl* ctrl;
  uint32_t *strip_cnt, *strip_spk, *strip_cur;
  uint64_t* strip_ovf;
  const PopDev* pops;
  const uint64_t* pois_thr;
  const int64_t* cls_wq;
  const uint32_t* cls_port;
  float *V, *Ie, *Isyn;
  int32_t* refr;
  uint8_t* strip_pois;
  const uint64_t* src_mask;
  const uint32_t *grp_ptr, *strip_deg;
  const uint32_t* strip_row;
  uint32_t* strip_list;
  uint64_t* ring_base;
  uint32_t* ring_cnt;
  const uint32_t* strip_pay;
  int64_t* strip_spill;
  uint32_t* log;
  uint64_t log_mask;
  SpikeRec* recent;
  uint64_t* blk_stats;
  const NeuronLif* nlif;
  const uint32_t* gen_off;
  const uint64_t* gen_step;
  uint32_t* gen_next;
  uint64_t* chunk_base;
  uint64_t chunk_ring;
};

StripNet strip_net(const NetDev& nd) {
  return StripNet{nd.N, nd.P, nd.R, nd.n_strips, nd.strip_n, nd.strip_lanes, nd.strip_cap, nd.npop,
                  nd.npois, nd.pois_len, nd.n_classes, nd.nblk_upd,
                  nd.ctrl, nd.strip_cnt, nd.strip_spk, nd.strip_cur, nd.strip_ovf,
                  nd.pops, nd.pois_thr, nd.cls_wq, nd.cls_port, nd.V, nd.Ie, nd.Isyn, nd.refr,
                  nd.strip_pois, nd.src_mask, nd.grp_ptr, nd.strip_deg,
                  nd.strip_row, nd.strip_list, nd.ring_base, nd.ring_cnt, nd.strip_pay, nd.strip_spill,
                  nd.log, nd.log_mask, nd.recent, nd.blk_stats, nd.nlif, nd.gen_off, nd.gen_step, nd.gen_next,
                  nd.chunk_base, nd.chunk_ring};
}

__device__ __forceinline__ int64_t* strip_acc(char* lds) { return reinterpret_cast<int64_t*>(lds + sizeof(StripHead)); }

template <class ND>
__device__ __forceinline__ void strip_classes(const ND& nd, StripHead& h) {
  for (uint32_t k = threadIdx.x; k < nd.n_classes; k += kT) {
    h.wq[k] = nd.cls_wq[k];
    h.port[k] = (uint8_t)nd.cls_port[k];
  }
}

// mult events of class cls onto neuron `loc` of the strip, now
template <class ND>
__device__ __forceinline__ void strip_now(const ND& nd, const StripHead& h, int64_t* acc, uint32_t loc, uint32_t cls,
                                          uint32_t mult) {
  atomicAdd((unsigned long long*)&acc[loc * nd.P + h.port[cls]], (unsigned long long)(h.wq[cls] * (int64_t)mult));
}

// ... in step slot r: into the strip's list of that slot or, where it is full,
// as a sum into its neuron's spill of that slot.
template <class ND>
__device__ __forceinline__ void strip_later(const ND& nd, StripHead& h, uint32_t t, uint32_t loc, uint32_t cls,
                                            uint32_t mult, uint32_t r) {
  const uint32_t at = atomicAdd(&h.cur[r], 1u);
  if (at < nd.strip_cap) {
    nd.strip_list[((size_t)t * nd.R + r) * nd.strip_cap + at] = loc << kBinLocalShift | mult << kBinMultShift | cls;
  } else {
    __hip_atomic_fetch_add((unsigned long long*)&nd.strip_spill[((size_t)r * nd.N + t * nd.strip_n + loc) * nd.P + h.port[cls]],
                           (unsigned long long)(h.wq[cls] * (int64_t)mult), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    atomicOr((unsigned long long*)&h.ovf, 1ull << r);
  }
}

// Rows onto strip t of kRows spikes that a lane has in flight (none: b = e).
struct Rows {
  uint32_t b[kRows], e[kRows], m[kRows];
};
template <class ND>
__device__ __forceinline__ void row_open(const ND& nd, uint32_t t, uint32_t entry, bool any, Rows& x, int q) {
  x.b[q] = x.e[q] = x.m[q] = 0;
  if (any) {
    const uint32_t* row = nd.strip_row + (size_t)(entry & kGidMask) * (nd.n_strips + 1) + t;
    x.b[q] = row[0];
    x.e[q] = row[1];
    x.m[q] = entry >> kMultShift;
  }
}

// Their synapses, 2^strip_lanes lanes to a row; ev(word, mult) takes one.  Called
// by whole waves.
template <class ND, class Ev>
__device__ __forceinline__ void rows_run(const ND& nd, Rows& x, Ev ev) {
  const uint32_t g = 1u << nd.strip_lanes, l = threadIdx.x & (g - 1u);
#pragma unroll
  for (int q = 0; q < kRows; ++q) x.b[q] += l;
  for (;;) {
    uint32_t w[kRows];
    bool any = false;
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      w[q] = 0;
      if (x.b[q] < x.e[q]) {
        w[q] = nd.strip_pay[x.b[q]];
        any = true;
      }
    }
    if (!__any(any)) break;
    // all words are waited for here: a wait behind the first event's store waits
    // for that too
#pragma unroll
    for (int q = 0; q < kRows; ++q) asm volatile("" : "+v"(w[q]));
#pragma unroll
    for (int q = 0; q < kRows; ++q)
      if (x.b[q] < x.e[q]) {
        ev(w[q], x.m[q]);
        x.b[q] += g;
      }
  }
}

// The rows of spikes from .. cnt, dealt to nsub groups of 2^strip_lanes lanes,
// this lane's group being `sub`; get(j) gives spike j's entry.
template <class ND, class Get, class Ev>
__device__ __forceinline__ void strip_rows(const ND& nd, uint32_t t, uint32_t sub, uint32_t nsub, uint32_t from,
                                           uint32_t cnt, Get get, Ev ev) {
  for (uint32_t j0 = from; j0 < cnt; j0 += kRows * nsub) {  // wave-uniform
    Rows x;
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      const uint32_t j = j0 + q * nsub + sub;
      row_open(nd, t, j < cnt ? get(j) : 0u, j < cnt, x, q);
    }
    rows_run(nd, x, ev);
  }
}

__device__ __forceinline__ uint32_t word_class(uint32_t w) { return w & (uint32_t)(kMaxClasses - 1); }
__device__ __forceinline__ uint32_t word_delay(uint32_t w) { return w >> kStripDelayShift & 63u; }
__device__ __forceinline__ uint32_t word_local(uint32_t w) { return w >> kStripLocalShift; }

// Entries of the list of arrival slot r: `first` is this thread's first.
template <class ND>
__device__ __forceinline__ void strip_take(const ND& nd, const StripHead& h, int64_t* acc, uint32_t t, uint32_t r,
                                           uint32_t cnt, uint32_t first) {
  const uint32_t* list = nd.strip_list + ((size_t)t * nd.R + r) * nd.strip_cap;
  for (uint32_t k = threadIdx.x; k < cnt; k += kT) {
    const uint32_t x = k == threadIdx.x ? first : list[k];
    strip_now(nd, h, acc, x >> kBinLocalShift, x & (uint32_t)(kMaxClasses - 1), x >> kBinMultShift & kMaxMult);
  }
}

// A thread's words of the tables that the block keeps in LDS, read at once:
// loads that end in one LDS write each wait one after the other.
struct TableWords {
  uint32_t pop, port;
  uint64_t thr;
  int64_t wq;
};
constexpr uint32_t kPopWords = sizeof(PopDev) / 4;

// kWaves8: eight waves a SIMD, so that a CU holds two blocks.
template <int P, bool kWaves8>
__global__ void __launch_bounds__(kT, kWaves8 ? 8 : 4) k_step_strip(StripNet nd, uint32_t rel) {
  extern __shared__ __align__(16) char lds[];
  StripHead& h = *reinterpret_cast<StripHead*>(lds);
  int64_t* acc = strip_acc(lds);
  const uint32_t t = blockIdx.x, N = nd.N, R = nd.R, tid = threadIdx.x, lane = tid & 63;
  const uint32_t i = t * nd.strip_n + tid, nsub = kT >> nd.strip_lanes, sub = tid >> nd.strip_lanes;
  const bool in = tid < nd.strip_n && i < N;
  // first reads, all at once: the step, the spikes of the last step (those of an
  // even and of an odd one) and their count, the tables, the neuron, the cursors
  const uint64_t n = nd.ctrl->step_base + rel;
  const uint4 cnts = *reinterpret_cast<const uint4*>(nd.strip_cnt);
  uint32_t x0[kRows], x1[kRows];
#pragma unroll
  for (int q = 0; q < kRows; ++q) {
    const uint32_t j = q * nsub + sub;
    x0[q] = j < N ? nd.strip_spk[j] : 0u;
    x1[q] = j < N ? nd.strip_spk[(size_t)N + j] : 0u;
  }
  const uint64_t ovf = nd.strip_ovf[t];
  const uint32_t cur = tid < R ? nd.strip_cur[t * R + tid] : 0u;
  const uint32_t pw = nd.npop * kPopWords, tw = nd.npois * kPoisKmax;
  TableWords tb;
  tb.pop = tid < pw ? reinterpret_cast<const uint32_t*>(nd.pops)[tid] : 0u;
  tb.thr = tid < tw && (tid & (kPoisKmax - 1)) < nd.pois_len ? nd.pois_thr[tid] : 0u;
  tb.wq = tid < nd.n_classes ? nd.cls_wq[tid] : 0;
  tb.port = tid < nd.n_classes ? nd.cls_port[tid] : 0u;
  float y = 0.f, Ie = 0.f, I[kMaxPorts] = {0.f, 0.f, 0.f, 0.f};
  int32_t r = 0;
  uint32_t pois = 0, gp = 0, deg = 0;
  uint64_t mask = 0;
  if (in) {
    y = nd.V[i];
    Ie = nd.Ie[i];
    r = nd.refr[i];
#pragma unroll
    for (int p = 0; p < P; ++p)
      if (P < kMaxPorts || p < (int)nd.P) I[p] = nd.Isyn[(size_t)i * nd.P + p];
    pois = nd.strip_pois[i];
    mask = nd.src_mask[i];
    gp = nd.grp_ptr[i];
    deg = nd.strip_deg[i];
  }
  for (uint32_t w = tid; w < nd.strip_n * nd.P; w += kT) acc[w] = 0;
  if (tid == 0) h.ovf = 0;

  // second reads: the rows of the first spikes, the list of this step
  const uint32_t rs = (uint32_t)(n % R), before = (rs ? rs : R) - 1, after = rs + 1 == R ? 0u : rs + 1;
  const uint32_t ps = (uint32_t)(n + 3) & 3u, par = (uint32_t)(n + 1) & 1u;
  const uint32_t cnt = ps == 0 ? cnts.x : ps == 1 ? cnts.y : ps == 2 ? cnts.z : cnts.w;  // spikes of step n - 1
  Rows rows;
#pragma unroll
  for (int q = 0; q < kRows; ++q) row_open(nd, t, par ? x1[q] : x0[q], q * nsub + sub < cnt, rows, q);
  const uint32_t first = tid < nd.strip_cap ? nd.strip_list[((size_t)t * R + rs) * nd.strip_cap + tid] : 0u;
  const uint64_t pos_n = n ? nd.ring_base[before] + nd.ring_cnt[before] : 0;  // raster position of the step's spikes
  if (tid < R) h.cur[tid] = cur;
  if (tid < pw) reinterpret_cast<uint32_t*>(h.spops)[tid] = tb.pop;
  for (uint32_t w = tid + kT; w < pw; w += kT)
    reinterpret_cast<uint32_t*>(h.spops)[w] = reinterpret_cast<const uint32_t*>(nd.pops)[w];
  if (tid < tw) h.sthr[tid] = tb.thr;
  if (tid < nd.n_classes) {
    h.wq[tid] = tb.wq;
    h.port[tid] = (uint8_t)tb.port;
  }
  if (t == 0 && tid == 0) {
    nd.ring_base[rs] = pos_n;
    nd.chunk_base[n & (nd.chunk_ring - 1)] = pos_n;
    nd.ring_cnt[after] = 0;
    nd.strip_cnt[(n + 1) & 3] = 0;
  }
  __syncthreads();
  auto ev = [&](uint32_t w, uint32_t m) {
    const uint32_t d = word_delay(w);
    uint32_t a = rs + d - 1;
    if (a >= R) a -= R;
    if (d == 1) strip_now(nd, h, acc, word_local(w), word_class(w), m);
    else strip_later(nd, h, t, word_local(w), word_class(w), m, a);
  };
  rows_run(nd, rows, ev);
  strip_take(nd, h, acc, t, rs, h.cur[rs], first);
  const uint32_t* spk = nd.strip_spk + (size_t)par * N;
  strip_rows(nd, t, sub, nsub, kRows * nsub, cnt, [&](uint32_t j) { return spk[j]; }, ev);
  asm volatile("" : "+v"(pois));  // read before another wave writes the next step's
  __syncthreads();
  if (tid < R) nd.strip_cur[t * R + tid] = tid == rs ? 0u : min(h.cur[tid], nd.strip_cap);
  const bool spilt = ovf >> rs & 1ull;  // block-uniform
  if (tid == 0 && (ovf | h.ovf)) nd.strip_ovf[t] = (ovf & ~(1ull << rs)) | h.ovf;

  // The Poisson counts do not depend on the dynamics: those of the next step are
  // drawn by threads from the block's end, most of which have nothing else to do
  // now (drawn for this step before the barrier they took 1.1 us of it).
  const uint32_t v = kT - 1 - tid, vi = t * nd.strip_n + v;
  const bool draws = nd.npois && v < nd.strip_n && vi < N;
  auto draw = [&] {
    const PopDev& pv = h.spops[find_pop(h.spops, nd.npop, vi)];
    if (pv.pois >= 0)
      nd.strip_pois[vi] = (uint8_t)poisson_draw(h.sthr + pv.pois * kPoisKmax, pv.seed, vi - pv.gid_base, n + 1);
  };
  if (draws && tid >= nd.strip_n) draw();

  uint32_t m = 0;
  bool mover = false;
  if (in) {
    const PopDev& pp = h.spops[find_pop(h.spops, nd.npop, i)];
    int64_t a[P];
#pragma unroll
    for (int p = 0; p < P; ++p) a[p] = P < kMaxPorts || p < (int)nd.P ? acc[tid * nd.P + p] : 0;
    if (spilt) {
      int64_t* sp = nd.strip_spill + ((size_t)rs * N + i) * nd.P;
#pragma unroll
      for (int p = 0; p < P; ++p)
        if (P < kMaxPorts || p < (int)nd.P) {
          a[p] += sp[p];
          sp[p] = 0;
        }
    }
    float x[kMaxPorts] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = 0; p < P; ++p) x[p] = __fmul_rn((float)(a[p] + (pp.pois >= 0 && p == pp.pois_port ? (int64_t)pois * pp.pois_wq : 0)), pp.scale[p]);
    if (pp.model >= kSpikeGen) {
      if (pp.model == kSpikeGen) {  // one spike per listed step n
        uint32_t c = nd.gen_next[i];
        const uint32_t e = nd.gen_off[i + 1];
        while (c < e && nd.gen_step[c] < n) ++c;
        while (c < e && nd.gen_step[c] == n) { ++m; ++c; }
        nd.gen_next[i] = c;
      } else {  // a parrot repeats the spikes arriving now
        m = x[0] > 0.f ? (uint32_t)x[0] : 0u;
      }
      if (m > kMaxMult) { mover = true; m = kMaxMult; }
    } else {
      const LifK k = lif_consts(nd, pp, i);
      bool s;
      if (pp.model == kLifDelta) {
        s = lif_delta_step(k, y, r, Ie, x[0]);
      } else {
        s = lif_exp_step(pp, k, y, I, r, Ie, x);
#pragma unroll
        for (int p = 0; p < P; ++p)
          if (p < pp.n_ports) nd.Isyn[(size_t)i * nd.P + p] = I[p];
      }
      nd.V[i] = y;
      nd.refr[i] = r;
      m = s ? 1u : 0u;
    }
  }
  if (mover) atomicOr(&nd.ctrl->overflow, 1u);
  const uint64_t bal = __ballot(m != 0);
  if (bal) {  // wave-uniform
    uint32_t wpos = 0;
    if (lane == 0) {
      wpos = __hip_atomic_fetch_add(&nd.ring_cnt[rs], (uint32_t)__popcll(bal), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_fetch_add(&nd.strip_cnt[n & 3], (uint32_t)__popcll(bal), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // spikes, pairs and events sent (those still to arrive are taken off when
    // the counters are read)
    uint64_t pairs = m ? __popcll(mask) : 0, events = m ? deg : 0;
#pragma unroll
    for (int k = 32; k > 0; k >>= 1) {
      pairs += __shfl_xor(pairs, k, 64);
      events += __shfl_xor(events, k, 64);
    }
    wpos = __shfl(wpos, 0, 64) + (uint32_t)__popcll(bal & lanemask_lt());
    if (m) {
      const uint32_t entry = i | (m << kMultShift);
      nd.strip_spk[(size_t)(n & 1) * N + wpos] = entry;
      nd.log[(pos_n + wpos) & nd.log_mask] = entry;
      nd.recent[(size_t)rs * N + wpos] = SpikeRec{entry, gp, mask};
    }
    if (lane == 0) {
      uint64_t* st = nd.blk_stats + (size_t)kBlkStats * (t % nd.nblk_upd);
      __hip_atomic_fetch_add(&st[2], (uint64_t)__popcll(bal), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_fetch_add(&st[3], pairs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_fetch_add(&st[4], events, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  if (draws && tid < nd.strip_n) draw();
}

// Before a readback at step n = step_base: the input of step n into acc[n & 1]
// (the other buffer cleared); the last block: the pairs and events still to
// arrive off those sent.
__global__ void __launch_bounds__(kT) k_strip_fold(NetDev nd) {
  extern __shared__ __align__(16) char lds[];
  StripHead& h = *reinterpret_cast<StripHead*>(lds);
  int64_t* acc = strip_acc(lds);
  const uint64_t n = nd.ctrl->step_base;
  const uint32_t t = blockIdx.x, N = nd.N, R = nd.R, rs = (uint32_t)(n % R);
  if (t == nd.n_strips) {
    uint64_t ev, pr;
    sent_pending<kT>(nd, n, ev, pr);
    ev = block_sum(ev, h.red);
    pr = block_sum(pr, h.red);
    if (threadIdx.x == 0) {
      nd.sel_stats[0] = nd.strip_sent[0] - pr;
      nd.sel_stats[1] = nd.strip_sent[1] - ev;
    }
    return;
  }
  strip_classes(nd, h);
  for (uint32_t w = threadIdx.x; w < nd.strip_n * nd.P; w += kT) acc[w] = 0;
  __syncthreads();
  const uint32_t have = nd.strip_cur[t * R + rs];
  strip_take(nd, h, acc, t, rs, have, threadIdx.x < have ? nd.strip_list[((size_t)t * R + rs) * nd.strip_cap + threadIdx.x] : 0u);
  const uint32_t* spk = nd.strip_spk + (size_t)((n + 1) & 1) * N;
  strip_rows(
      nd, t, threadIdx.x >> nd.strip_lanes, kT >> nd.strip_lanes, 0u, n ? nd.strip_cnt[(n + 3) & 3] : 0u,
      [&](uint32_t j) { return spk[j]; },
      [&](uint32_t w, uint32_t m) {
        if (word_delay(w) == 1) strip_now(nd, h, acc, word_local(w), word_class(w), m);
      });
  __syncthreads();
  const bool spilt = nd.strip_ovf[t] >> rs & 1ull;
  const uint32_t first = t * nd.strip_n * nd.P, end = min(nd.strip_n * nd.P, N * nd.P - first);
  const size_t stride = (size_t)N * nd.P;
  for (uint32_t w = threadIdx.x; w < end; w += kT) {
    nd.acc[inbuf(n) * stride + first + w] = acc[w] + (spilt ? nd.strip_spill[rs * stride + first + w] : 0);
    nd.acc[inbuf(n + 1) * stride + first + w] = 0;
  }
}

// At the start and after a restore, at step n = step_base (the spill cleared): the
// lists from the spikes in flight, the Poisson counts of step n; the last block:
// the spikes of step n - 1, the pairs and events.
__global__ void __launch_bounds__(kT) k_strip_restore(NetDev nd) {
  extern __shared__ __align__(16) char lds[];
  StripHead& h = *reinterpret_cast<StripHead*>(lds);
  const uint64_t n = nd.ctrl->step_base;
  const uint32_t t = blockIdx.x, N = nd.N, R = nd.R, lane = threadIdx.x & 63;
  if (t == nd.n_strips) {
    const uint32_t slot = (uint32_t)((n + R - 1) % R), cnt = n ? min(nd.ring_cnt[slot], N) : 0u;
    for (uint32_t j = threadIdx.x; j < cnt; j += kT)
      nd.strip_spk[(size_t)((n + 1) & 1) * N + j] = nd.recent[(size_t)slot * N + j].entry;
    if (threadIdx.x < 4) nd.strip_cnt[threadIdx.x] = threadIdx.x == ((n + 3) & 3) ? cnt : 0u;
    uint64_t ev, pr;
    sent_pending<kT>(nd, n, ev, pr);
    for (uint32_t b = threadIdx.x; b < nd.sel_grid; b += kT) { pr += nd.sel_stats[2 * b]; ev += nd.sel_stats[2 * b + 1]; }
    ev = block_sum(ev, h.red);
    pr = block_sum(pr, h.red);
    if (threadIdx.x == 0) { nd.strip_sent[0] = pr; nd.strip_sent[1] = ev; }
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < 2 * nd.sel_grid; b += kT) nd.sel_stats[b] = 0;  // set when read
    return;
  }
  strip_classes(nd, h);
  if (threadIdx.x < 64) h.cur[threadIdx.x] = 0;
  if (threadIdx.x == 0) h.ovf = 0;
  __syncthreads();
  for (uint32_t d = 2 + (threadIdx.x >> 6); d <= nd.dmax && d <= n; d += kWaves) {  // wave-uniform
    const uint32_t slot = (uint32_t)((n - d) % R);
    const SpikeRec* recs = nd.recent + (size_t)slot * N;
    strip_rows(
        nd, t, lane >> nd.strip_lanes, 64u >> nd.strip_lanes, 0u, min(nd.ring_cnt[slot], N),
        [&](uint32_t j) { return recs[j].entry; },
        [&](uint32_t w, uint32_t m) {
          uint32_t a = slot + word_delay(w);
          if (a >= R) a -= R;
          if (word_delay(w) >= d) strip_later(nd, h, t, word_local(w), word_class(w), m, a);
        });
  }
  __syncthreads();
  if (threadIdx.x < R) nd.strip_cur[t * R + threadIdx.x] = min(h.cur[threadIdx.x], nd.strip_cap);
  if (threadIdx.x == 0) nd.strip_ovf[t] = h.ovf;
  const uint32_t i = t * nd.strip_n + threadIdx.x;
  if (threadIdx.x < nd.strip_n && i < N) {
    const PopDev& pp = nd.pops[find_pop(nd.pops, nd.npop, i)];
    nd.strip_pois[i] = pp.pois < 0 ? 0
                                   : (uint8_t)poisson_draw(nd.pois_thr + (size_t)pp.pois * kPoisKmax, pp.seed,
                                                           i - pp.gid_base, n);
  }
}

// ---- set-up: each source's synapses by strip, a block per source ----
// Bound by the latency of its reads (source, offsets, row): a row is read once,
// kept in registers while its words are counted by strip (the count's return is
// a word's rank in it), put in order in LDS and written in order; rows beyond
// kRowWords are read twice and written where they belong.  3 10^8 synapses in
// rows of 2,100 .. 7,900: 0.65 ms; 1.25 with half of them beyond (256 threads,
// 4,096 words), 1.64 with all.
constexpr int kRowRegs = 16;
constexpr int kRT = 512;
constexpr uint32_t kRowWords = kRowRegs * kRT;

__global__ void __launch_bounds__(kRT) k_strip_rows(NetDev nd, uint32_t shift, uint32_t magic, uint32_t* row, uint32_t* pay, uint32_t* deg) {
  __shared__ uint64_t red[kRT / 64];
  __shared__ uint32_t cnt[kStripMax], stage[kRowWords];
  const uint32_t s = blockIdx.x, S = nd.n_strips, g0 = nd.grp_ptr[s], cls_mask = (1u << nd.cls_bits) - 1u;
  const uint64_t mask = nd.src_mask[s], o = nd.grp_off[g0];
  const uint32_t len = (uint32_t)(nd.grp_off[g0 + (uint32_t)__popcll(mask)] - o);
  const uint32_t* in = nd.payload + o;
  const bool fits = len <= kRowWords;
  uint32_t w[kRowRegs], rank[kRowRegs];
  if (fits) {
#pragma unroll
    for (int q = 0; q < kRowRegs; ++q) {
      const uint32_t j = q * kRT + threadIdx.x;
      w[q] = j < len ? in[j] : 0u;
    }
  }
  // lane d: where the groups of delays from d on begin; a synapse's delay is the
  // last that is not behind it
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t begin = (uint32_t)(nd.grp_off[g0 + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull))] - o);
  for (uint32_t k = threadIdx.x; k < S; k += kRT) cnt[k] = 0;
  __syncthreads();
  // strip of a target: a quotient of 64s (or, alone, 32s) by multiplication, 24 bits
  // wide; exact while (N / 64) (strip_n / 64) < 2^20
  auto strip = [&](uint32_t x) { return (uint32_t)__umul24(x >> (nd.cls_bits + shift), magic) >> 20; };
  // delay of word j, consecutive words j - lane on in a wave (all its lanes)
  auto delay = [&](uint32_t j) {
    const uint32_t j0 = __builtin_amdgcn_readfirstlane(j);
    uint32_t d = (uint32_t)__popcll(__ballot(begin <= j0)) - 1;
    const uint32_t last = (uint32_t)__popcll(__ballot(begin <= j0 + 63)) - 1;
    for (uint32_t k = d + 1; k <= last; ++k)  // wave-uniform
      if (__builtin_amdgcn_readlane(begin, k) <= j) d = k;
    return d;
  };
  auto word = [&](uint32_t x, uint32_t k, uint32_t d) {
    return ((x >> nd.cls_bits) - (uint32_t)__umul24(k, nd.strip_n)) << kStripLocalShift | d << kStripDelayShift | (x & cls_mask);
  };
  if (fits) {
#pragma unroll
    for (int q = 0; q < kRowRegs; ++q)
      if (q * kRT + threadIdx.x < len) {
        const uint32_t k = strip(w[q]);
        rank[q] = k << 16 | atomicAdd(&cnt[k], 1u);
      }
  } else {
    for (uint32_t j = threadIdx.x; j < len; j += kRT) atomicAdd(&cnt[strip(in[j])], 1u);
  }
  __syncthreads();
  constexpr int kPer = kStripMax / kRT;
  uint32_t c[kPer];
  uint64_t sum = 0, total;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const uint32_t k = threadIdx.x * kPer + q;
    c[q] = k < S ? cnt[k] : 0u;
    sum += c[q];
  }
  uint32_t at = (uint32_t)block_excl_scan(sum, red, &total);
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const uint32_t k = threadIdx.x * kPer + q;
    if (k < S) cnt[k] = at;
    at += c[q];
  }
  if (threadIdx.x == 0) deg[s] = len;
  __syncthreads();
  for (uint32_t k = threadIdx.x; k <= S; k += kRT) row[(size_t)s * (S + 1) + k] = (uint32_t)o + (k < S ? cnt[k] : len);
  if (fits) {
#pragma unroll
    for (int q = 0; q < kRowRegs; ++q) {
      const uint32_t j = q * kRT + threadIdx.x;
      if (j - lane >= len) break;  // wave-uniform
      const uint32_t d = delay(j);
      if (j < len) {
        const uint32_t k = rank[q] >> 16;
        stage[cnt[k] + (rank[q] & 0xffffu)] = word(w[q], k, d);
      }
    }
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < len; j += kRT) pay[o + j] = stage[j];
  } else {
    __syncthreads();
    for (uint32_t j = threadIdx.x; j - lane < len; j += kRT) {  // wave-uniform
      const uint32_t d = delay(j);
      if (j >= len) continue;
      const uint32_t x = in[j], k = strip(x);
      pay[o + atomicAdd(&cnt[k], 1u)] = word(x, k, d);
    }
  }
}

size_t strip_lds(const NetDev& nd) { return sizeof(StripHead) + (size_t)nd.strip_n * nd.P * 8; }

}  // namespace

hipError_t launch_strip_step(const NetDev& nd, uint32_t rel, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  // with fewer scalar registers (they hold the network's pointers) a block takes
  // 0.8 us longer, which pays where there are more blocks than CUs: 5,000 neurons
  // in 79 strips 6.7 and 7.7 us a step, 300,000 in 293 48.6 and 43.0, 450,000 in
  // 440 64.1 and 54.5
  auto k = nd.n_strips <= 256
               ? (nd.P == 1 ? k_step_strip<1, false> : nd.P == 2 ? k_step_strip<2, false> : k_step_strip<kMaxPorts, false>)
               : (nd.P == 1 ? k_step_strip<1, true> : nd.P == 2 ? k_step_strip<2, true> : k_step_strip<kMaxPorts, true>);
  if (start) hipExtLaunchKernelGGL(k, dim3(nd.n_strips), dim3(kT), strip_lds(nd), s, start, stop, 0, strip_net(nd), rel);
  else hipLaunchKernelGGL(k, dim3(nd.n_strips), dim3(kT), strip_lds(nd), s, strip_net(nd), rel);
  return hipGetLastError();
}

hipError_t launch_strip_fold(const NetDev& nd, hipStream_t s) {
  hipLaunchKernelGGL(k_strip_fold, dim3(nd.n_strips + 1), dim3(kT), strip_lds(nd), s, nd);
  return hipGetLastError();
}

hipError_t launch_strip_restore(const NetDev& nd, hipStream_t s) {
  hipLaunchKernelGGL(k_strip_restore, dim3(nd.n_strips + 1), dim3(kT), strip_lds(nd), s, nd);
  return hipGetLastError();
}

hipError_t launch_strip_rows(const NetDev& nd, uint32_t* row, uint32_t* pay, uint32_t* deg, hipStream_t s) {
  const uint32_t shift = nd.strip_n < 64 ? 5 : 6;
  const uint32_t u = nd.strip_n >> shift, magic = ((1u << 20) + u - 1) / u;
  hipLaunchKernelGGL(k_strip_rows, dim3(nd.N), dim3(kRT), 0, s, nd, shift, magic, row, pay, deg);
  return hipGetLastError();
}

}  // namespace snn
