// kernels_small.hip -- many steps of a small LIF network in one block.
//
// A step of a small network is bound by latency: as a launch of its own it
// is 1.6 us of launch and a chain of dependent device reads and atomics (8.1
// us in all for 1,000 neurons with 870 events a step).  Here one 1,024-thread
// block runs all the steps of a launch: the neurons' state stays in
// registers, the steps are separated by block barriers, and a spike is
// delivered at once to all its synapses, into a ring of inputs by arrival step
// (delays 1 .. Dmax), so that no step looks again at the spikes in flight.
// The ring lies in LDS as 16-bit counts of at most four weight classes onto a
// neuron (as in kernels_pull.hip); networks whose ring does not fit a CU's LDS
// are not small (with the ring in global memory a step of 2,000 neurons with
// 5,800 events took 11.8 us, against 8.1 by a launch per step).
// The synapses of a source are one row of 32-bit words (target, delay, class).
// The Poisson counts of a launch's steps do not depend on its dynamics: they
// are drawn by the whole chip beforehand, a byte each (in the block the
// generator alone would take 3.9 us a step).
//
// The spike books (raster ring, records, counts by step) are those of the
// other step kernels, so readback, snapshots and STDP-free restarts are the
// same; the input of the next step is put into acc when it is read.
#include "step_dev.h"

namespace snn {

namespace {

constexpr int kT = 1024;
constexpr int kWaves = kT / 64;
constexpr int kInFlight = 4;  // words of a row in flight per lane

struct SmallHead {
  PopDev spops[kPopLds];
  PullPop pw[kPopLds];
  uint64_t red[2][kWaves];
  uint32_t n_spk[2];  // spikes of this step, of the next
};
// LDS of the block: the head, the rows' ends, the step's spikes (gid |
// multiplicity << kMultShift), then the ring.
struct SmallLds {
  SmallHead& h;
  uint32_t* row;   // [N + 1]
  uint32_t* spk;   // [N]
  uint32_t* ring;  // [R][N][pull_words]
};
__host__ __device__ __forceinline__ size_t small_tail(uint32_t N) {
  return (sizeof(SmallHead) + ((size_t)2 * N + 1) * 4 + 15) & ~(size_t)15;
}
__device__ __forceinline__ SmallLds small_lds(char* p, uint32_t N) {
  uint32_t* row = reinterpret_cast<uint32_t*>(p + sizeof(SmallHead));
  return SmallLds{*reinterpret_cast<SmallHead*>(p), row, row + N + 1, reinterpret_cast<uint32_t*>(p + small_tail(N))};
}
static_assert(sizeof(SmallHead) % 8 == 0, "what follows is read in 32-bit words");

// One word of a row: target | delay << 13 | count << 19.
constexpr uint32_t kDelShift = 13, kClsShift = 19, kTgtMask = (1u << kDelShift) - 1;
static_assert(kSmallN <= 1u << kDelShift && kSmallN <= 2 * kT, "target bits of a row word; neurons of the threads");

// A spike of multiplicity mult in step slot r0 (step mod R) to the synapse
// `w` of one of its rows.
__device__ __forceinline__ void small_add(const NetDev& nd, const SmallLds& sh, uint32_t w, uint32_t mult, uint32_t r0) {
  const uint32_t tgt = w & kTgtMask, c = w >> kClsShift;
  uint32_t r = r0 + ((w >> kDelShift) & 63u);
  if (r >= nd.R) r -= nd.R;
  const uint32_t nw = nd.pull_words;
  atomicAdd(&sh.ring[r * nd.N * nw + (nw == 1 ? tgt : 2 * tgt + (c >> 1))], mult << ((c & 1) * 16));
}

// Input a[] of neuron i (population record pw) from ring slot r, cleared.
template <int P>
__device__ __forceinline__ void small_input(const NetDev& nd, const SmallLds& sh, const PullPop& pw, uint32_t r, uint32_t i,
                                            int64_t* a) {
  const uint32_t nw = nd.pull_words;
  uint32_t* c = &sh.ring[(r * nd.N + i) * nw];
  const uint32_t c0 = c[0], c1 = nw == 2 ? c[1] : 0u;
  c[0] = 0;
  if (nw == 2) c[1] = 0;
#pragma unroll
  for (int p = 0; p < P; ++p) a[p] = 0;
#pragma unroll
  for (int k = 0; k < kPullSlots; ++k) {
    const uint32_t v = ((k & 2) ? c1 : c0) >> ((k & 1) * 16) & 0xffffu;
#pragma unroll
    for (int p = 0; p < P; ++p)
      if (P == 1 || (int)pw.port[k] == p) a[p] += pw.wq[k] * (int64_t)v;
  }
}

// The rows of spikes 0 .. ns in step slot r0; get(j, row, end, mult) gives a
// spike's.  Units of 64 words of a row are dealt to the waves; a wave finds
// its units by a scan of the rows' units over its lanes.
template <class Get>
__device__ __forceinline__ void small_deliver(const NetDev& nd, const SmallLds& sh, uint32_t ns, uint32_t r0, Get get) {
  const uint32_t lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t first = wv;  // the wave's next unit, counted from the present 64 rows' first
  for (uint32_t s0 = 0; s0 < ns; s0 += 64) {  // wave-uniform
    uint32_t row = 0, end = 0, mult = 0;
    if (s0 + lane < ns) get(s0 + lane, row, end, mult);
    const uint32_t nu = (end - row + 63) >> 6;
    uint32_t incl = nu;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(incl, o, 64);
      if (lane >= (uint32_t)o) incl += y;
    }
    const uint32_t total = __builtin_amdgcn_readlane(incl, 63);
    uint32_t u = first;
    for (; u < total; u += kInFlight * kWaves) {  // wave-uniform
      uint32_t w[kInFlight], m[kInFlight];
#pragma unroll
      for (int q = 0; q < kInFlight; ++q) {
        const uint32_t v = u + q * kWaves;
        w[q] = 0xffffffffu;
        m[q] = 0;
        if (v < total) {  // wave-uniform
          const int k = __popcll(__ballot(incl <= v));  // the row that holds unit v
          const uint32_t b = __builtin_amdgcn_readlane(row, k), e = __builtin_amdgcn_readlane(end, k);
          const uint32_t j = b + ((v - (__builtin_amdgcn_readlane(incl, k) - __builtin_amdgcn_readlane(nu, k))) << 6) + lane;
          if (j < e) {
            w[q] = nd.small_pay[j];
            m[q] = __builtin_amdgcn_readlane(mult, k);
          }
        }
      }
#pragma unroll
      for (int q = 0; q < kInFlight; ++q)
        if (m[q]) small_add(nd, sh, w[q], m[q], r0);
    }
    first = (first + kWaves - total % kWaves) % kWaves;  // the next rows' units go on in turn
  }
}

__device__ __forceinline__ uint64_t wave_sum(uint64_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ void small_begin(const NetDev& nd, const SmallLds& sh) {
  for (uint32_t w = threadIdx.x; w < nd.npop * (uint32_t)(sizeof(PopDev) / 4); w += kT)
    reinterpret_cast<uint32_t*>(sh.h.spops)[w] = reinterpret_cast<const uint32_t*>(nd.pops)[w];
  for (uint32_t i = threadIdx.x; i <= nd.N; i += kT) sh.row[i] = nd.small_row[i];
  if (threadIdx.x < nd.npop) sh.h.pw[threadIdx.x] = nd.pull_pop[threadIdx.x];
  for (uint32_t w = threadIdx.x; w < nd.R * nd.N * nd.pull_words; w += kT) sh.ring[w] = nd.small_ring[w];
  if (threadIdx.x < 2) sh.h.n_spk[threadIdx.x] = 0;
  __syncthreads();
}

// Steps from base to a generator's emission c (of e): never for none, or too far.
__device__ __forceinline__ uint32_t gen_wait(const NetDev& nd, uint32_t c, uint32_t e, uint64_t base) {
  return c < e ? (uint32_t)min(nd.gen_step[c] - base, (uint64_t)0xffffffffull) : 0xffffffffu;
}

__device__ __forceinline__ SpikeRec spike_rec(const NetDev& nd, uint32_t entry) {
  return SpikeRec{entry, nd.grp_ptr[entry & kGidMask], nd.src_mask[entry & kGidMask]};
}

// Steps ctrl->step_base .. + steps of the network; a thread keeps neurons
// threadIdx.x + 1024 q.
template <int NPT, int P>
__global__ void __launch_bounds__(kT) k_small(NetDev nd, uint32_t steps) {
  extern __shared__ __align__(16) char lds[];
  const SmallLds sh = small_lds(lds, nd.N);
  const uint64_t base = nd.ctrl->step_base;
  const uint32_t N = nd.N, R = nd.R;
  uint64_t pos = step_pos(nd, base);  // raster position of the step's spikes
  small_begin(nd, sh);
  const uint32_t lane = threadIdx.x & 63;
  float y[NPT], Ie[NPT], I[NPT][P];
  int32_t r[NPT];
  uint32_t pop[NPT], pk[NPT];
#pragma unroll
  for (int q = 0; q < NPT; ++q) {
    const uint32_t i = threadIdx.x + q * kT;
    if (i >= N) continue;
    pop[q] = find_pop(sh.h.spops, nd.npop, i);
    y[q] = nd.V[i];
    Ie[q] = nd.Ie[i];
    r[q] = nd.refr[i];
#pragma unroll
    for (int p = 0; p < P; ++p) I[q][p] = nd.Isyn[(size_t)i * P + p];
    pk[q] = nd.npois ? nd.small_pois[i] : 0;
    if (sh.h.spops[pop[q]].model == kSpikeGen) {  // y, r: next emission (counted from base, as bits) and cursor
      uint32_t c = nd.gen_next[i];
      const uint32_t e = nd.gen_off[i + 1];
      while (c < e && nd.gen_step[c] < base) ++c;
      r[q] = (int32_t)c;
      y[q] = __uint_as_float(gen_wait(nd, c, e, base));
    }
  }
  uint64_t nspk = 0, nev = 0, npairs = 0;
  bool mover = false;
  uint32_t rs = (uint32_t)(base % R);  // step slot
  for (uint32_t t = 0; t < steps; ++t) {
    const uint64_t n = base + t;
    if (threadIdx.x == 0) {
      nd.ring_base[rs] = pos;
      nd.chunk_base[n & (nd.chunk_ring - 1)] = pos;
      sh.h.n_spk[(t + 1) & 1] = 0;
    }
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
      const uint32_t i = threadIdx.x + q * kT;
      uint32_t m = 0;
      if (i < N) {
        // one neuron a thread: its constants stay in registers over the steps;
        // more: they are read from LDS each step, else they spill
        if constexpr (NPT > 1) asm volatile("" : "+v"(pop[q]));
        const PopDev& pp = sh.h.spops[pop[q]];
        int64_t a[P];
        small_input<P>(nd, sh, sh.h.pw[pop[q]], rs, i, a);
        if (pp.pois >= 0) {
#pragma unroll
          for (int p = 0; p < P; ++p)
            if (p == pp.pois_port) a[p] += (int64_t)pk[q] * pp.pois_wq;
        }
        float x[kMaxPorts], Iq[kMaxPorts];
#pragma unroll
        for (int p = 0; p < kMaxPorts; ++p) {
          x[p] = p < P ? __fmul_rn((float)a[p < P ? p : 0], pp.scale[p]) : 0.f;
          Iq[p] = p < P ? I[q][p < P ? p : 0] : 0.f;
        }
        if (pp.model >= kSpikeGen) {
          if (pp.model == kSpikeGen) {
            if (__float_as_uint(y[q]) == t) {
              const uint32_t e = nd.gen_off[i + 1];
              uint32_t c = (uint32_t)r[q];
              while (c < e && nd.gen_step[c] == n) { ++m; ++c; }
              r[q] = (int32_t)c;
              y[q] = __uint_as_float(gen_wait(nd, c, e, base));
            }
          } else {
            m = a[0] > 0 ? (uint32_t)x[0] : 0u;
          }
        } else {
          const LifK k = lif_consts(nd, pp, i);
          bool s;
          if (pp.model == kLifDelta) s = lif_delta_step(k, y[q], r[q], Ie[q], x[0]);
          else s = lif_exp_step(pp, k, y[q], Iq, r[q], Ie[q], x);
#pragma unroll
          for (int p = 0; p < P; ++p) I[q][p] = Iq[p];
          m = s ? 1u : 0u;
        }
        if (m > kMaxMult) { mover = true; m = kMaxMult; }
      }
      const uint64_t bal = __ballot(m != 0);
      if (bal) {  // wave-uniform: the wave's spikes, in gid order
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&sh.h.n_spk[t & 1], (uint32_t)__popcll(bal));
        at = __shfl(at, 0, 64) + (uint32_t)__popcll(bal & lanemask_lt());
        if (m) sh.spk[at] = i | (m << kMultShift);
      }
    }
    __syncthreads();
    const uint32_t ns = sh.h.n_spk[t & 1];
#pragma unroll
    for (int q = 0; q < NPT; ++q)  // the next step's Poisson counts, on their way during the delivery
      if (nd.npois && t + 1 < steps && threadIdx.x + q * kT < N) pk[q] = nd.small_pois[(size_t)(t + 1) * N + threadIdx.x + q * kT];
    // the thread's first spike's record, its reads on their way during the delivery
    SpikeRec rec = {0u, 0u, 0ull};
    if (threadIdx.x < ns) rec = spike_rec(nd, sh.spk[threadIdx.x]);
    small_deliver(nd, sh, ns, rs, [&](uint32_t j, uint32_t& b, uint32_t& e, uint32_t& m) {
      const uint32_t x = sh.spk[j];
      b = sh.row[x & kGidMask];
      e = sh.row[(x & kGidMask) + 1];
      m = x >> kMultShift;
    });
    for (uint32_t j = threadIdx.x; j < ns; j += kT) {
      if (j >= kT) rec = spike_rec(nd, sh.spk[j]);
      const uint32_t g = rec.entry & kGidMask;
      nd.log[(pos + j) & nd.log_mask] = rec.entry;
      nd.recent[(size_t)rs * N + j] = rec;
      nspk += 1;
      nev += sh.row[g + 1] - sh.row[g];
      npairs += __popcll(rec.mask);
    }
    if (threadIdx.x == 0) nd.ring_cnt[rs] = ns;
    pos += ns;
    if (++rs == R) rs = 0;
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < NPT; ++q) {
    const uint32_t i = threadIdx.x + q * kT;
    if (i >= N) continue;
    const int32_t model = sh.h.spops[pop[q]].model;
    if (model == kSpikeGen) nd.gen_next[i] = (uint32_t)r[q];
    if (model >= kSpikeGen) continue;
    nd.V[i] = y[q];
    nd.refr[i] = r[q];
#pragma unroll
    for (int p = 0; p < P; ++p)
      if (model == kLifExp && p < sh.h.spops[pop[q]].n_ports) nd.Isyn[(size_t)i * P + p] = I[q][p];
  }
  for (uint32_t w = threadIdx.x; w < R * N * nd.pull_words; w += kT) nd.small_ring[w] = sh.ring[w];
  nspk = wave_sum(nspk);
  nev = wave_sum(nev);
  npairs = wave_sum(npairs);
  if (lane == 0 && nspk) {
    __hip_atomic_fetch_add(&nd.blk_stats[2], nspk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_add(&nd.small_sent[0], npairs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_add(&nd.small_sent[1], nev, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (mover) atomicOr(&nd.ctrl->overflow, 1u);
  if (threadIdx.x == 0) {
    nd.ring_cnt[rs] = 0;  // the next step's counter, as the other step kernels leave it
    nd.ctrl->step_base = base + steps;
  }
}

// Poisson counts of steps step_base .. + steps, a byte each (at most 127).
__global__ void __launch_bounds__(kB) k_small_poisson(NetDev nd, uint32_t steps) {
  const uint32_t x = blockIdx.x * kB + threadIdx.x;
  if (x >= steps * nd.N) return;
  const uint32_t t = x / nd.N, i = x - t * nd.N;
  const PopDev& pp = nd.pops[find_pop(nd.pops, nd.npop, i)];
  nd.small_pois[x] = pp.pois >= 0 ? (uint8_t)poisson_draw(nd.pois_thr + (size_t)pp.pois * kPoisKmax, pp.seed,
                                                          i - pp.gid_base, nd.ctrl->step_base + t)
                                  : 0;
}

// Before a readback at step n = step_base: the waiting input of step n into
// acc[n & 1] (the other buffer cleared), and the pairs and events delivered so
// far: those of every spike sent less those that arrive after step n.
// Block 0: the counts; the others: the input.
__global__ void __launch_bounds__(kT) k_small_fold(NetDev nd) {
  const uint64_t n = nd.ctrl->step_base;
  if (blockIdx.x > 0) {
    const uint32_t i = (blockIdx.x - 1) * kT + threadIdx.x;
    if (i >= nd.N) return;
    const uint32_t r = (uint32_t)(n % nd.R);
    int64_t a[kMaxPorts] = {0, 0, 0, 0};
    const uint32_t* c = nd.small_ring + ((size_t)r * nd.N + i) * nd.pull_words;
    const PullPop& pw = nd.pull_pop[find_pop(nd.pops, nd.npop, i)];
    for (int k = 0; k < 2 * (int)nd.pull_words; ++k)
      a[pw.port[k]] += pw.wq[k] * (int64_t)(c[k >> 1] >> ((k & 1) * 16) & 0xffffu);
    for (uint32_t p = 0; p < nd.P; ++p) {
      nd.acc[((size_t)inbuf(n) * nd.N + i) * nd.P + p] = a[p];
      nd.acc[((size_t)inbuf(n + 1) * nd.N + i) * nd.P + p] = 0;
    }
    return;
  }
  __shared__ uint64_t red[kWaves];
  uint64_t ev, pr;
  sent_pending<kT>(nd, n, ev, pr);
  ev = block_sum(ev, red);
  pr = block_sum(pr, red);
  if (threadIdx.x == 0) {
    nd.sel_stats[0] = nd.small_sent[0] - pr;
    nd.sel_stats[1] = nd.small_sent[1] - ev;
  }
}

// After a restore at step n = step_base: the ring from the spikes in flight,
// and the pairs and events of the spikes sent from those delivered.
__global__ void __launch_bounds__(kT) k_small_restore(NetDev nd) {
  extern __shared__ __align__(16) char lds[];
  const SmallLds sh = small_lds(lds, nd.N);
  const uint64_t n = nd.ctrl->step_base;
  small_begin(nd, sh);  // the ring is cleared
  uint64_t ev = 0, pr = 0;
  for (uint32_t d = 1; d <= nd.dmax && d <= n; ++d) {
    const uint32_t slot = (uint32_t)((n - d) % nd.R), cnt = min(nd.ring_cnt[slot], nd.N);
    const SpikeRec* recs = nd.recent + (size_t)slot * nd.N;
    for (uint32_t j = threadIdx.x; j < cnt; j += kT) {  // what arrives after step n
      const uint32_t all = recs[j].grp_ptr + (uint32_t)__popcll(recs[j].mask);
      const uint32_t g = recs[j].grp_ptr + (uint32_t)__popcll(recs[j].mask & ((2ull << d) - 1ull));
      pr += all - g;
      ev += nd.grp_off[all] - nd.grp_off[g];
    }
    small_deliver(nd, sh, cnt, slot, [&](uint32_t j, uint32_t& b, uint32_t& e, uint32_t& m) {  // from step n on
      const SpikeRec rec = recs[j];
      b = (uint32_t)nd.grp_off[rec.grp_ptr + (uint32_t)__popcll(rec.mask & ((1ull << d) - 1ull))];
      e = (uint32_t)nd.grp_off[rec.grp_ptr + (uint32_t)__popcll(rec.mask)];
      m = rec.entry >> kMultShift;
    });
  }
  __syncthreads();
  for (uint32_t w = threadIdx.x; w < nd.R * nd.N * nd.pull_words; w += kT) nd.small_ring[w] = sh.ring[w];
  uint64_t s0 = 0, s1 = 0;
  for (uint32_t b = threadIdx.x; b < nd.sel_grid; b += kT) { s0 += nd.sel_stats[2 * b]; s1 += nd.sel_stats[2 * b + 1]; }
  pr = block_sum(pr + s0, sh.h.red[0]);
  ev = block_sum(ev + s1, sh.h.red[1]);
  if (threadIdx.x == 0) { nd.small_sent[0] = pr; nd.small_sent[1] = ev; }
  __syncthreads();
  for (uint32_t b = threadIdx.x; b < 2 * nd.sel_grid; b += kT) nd.sel_stats[b] = 0;  // set when read
}

// ---- set-up: rows of 32-bit words, a block per source ----
__global__ void __launch_bounds__(64) k_small_rows(NetDev nd, uint32_t* row, uint32_t* pay) {
  const uint32_t s = blockIdx.x, g0 = nd.grp_ptr[s], cls_mask = (1u << nd.cls_bits) - 1u;
  if (threadIdx.x == 0) {
    row[s] = (uint32_t)nd.grp_off[g0];
    if (s + 1 == nd.N) row[nd.N] = (uint32_t)nd.n_syn;
  }
  uint64_t mask = nd.src_mask[s];
  for (uint32_t g = g0; mask; ++g, mask &= mask - 1) {
    const uint32_t d = (uint32_t)__ffsll((unsigned long long)mask) - 1;
    for (uint64_t j = nd.grp_off[g] + threadIdx.x; j < nd.grp_off[g + 1]; j += 64) {
      const uint32_t w = nd.payload[j], c = w & cls_mask;
      pay[j] = (w >> nd.cls_bits) | (d << kDelShift) | ((uint32_t)nd.pull_slot[c] << kClsShift);
    }
  }
}

}  // namespace

size_t small_lds_bytes(const NetDev& nd) {
  return small_tail(nd.N) + (size_t)nd.R * nd.N * nd.pull_words * 4;
}

hipError_t launch_small_steps(const NetDev& nd, uint32_t steps, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  if (nd.npois) {
    const dim3 grid((uint32_t)(((uint64_t)steps * nd.N + kB - 1) / kB));
    launch(k_small_poisson, grid, dim3(kB), s, start, nullptr, nd, steps);
    if (start) start = nullptr;
  }
  auto k = nd.N <= kT ? (nd.P == 1 ? k_small<1, 1> : k_small<1, 2>) : (nd.P == 1 ? k_small<2, 1> : k_small<2, 2>);
  if (stop) hipExtLaunchKernelGGL(k, dim3(1), dim3(kT), small_lds_bytes(nd), s, start, stop, 0, nd, steps);
  else hipLaunchKernelGGL(k, dim3(1), dim3(kT), small_lds_bytes(nd), s, nd, steps);
  return hipGetLastError();
}

hipError_t launch_small_fold(const NetDev& nd, hipStream_t s) {
  hipLaunchKernelGGL(k_small_fold, dim3(1 + (nd.N + kT - 1) / kT), dim3(kT), 0, s, nd);
  return hipGetLastError();
}

hipError_t launch_small_restore(const NetDev& nd, hipStream_t s) {
  hipLaunchKernelGGL(k_small_restore, dim3(1), dim3(kT), small_lds_bytes(nd), s, nd);
  return hipGetLastError();
}

hipError_t launch_small_rows(const NetDev& nd, uint32_t* row, uint32_t* pay, hipStream_t s) {
  hipLaunchKernelGGL(k_small_rows, dim3(nd.N), dim3(64), 0, s, nd, row, pay);
  return hipGetLastError();
}

}  // namespace snn
