// kernels_build.hip -- on-device connectivity build (the paper keeps this on
// the host and names building it on the GPU as future work, Sec. 4).
//
// Connection rules (Sec. 2.1), one Philox4x64-10 block per work item, key
// (seed, 0), tag CONN, gids and p counted inside the projection's instance:
//   fixed in-degree  -- target t draws K sources: block (t, p << 40 | k >> 1),
//                       words 2(k&1) (source) and 2(k&1)+1 (delay);
//   fixed out-degree -- source s draws K targets: block (s, p << 40 | k >> 1),
//                       words 2(k&1) (target) and 2(k&1)+1 (delay);
//   all-to-all       -- target t, source index k: block (t, p << 40 | k >> 1),
//                       word 2(k&1)+1 (delay);
//   one-to-one       -- target t: block (t, p << 40), word 1 (delay);
//   fixed total      -- synapse j: block (j, p << 40), words 0 (source),
//                       1 (target), 2 (delay);
//   user-defined     -- synapse j as listed (no draw).
// A uniform index in a range of m is floor(u m / 2^64); a delay is the top 32
// bits of its word against the projection's threshold table.  A weight drawn
// from a distribution (Sec. 2.1) is the level of the top 32 bits of word k&3
// of block (c0, p << 40 | k >> 2) with tag WEIGHT, c0 the first counter word
// of the synapse's connection draw and k its draw index (0 for one-to-one
// and the fixed total number), against the level thresholds.
//
// Layout (Sec. 2.2, Fig. 1): synapses grouped per source into connection
// groups of equal delay, groups ordered by delay.  Build = counting sort by
// (source, delay) -- histogram, exclusive scan, scatter -- then every group is
// sorted by payload (target << 6 | class) so that the CSR is the unique
// canonical arrangement (source, delay, target, port, weight).
//
// The draws come by target, so their sources are random: counted and placed by
// device atomics on one counter per (source, delay), each synapse costs two of
// them and a 4-byte write anywhere in the CSR, and is drawn twice.  Networks
// of kBinBuildMin synapses and more are drawn once into bins of consecutive
// sources (8 bytes a synapse: source and delay, payload; a block reserves a
// bin's range for all its draws at once, so that writes fill lines), and a
// block per bin counts and places its synapses with counters in LDS.  3.0 10^8
// synapses (microcircuit stand-in): counting 11.1 and placing 23.4 ms by device
// atomics; through bins drawing 5.2, counting 0.5 and placing 4.8 ms.  Below
// 2^20 synapses the extra tables cost what the bins save (3 10^5: 0.76 against
// 0.88 ms in all, 2.5 10^6: 1.32 against 0.97 ms), and below 8 a neuron.  Where a bin overflows
// (sources drawn far from uniformly) or the scratch does not fit, the atomics
// do it.
#include <algorithm>

#include "kernels.h"
#include "philox_dev.h"

namespace snn {

namespace {

constexpr int kB = 256;
constexpr int kTagWeight = 3;  // Philox tag of the weight draws (connections 1, Poisson 2)

__device__ __forceinline__ uint32_t find_proj(const ProjDev* projs, uint32_t nproj, uint64_t q) {
  uint32_t lo = 0, hi = nproj;  // largest p with pair_begin <= q
  while (hi - lo > 1) {
    uint32_t mid = (lo + hi) >> 1;
    if (projs[mid].pair_begin <= q) lo = mid; else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ uint32_t draw_delay(const uint64_t* thr, uint32_t dmax, uint32_t u) {
  // smallest d in [1, dmax] with u < thr[d]; thr is non-decreasing, thr[dmax] = 2^32
  uint32_t lo = 1, hi = dmax;
  while (lo < hi) {
    uint32_t mid = (lo + hi) >> 1;
    if ((uint64_t)u < thr[mid]) hi = mid; else lo = mid + 1;
  }
  return lo;
}

__device__ __forceinline__ uint32_t draw_level(const uint64_t* thr, uint32_t levels, uint32_t u) {
  // smallest j with u < thr[j]; thr[levels - 1] = 2^32
  uint32_t lo = 0, hi = levels - 1;
  while (lo < hi) {
    uint32_t mid = (lo + hi) >> 1;
    if ((uint64_t)u < thr[mid]) hi = mid; else lo = mid + 1;
  }
  return lo;
}

__device__ __forceinline__ uint32_t find_pop(const uint32_t* pop_first, uint32_t npop, uint32_t gid) {
  uint32_t lo = 0, hi = npop;
  while (hi - lo > 1) {
    uint32_t mid = (lo + hi) >> 1;
    if (pop_first[mid] <= gid) lo = mid; else hi = mid;
  }
  return lo;
}

// The synapses of a work item (Sec. 2.1 rules; counter layout above): entity e
// and pair kp of projection p (pr), up to two synapses, each handed to
// emit(h, source, target, delay, class), h = 0 or 1.  Without kClass the class
// is not looked up (no weight is drawn).
template <bool kClass, class F>
__device__ __forceinline__ void gen_item(const ProjDev& pr, uint32_t p, uint64_t e, uint32_t kp, uint32_t dmax_cfg,
                                         const uint16_t* cls_of, const ProjW* pw, const uint32_t* pop_first,
                                         uint32_t npop, F emit) {
  // entity gid (instance-local in the counter): target, source, or none
  const uint32_t ent = pr.rule == kRuleOutDegree ? pr.src_first + (uint32_t)e
                     : pr.rule == kRuleTotal ? 0u : pr.tgt_first + (uint32_t)e;
  if (pr.rule == kRuleList) {  // user-defined: synapse e as listed, no draw
    const uint32_t src = pr.lsrc[e], tgt = pr.ltgt[e];
    uint32_t cls = 0;
    if (kClass) {
      const uint32_t k = pr.tpop ? pr.tpop - 1 : find_pop(pop_first, npop, tgt);
      const ProjW& w = pw[p];
      cls = w.levels ? w.cls[(k - w.pop0) * w.levels + w.lvl[e]] : cls_of[(size_t)p * npop + k];
    }
    emit(0, src, tgt, (uint32_t)pr.ldel[e], cls);
    return;
  }
  const uint64_t c0 = pr.rule == kRuleTotal ? e : (uint64_t)(ent - pr.gid_base);
  const uint64_t c1 = ((uint64_t)pr.index << 40) | kp;
  const U64x4 blk = philox4x64_10(c0, c1, kTagConn, 0, pr.seed, 0);
  const int nh = (pr.rule == kRuleOneToOne || pr.rule == kRuleTotal) ? 1 : 2;
  // weight draws of this item's synapses (drawn projections)
  U64x4 wblk = {};
  if (kClass && pw[p].levels)
    wblk = philox4x64_10(c0, ((uint64_t)pr.index << 40) | (kp >> 1), kTagWeight, 0, pr.seed, 0);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t k = 2 * kp + h;
    if (h >= nh || k >= pr.K) break;
    uint32_t src, tgt, d;
    switch (pr.rule) {
      case kRuleOutDegree:
        src = ent;
        tgt = pr.tgt_first + (uint32_t)__umul64hi(blk.w[2 * h], (uint64_t)pr.tgt_n);
        d = draw_delay(pr.thr, dmax_cfg, (uint32_t)(blk.w[2 * h + 1] >> 32));
        break;
      case kRuleAllToAll:
        src = pr.src_first + k;
        tgt = ent;
        d = draw_delay(pr.thr, dmax_cfg, (uint32_t)(blk.w[2 * h + 1] >> 32));
        break;
      case kRuleOneToOne:
        src = pr.src_first + (uint32_t)e;
        tgt = ent;
        d = draw_delay(pr.thr, dmax_cfg, (uint32_t)(blk.w[1] >> 32));
        break;
      case kRuleTotal:
        src = pr.src_first + (uint32_t)__umul64hi(blk.w[0], (uint64_t)pr.src_n);
        tgt = pr.tgt_first + (uint32_t)__umul64hi(blk.w[1], (uint64_t)pr.tgt_n);
        d = draw_delay(pr.thr, dmax_cfg, (uint32_t)(blk.w[2] >> 32));
        break;
      default:  // fixed in-degree
        src = pr.src_first + (uint32_t)__umul64hi(blk.w[2 * h], (uint64_t)pr.src_n);
        tgt = ent;
        d = draw_delay(pr.thr, dmax_cfg, (uint32_t)(blk.w[2 * h + 1] >> 32));
        break;
    }
    uint32_t cls = 0;
    if (kClass) {
      const uint32_t kpop = pr.tpop ? pr.tpop - 1 : find_pop(pop_first, npop, tgt);
      const ProjW& w = pw[p];
      if (w.levels) {
        const uint32_t kk = k & 3u;  // word of the weight block
        const uint64_t u = kk == 0 ? wblk.w[0] : kk == 1 ? wblk.w[1] : kk == 2 ? wblk.w[2] : wblk.w[3];
        const uint32_t j = draw_level(w.thr, w.levels, (uint32_t)(u >> 32));
        cls = w.cls[(kpop - w.pop0) * w.levels + j];
      } else {
        cls = cls_of[(size_t)p * npop + kpop];
      }
    }
    emit(h, src, tgt, d, cls);
  }
}

// Item q of each lane, consecutive over the wave from its lane 0 on (lanes past
// the last item may have left).  The wave goes through the projections its items
// lie in, mostly one: its record, its first item's entity and the rule's branch
// are the wave's, so that a lane has no search and no 64-bit division of its own
// (714 vector instructions an item with them, of which the generator takes 290;
// 3.0 10^8 synapses into bins 5.3 -> 4.5 ms).
template <bool kClass, class F>
__device__ __forceinline__ void gen_wave(const ProjDev* __restrict__ projs, uint32_t nproj, uint64_t total_pairs,
                                         uint64_t q, uint32_t dmax_cfg, const uint16_t* cls_of, const ProjW* pw,
                                         const uint32_t* pop_first, uint32_t npop, F emit) {
  const uint64_t q0 = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)q) |
                      (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(q >> 32)) << 32;
  const uint64_t last = min(q0 + 64, total_pairs);
  for (uint64_t from = q0; from < last;) {  // wave-uniform
    const uint32_t p = find_proj(projs, nproj, from);
    const ProjDev& pr = projs[p];
    const uint64_t end = p + 1 < nproj ? min(projs[p + 1].pair_begin, total_pairs) : total_pairs;
    const uint64_t local = from - pr.pair_begin, e0 = local / pr.kpairs;
    if (q >= from && q < end) {
      const uint32_t t = (uint32_t)(local - e0 * pr.kpairs) + (uint32_t)(q - from);
      const uint32_t de = pr.kpairs >= 64 ? (t >= pr.kpairs ? 1u : 0u) : t / pr.kpairs;
      gen_item<kClass>(pr, p, e0 + de, t - de * pr.kpairs, dmax_cfg, cls_of, pw, pop_first, npop, emit);
    }
    from = end;
  }
}

// Every synapse counted (histogram) or scattered into its (source, delay)
// bucket by device atomics.
template <bool kScatter>
__global__ void __launch_bounds__(kB) k_gen(const ProjDev* __restrict__ projs, uint32_t nproj, uint64_t total_pairs,
                                             uint32_t dmax_cfg, uint32_t D1, uint32_t* cnt,
                                             unsigned long long* cursor, uint32_t* payload, const uint16_t* cls_of,
                                             const ProjW* pw, const uint32_t* pop_first, uint32_t npop,
                                             uint32_t cls_bits) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; q < total_pairs; q += stride)
    gen_wave<kScatter>(projs, nproj, total_pairs, q, dmax_cfg, cls_of, pw, pop_first, npop,
                       [&](int, uint32_t src, uint32_t tgt, uint32_t d, uint32_t cls) {
                         const uint64_t bucket = (uint64_t)src * D1 + d;
                         if (!kScatter) {
                           atomicAdd(&cnt[bucket], 1u);
                         } else {
                           const unsigned long long slot = atomicAdd(&cursor[bucket], 1ull);
                           payload[slot] = (tgt << cls_bits) | cls;
                         }
                       });
}

// ---- drawn once, through bins of consecutive sources ----
constexpr int kBT = 1024;     // threads of the three kernels
// Work items of a thread of k_bin_gen, up to 2 synapses each: as many as stay in
// registers at eight waves a SIMD (two blocks on a CU).  8 items with one block
// 4.5 ms for 3.0 10^8 synapses, with two 3.85 (in scratch memory), 4 items 3.2.
constexpr int kBinItems = 4;

// Block = kBT * kBinItems work items.  Their synapses stay in registers while
// they are counted per bin in LDS; one device atomic per touched bin reserves
// its place, then each synapse is written.  A bin that is full sets *over.
__global__ void __launch_bounds__(kBT, 8) k_bin_gen(const ProjDev* __restrict__ projs, uint32_t nproj,
                                                 uint64_t total_pairs, uint32_t dmax_cfg, const uint16_t* cls_of,
                                                 const ProjW* pw, const uint32_t* pop_first, uint32_t npop,
                                                 uint32_t cls_bits, BinBuild bb) {
  extern __shared__ uint32_t sbuf[];
  uint32_t* cur = sbuf;               // synapses of the block per bin, then the bin's cursor
  uint32_t* first = sbuf + bb.nbin;   // first source of each bin
  for (uint32_t b = threadIdx.x; b < bb.nbin; b += kBT) { cur[b] = 0; first[b] = bb.first[b]; }
  __syncthreads();
  uint32_t hi[2 * kBinItems], lo[2 * kBinItems], bin[kBinItems];
#pragma unroll
  for (int it = 0; it < kBinItems; ++it) {
    const uint64_t q = ((uint64_t)blockIdx.x * kBinItems + it) * kBT + threadIdx.x;
    bin[it] = 0xffffffffu;
    if (q < total_pairs)
      gen_wave<true>(projs, nproj, total_pairs, q, dmax_cfg, cls_of, pw, pop_first, npop,
                     [&](int h, uint32_t src, uint32_t tgt, uint32_t d, uint32_t cls) {
                       const uint32_t b = bb.of_src[src];
                       atomicAdd(&cur[b], 1u);
                       const uint32_t x = ((src - first[b]) << 6) | d, y = (tgt << cls_bits) | cls;
                       if (h == 0) { hi[2 * it] = x; lo[2 * it] = y; bin[it] = (bin[it] & 0xffff0000u) | b; }
                       else { hi[2 * it + 1] = x; lo[2 * it + 1] = y; bin[it] = (bin[it] & 0xffffu) | (b << 16); }
                     });
  }
  __syncthreads();
  for (uint32_t b = threadIdx.x; b < bb.nbin; b += kBT)
    if (cur[b]) {
      const uint32_t c = cur[b];
      const uint32_t at = __hip_atomic_fetch_add(&bb.cnt[b], c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (at + c > bb.cap[b] || at + c < at) { *bb.over = 1u; cur[b] = 0xffffffffu; }
      else cur[b] = at;
    }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < kBinItems; ++it)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t b = h ? bin[it] >> 16 : bin[it] & 0xffffu;
      if (b == 0xffffu || cur[b] == 0xffffffffu) continue;  // none, or no room (all of the block's)
      const uint32_t at = atomicAdd(&cur[b], 1u);
      bb.rec[bb.off[b] + at] = make_uint2(hi[2 * it + h], lo[2 * it + h]);
    }
}

// Block = one bin: its synapses per (source, delay), counted in LDS.
__global__ void __launch_bounds__(kBT) k_bin_count(BinBuild bb, uint32_t D1, uint32_t* cnt) {
  extern __shared__ uint32_t sbuf[];
  const uint32_t b = blockIdx.x, f = bb.first[b], words = (bb.first[b + 1] - f) * D1;
  for (uint32_t w = threadIdx.x; w < words; w += kBT) sbuf[w] = 0;
  __syncthreads();
  const uint2* rec = bb.rec + bb.off[b];
  const uint32_t n = bb.cnt[b];
  for (uint32_t j = threadIdx.x; j < n; j += kBT) {
    const uint32_t x = rec[j].x;
    atomicAdd(&sbuf[(x >> 6) * D1 + (x & 63u)], 1u);
  }
  __syncthreads();
  for (uint32_t w = threadIdx.x; w < words; w += kBT) cnt[(uint64_t)f * D1 + w] = sbuf[w];
}

// Block = one bin: its synapses placed at their (source, delay) groups, the
// cursors (counted from the bin's first synapse) in LDS.
__global__ void __launch_bounds__(kBT) k_bin_place(BinBuild bb, uint32_t D1, const uint64_t* __restrict__ off,
                                                   uint32_t* __restrict__ payload) {
  extern __shared__ uint32_t sbuf[];
  const uint32_t b = blockIdx.x, f = bb.first[b], words = (bb.first[b + 1] - f) * D1;
  const uint64_t base = off[(uint64_t)f * D1];
  for (uint32_t w = threadIdx.x; w < words; w += kBT) sbuf[w] = (uint32_t)(off[(uint64_t)f * D1 + w] - base);
  __syncthreads();
  const uint2* rec = bb.rec + bb.off[b];
  const uint32_t n = bb.cnt[b];
  for (uint32_t j0 = 0; j0 < n; j0 += 4 * kBT) {
    uint2 r[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t j = j0 + u * kBT + threadIdx.x;
      r[u] = j < n ? rec[j] : make_uint2(0xffffffffu, 0u);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (r[u].x != 0xffffffffu) payload[base + atomicAdd(&sbuf[(r[u].x >> 6) * D1 + (r[u].x & 63u)], 1u)] = r[u].y;
  }
}

// Block = one bin: its synapses brought to their sources' rows (words into
// payload, delays into del), for k_row_sort to order.  kRowChunk of them at a
// time are put in source order in LDS, so that a source's are written side by
// side: placed at their (source, delay) groups at once, each by itself, 3.0 10^8
// took 4.8 ms (every 4-byte store a line of its own), and the sorting of the
// groups, a wave each behind two dependent reads, another 2.7; now 1.1 here and
// 2.8 in k_row_sort.
constexpr int kRowItems = 8;
constexpr uint32_t kRowChunk = kRowItems * kBT;
__global__ void __launch_bounds__(kBT) k_bin_rows(BinBuild bb, uint32_t D1, const uint64_t* __restrict__ off,
                                                  uint32_t* __restrict__ payload, uint8_t* __restrict__ del) {
  extern __shared__ uint32_t sbuf[];
  uint32_t* word = sbuf;                                            // [kRowChunk]
  uint16_t* src = reinterpret_cast<uint16_t*>(word + kRowChunk);    // [kRowChunk]
  uint8_t* dly = reinterpret_cast<uint8_t*>(src + kRowChunk);       // [kRowChunk]
  uint32_t* cur = reinterpret_cast<uint32_t*>(dly + kRowChunk);     // [kBT] next place of a source
  uint32_t* cnt = cur + kBT;                                        // [kBT] the chunk's synapses of a source
  uint32_t* first = cnt + kBT;                                      // [kBT] ... and their place in the chunk
  __shared__ uint32_t wsum[kBT / 64];
  const uint32_t b = blockIdx.x, f = bb.first[b], ns = bb.first[b + 1] - f, tid = threadIdx.x;
  const uint64_t base = off[(uint64_t)f * D1];
  if (tid < ns) cur[tid] = (uint32_t)(off[(uint64_t)(f + tid) * D1] - base);
  const uint2* rec = bb.rec + bb.off[b];
  const uint32_t n = bb.cnt[b];
  for (uint32_t j0 = 0; j0 < n; j0 += kRowChunk) {  // block-uniform
    const uint32_t m = min(kRowChunk, n - j0);
    uint2 r[kRowItems];
    uint32_t rank[kRowItems];
#pragma unroll
    for (int u = 0; u < kRowItems; ++u) {
      const uint32_t j = u * kBT + tid;
      r[u] = j < m ? rec[j0 + j] : make_uint2(0u, 0u);
    }
    cnt[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kRowItems; ++u)
      if (u * kBT + tid < m) rank[u] = atomicAdd(&cnt[r[u].x >> 6], 1u);
    __syncthreads();
    const uint32_t c = cnt[tid];
    uint32_t incl = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(incl, o, 64);
      if ((tid & 63) >= (uint32_t)o) incl += y;
    }
    if ((tid & 63) == 63) wsum[tid >> 6] = incl;
    __syncthreads();
    uint32_t before = 0;
    for (uint32_t w = 0; w < tid >> 6; ++w) before += wsum[w];
    first[tid] = before + incl - c;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kRowItems; ++u)
      if (u * kBT + tid < m) {
        const uint32_t s = r[u].x >> 6, at = first[s] + rank[u];
        word[at] = r[u].y;
        src[at] = (uint16_t)s;
        dly[at] = (uint8_t)(r[u].x & 63u);
      }
    __syncthreads();
    for (uint32_t j = tid; j < m; j += kBT) {
      const uint32_t s = src[j];
      const uint64_t at = base + cur[s] + (j - first[s]);
      payload[at] = word[j];
      del[at] = dly[j];
    }
    __syncthreads();
    if (tid < ns) cur[tid] += c;
  }
}

uint32_t grid_for(uint64_t work, uint32_t per_block, uint32_t cap) {
  uint64_t g = (work + per_block - 1) / per_block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (uint32_t)g;
}

// ---------------------------------------------------------------- scan
constexpr int kScanItems = 16;
constexpr uint64_t kScanTile = (uint64_t)kB * kScanItems;

// inclusive wave scan of 64-bit values
__device__ __forceinline__ uint64_t wave_incl_scan(uint64_t v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t t = __shfl_up(v, o, 64);
    if (lane >= o) v += t;
  }
  return v;
}

// exclusive block scan for blockDim.x == kB; returns exclusive prefix, *total = block sum
__device__ __forceinline__ uint64_t block_excl_scan(uint64_t v, uint64_t* lds4, uint64_t* total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint64_t incl = wave_incl_scan(v);
  if (lane == 63) lds4[wv] = incl;
  __syncthreads();
  uint64_t before = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < kB / 64; ++i) {
    const uint64_t x = lds4[i];
    if (i < wv) before += x;
    tot += x;
  }
  __syncthreads();
  *total = tot;
  return before + incl - v;
}

template <typename T>
__global__ void __launch_bounds__(kB) k_tile_sums(const T* __restrict__ in, uint64_t n, uint64_t* sums) {
  __shared__ uint64_t lds[kB / 64];
  const uint64_t base = (uint64_t)blockIdx.x * kScanTile + (uint64_t)threadIdx.x * kScanItems;
  uint64_t s = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const uint64_t j = base + i;
    if (j < n) s += (uint64_t)in[j];
  }
  uint64_t tot;
  (void)block_excl_scan(s, lds, &tot);
  if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

template <typename T>
__global__ void __launch_bounds__(kB) k_tile_scan(const T* __restrict__ in, uint64_t n, const uint64_t* tile_off,
                                                   uint64_t* out, uint64_t* total_out) {
  __shared__ uint64_t lds[kB / 64];
  const uint64_t base = (uint64_t)blockIdx.x * kScanTile + (uint64_t)threadIdx.x * kScanItems;
  uint64_t v[kScanItems];
  uint64_t s = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const uint64_t j = base + i;
    v[i] = (j < n) ? (uint64_t)in[j] : 0;
    s += v[i];
  }
  uint64_t tot;
  uint64_t run = block_excl_scan(s, lds, &tot) + (tile_off ? tile_off[blockIdx.x] : 0);
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const uint64_t j = base + i;
    if (j < n) out[j] = run;
    run += v[i];
  }
  if (total_out && blockIdx.x == gridDim.x - 1 && threadIdx.x == kB - 1) *total_out = run;
}

template <typename T>
hipError_t scan_impl(const T* in, uint64_t n, uint64_t* out, uint64_t* tmp, hipStream_t s) {
  // out has n + 1 entries; out[n] = total
  const uint64_t tiles = (n + kScanTile - 1) / kScanTile;
  if (n == 0) {
    return hipMemsetAsync(out, 0, sizeof(uint64_t), s);
  }
  if (tiles == 1) {
    hipLaunchKernelGGL(k_tile_scan<T>, dim3(1), dim3(kB), 0, s, in, n, (const uint64_t*)nullptr, out, out + n);
    return hipGetLastError();
  }
  uint64_t* sums = tmp;             // tiles
  uint64_t* sums_scan = tmp + tiles;  // tiles + 1
  uint64_t* rest = sums_scan + tiles + 1;
  hipLaunchKernelGGL(k_tile_sums<T>, dim3((uint32_t)tiles), dim3(kB), 0, s, in, n, sums);
  hipError_t e = scan_impl<uint64_t>(sums, tiles, sums_scan, rest, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_tile_scan<T>, dim3((uint32_t)tiles), dim3(kB), 0, s, in, n, (const uint64_t*)sums_scan, out,
                     out + n);
  return hipGetLastError();
}

__global__ void __launch_bounds__(kB) k_masks(const uint32_t* __restrict__ cnt, uint32_t N, uint32_t D1, uint64_t* mask,
                                              uint64_t* ngroups, uint32_t* longest) {
  const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= N) return;
  uint64_t m = 0;
  uint32_t ng = 0, len = 0;
  for (uint32_t d = 1; d < D1; ++d) {
    const uint32_t c = cnt[(uint64_t)s * D1 + d];
    if (c) { m |= 1ull << d; ++ng; }
    len += c;
  }
  if (longest) atomicMax(longest, len);
  mask[s] = m;
  ngroups[s] = ng;
}

__global__ void __launch_bounds__(kB) k_grp_off(const uint32_t* __restrict__ cnt, const uint64_t* __restrict__ off,
                                                const uint64_t* __restrict__ grp_ptr64, uint32_t N, uint32_t D1,
                                                uint64_t* grp_off, uint32_t* grp_ptr32) {
  const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s > N) return;
  grp_ptr32[s] = (uint32_t)grp_ptr64[s];
  if (s == N) return;
  uint64_t g = grp_ptr64[s];
  for (uint32_t d = 1; d < D1; ++d) {
    const uint64_t b = (uint64_t)s * D1 + d;
    if (cnt[b]) grp_off[g++] = off[b];
  }
}

// ------------------------------------------------------------ group sorting
// Short groups, one wave per group: a bitonic network over 64 R keys in
// registers (element 64 r + lane in register r), R the smallest of 1, 2, .. 16
// that holds the group; the padding sorts to the end.  Bound by its vector
// instructions: 130 keys take ~500 a wave, where ranking every key against
// every other took ~1,400; 3.0 10^8 synapses in groups of 1 to ~900: 13.8 ms
// by ranks up to 512 keys and a block sort beyond, now 2.7 ms.
// Longer groups are listed for the block sort.
constexpr uint32_t kWaveSortMax = 1024;
constexpr uint32_t kBlockSortMax = 16384;
constexpr int kRowSortRegs = 16;  // words of a row per thread of k_row_sort
// ... for rows of that many words on the average: in shorter ones most of a block
// has no word, and a wave per group is faster (builds by group and by row, 6.4
// 10^6 synapses in rows of 64: 2.66 and 2.85 ms; 1.3 10^7 of 128: 3.15, 3.11; 10^7
// of 200: 2.30, 2.22)
constexpr uint64_t kRowSortMean = 128;

template <int R>
__device__ __forceinline__ void wave_sort(uint32_t* v, uint32_t lane) {
#pragma unroll
  for (int k = 2; k <= 64 * R; k <<= 1) {
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1) {
      if (j >= 64) {  // partners in one lane's registers
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int p = r ^ (j >> 6);
          if (p > r) {
            const bool up = ((r << 6) & k) == 0;  // k > 64 here: the direction does not depend on the lane
            const uint32_t a = min(v[r], v[p]), b = max(v[r], v[p]);
            v[r] = up ? a : b;
            v[p] = up ? b : a;
          }
        }
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const uint32_t x = v[r], y = __shfl_xor(x, j, 64);
          const bool up = (k >= 64 ? ((r << 6) & k) : (int)(lane & k)) == 0;
          const bool low = (lane & j) == 0;
          v[r] = (up == low) ? min(x, y) : max(x, y);
        }
      }
    }
  }
}

template <int R>
__device__ __forceinline__ void sort_group(const uint32_t* in, uint32_t* p, uint32_t L, uint32_t lane) {
  uint32_t v[R];
#pragma unroll
  for (int r = 0; r < R; ++r) v[r] = (64 * r + lane < L) ? in[64 * r + lane] : 0xffffffffu;
  wave_sort<R>(v, lane);
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (64 * r + lane < L) p[64 * r + lane] = v[r];
}

__global__ void __launch_bounds__(kB) k_segsort_wave(const uint64_t* __restrict__ grp_off, uint64_t n_groups,
                                                     uint32_t* payload, unsigned long long* longer, uint32_t* n_longer,
                                                     uint64_t cap) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t nw = (uint64_t)gridDim.x * (kB / 64);
  for (uint64_t g = (uint64_t)blockIdx.x * (kB / 64) + wv; g < n_groups; g += nw) {  // wave-uniform
    const uint64_t b = grp_off[g];
    const uint64_t L64 = grp_off[g + 1] - b;
    if (L64 <= 1) continue;
    if (L64 > kWaveSortMax) {
      if (lane == 0) {
        const uint32_t k = atomicAdd(n_longer, 1u);
        if (k < cap) longer[k] = g;
      }
      continue;
    }
    const uint32_t L = (uint32_t)L64;
    if (L <= 64) sort_group<1>(payload + b, payload + b, L, lane);
    else if (L <= 128) sort_group<2>(payload + b, payload + b, L, lane);
    else if (L <= 256) sort_group<4>(payload + b, payload + b, L, lane);
    else if (L <= 512) sort_group<8>(payload + b, payload + b, L, lane);
    else sort_group<16>(payload + b, payload + b, L, lane);
  }
}

// The same from the rows of k_bin_rows: a block reads a source's row, places its
// words at their groups in LDS, and its waves sort these into the payload.  A
// block has a thread for 16 words of a row: a launch for each block size (with the
// largest for all, 3.0 10^8 synapses in rows of 2,100 .. 8,200 took 3.3 ms, now
// 2.8).
template <int kTh>
__global__ void __launch_bounds__(kTh) k_row_sort(const uint64_t* __restrict__ off, const uint32_t* __restrict__ grp_ptr,
                                                  uint32_t D1, const uint8_t* __restrict__ del, uint32_t* payload,
                                                  uint32_t above, unsigned long long* longer, uint32_t* n_longer,
                                                  uint64_t cap) {
  constexpr int kItems = kRowSortRegs;
  __shared__ uint32_t buf[kItems * kTh], cur[64], first[65];
  const uint32_t s = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint64_t o = off[(uint64_t)s * D1];
  const uint32_t len = (uint32_t)(off[(uint64_t)(s + 1) * D1] - o);
  if (len <= above || len > (uint32_t)(kItems * kTh)) return;  // block-uniform: another launch's
  uint32_t w[kItems], d[kItems];
#pragma unroll
  for (int q = 0; q < kItems; ++q) {
    const uint32_t j = q * kTh + tid;
    w[q] = j < len ? payload[o + j] : 0u;
    d[q] = j < len ? del[o + j] : 0u;
  }
  if (tid < 64) {
    const uint32_t x = tid < D1 ? (uint32_t)(off[(uint64_t)s * D1 + tid] - o) : len;
    first[tid] = x;
    cur[tid] = x;
    if (tid == 0) first[64] = len;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kItems; ++q)
    if (q * kTh + tid < len) buf[atomicAdd(&cur[d[q]], 1u)] = w[q];
  __syncthreads();
  for (uint32_t k = wv; k < D1; k += kTh / 64) {  // wave-uniform
    const uint32_t b = first[k], L = first[k + 1] - b;
    if (L == 0) continue;
    uint32_t* out = payload + o + b;
    const uint32_t* in = buf + b;
    if (L > kWaveSortMax) {
      for (uint32_t j = lane; j < L; j += 64) out[j] = in[j];
      const uint32_t g = grp_ptr[s] + (uint32_t)__popcll(__ballot(lane < k && first[lane + 1] > first[lane]));
      if (lane == 0) {
        const uint32_t at = atomicAdd(n_longer, 1u);
        if (at < cap) longer[at] = g;
      }
    } else if (L <= 64) sort_group<1>(in, out, L, lane);
    else if (L <= 128) sort_group<2>(in, out, L, lane);
    else if (L <= 256) sort_group<4>(in, out, L, lane);
    else if (L <= 512) sort_group<8>(in, out, L, lane);
    else sort_group<16>(in, out, L, lane);
  }
}

// Bitonic sort in LDS for the listed groups, of (kWaveSortMax, kBlockSortMax];
// one block per group; longer groups are listed for the host.
constexpr int kSB = 1024;
__global__ void __launch_bounds__(kSB) k_segsort_block(const uint64_t* __restrict__ grp_off,
                                                       const unsigned long long* __restrict__ longer,
                                                       const uint32_t* __restrict__ n_longer, uint32_t* payload,
                                                       unsigned long long* big, uint32_t* nbig, uint32_t big_cap) {
  extern __shared__ uint32_t sbuf[];
  const uint32_t n = *n_longer;
  for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const uint64_t g = longer[i];
    const uint64_t b = grp_off[g];
    const uint64_t L64 = grp_off[g + 1] - b;
    if (L64 > kBlockSortMax) {
      if (threadIdx.x == 0) {
        const uint32_t k = atomicAdd(nbig, 1u);
        if (k < big_cap) big[k] = g;
      }
      continue;
    }
    const uint32_t L = (uint32_t)L64;
    uint32_t M = 1;
    while (M < L) M <<= 1;
    for (uint32_t i = threadIdx.x; i < M; i += kSB) sbuf[i] = (i < L) ? payload[b + i] : 0xFFFFFFFFu;
    __syncthreads();
    for (uint32_t k = 2; k <= M; k <<= 1) {
      for (uint32_t j = k >> 1; j > 0; j >>= 1) {
        for (uint32_t i = threadIdx.x; i < M; i += kSB) {
          const uint32_t ix = i ^ j;
          if (ix > i) {
            const uint32_t a = sbuf[i], c = sbuf[ix];
            const bool up = (i & k) == 0;
            if ((a > c) == up) { sbuf[i] = c; sbuf[ix] = a; }
          }
        }
        __syncthreads();
      }
    }
    for (uint32_t i = threadIdx.x; i < L; i += kSB) payload[b + i] = sbuf[i];
    __syncthreads();
  }
}


// ------------------------------------------------------------ tile runs
// A group's synapses are sorted by target, so those onto one tile of the
// binned delivery lie together: a run.  One wave per group finds the run
// starts (a synapse whose tile differs from its predecessor's) with a ballot
// over 64 synapses at a time.  Pass kFill = false counts them per group;
// pass kFill = true writes run k of group g as run_desc[grp_run[g] + k] =
// tile << kRunLenBits | length, in synapse order: each start closes the run
// before it (the previous start in the window, or the run still open from
// the earlier windows), and the last run closes at the group's end.  A group
// of kRunMaxGroup synapses or more sets *too_long (no runs for the network).
template <bool kFill>
__global__ void __launch_bounds__(kB) k_runs(const uint64_t* __restrict__ grp_off, uint64_t n_groups,
                                             const uint32_t* __restrict__ payload, uint32_t cls_bits, uint32_t tsh,
                                             uint32_t* __restrict__ cnt, const uint64_t* __restrict__ grp_run,
                                             uint32_t* __restrict__ run_desc, uint32_t* too_long) {
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t nwaves = ((uint64_t)gridDim.x * kB) >> 6;
  for (uint64_t g = ((uint64_t)blockIdx.x * kB + threadIdx.x) >> 6; g < n_groups; g += nwaves) {
    const uint64_t a = grp_off[g], b = grp_off[g + 1];
    if (!kFill && lane == 0 && b - a >= kRunMaxGroup) atomicOr(too_long, 1u);
    uint64_t runs = 0;                 // run starts before this window
    uint32_t prev_tile = 0xffffffffu;  // tile of the synapse before the window
    uint64_t open_pos = a;             // first synapse of the open run
    uint32_t open_tile = 0;
    const uint64_t base = kFill ? grp_run[g] : 0;
    for (uint64_t j0 = a; j0 < b; j0 += 64) {  // wave-uniform
      const uint64_t j = j0 + lane;
      const bool in = j < b;
      const uint32_t t = in ? (payload[j] >> cls_bits) >> tsh : 0xffffffffu;
      const uint32_t left = __shfl(t, (int)(lane ? lane - 1 : 0), 64);
      const bool start = in && t != (lane ? left : prev_tile);
      const uint64_t m = __ballot(start);
      if (kFill) {
        const uint64_t below = m & ((1ull << lane) - 1ull);
        const uint32_t pl = below ? 63u - (uint32_t)__clzll(below) : 0u;
        const uint32_t tile_pl = __shfl(t, (int)pl, 64);
        const uint64_t k = runs + (uint64_t)__popcll(below);
        if (start && k > 0) {
          const uint64_t pos = below ? j0 + pl : open_pos;
          const uint32_t tile = below ? tile_pl : open_tile;
          run_desc[base + k - 1] = (tile << kRunLenBits) | (uint32_t)(j - pos);
        }
      }
      if (m) {
        const uint32_t hb = 63u - (uint32_t)__clzll(m);
        open_pos = j0 + hb;
        open_tile = __shfl(t, (int)hb, 64);
      }
      const uint32_t last = (uint32_t)((b - j0 < 64 ? b - j0 : 64) - 1);
      prev_tile = __shfl(t, (int)last, 64);
      runs += (uint64_t)__popcll(m);
    }
    if (lane == 0) {
      if (!kFill) cnt[g] = (uint32_t)runs;
      else if (runs) run_desc[base + runs - 1] = (open_tile << kRunLenBits) | (uint32_t)(b - open_pos);
    }
  }
}

}  // namespace

hipError_t launch_gen_count(const ProjDev* projs, uint32_t nproj, uint64_t total_pairs, uint32_t dmax_cfg,
                            uint32_t D1, uint32_t* cnt, hipStream_t s) {
  if (total_pairs == 0) return hipSuccess;
  hipLaunchKernelGGL(k_gen<false>, dim3(grid_for(total_pairs, kB, 65536)), dim3(kB), 0, s, projs, nproj, total_pairs,
                     dmax_cfg, D1, cnt, (unsigned long long*)nullptr, (uint32_t*)nullptr, (const uint16_t*)nullptr,
                     (const ProjW*)nullptr, (const uint32_t*)nullptr, 0u, 0u);
  return hipGetLastError();
}

hipError_t launch_gen_scatter(const ProjDev* projs, uint32_t nproj, uint64_t total_pairs, uint32_t dmax_cfg,
                              uint32_t D1, uint64_t* cursor, uint32_t* payload, const uint16_t* cls_of,
                              const ProjW* pw, const uint32_t* pop_first, uint32_t npop, uint32_t cls_bits,
                              hipStream_t s) {
  if (total_pairs == 0) return hipSuccess;
  hipLaunchKernelGGL(k_gen<true>, dim3(grid_for(total_pairs, kB, 65536)), dim3(kB), 0, s, projs, nproj, total_pairs,
                     dmax_cfg, D1, (uint32_t*)nullptr, (unsigned long long*)cursor, payload, cls_of, pw, pop_first,
                     npop, cls_bits);
  return hipGetLastError();
}

size_t scan_tmp_words(uint64_t n) {
  size_t w = 0;
  uint64_t m = n;
  while (true) {
    const uint64_t tiles = (m + kScanTile - 1) / kScanTile;
    if (tiles <= 1) break;
    w += 2 * tiles + 1;
    m = tiles;
  }
  return w + 1;
}

hipError_t launch_scan_u32(const uint32_t* in, uint64_t n, uint64_t* out, uint64_t* tmp, hipStream_t s) {
  return scan_impl<uint32_t>(in, n, out, tmp, s);
}

hipError_t launch_scan_u64(const uint64_t* in, uint64_t n, uint64_t* out, uint64_t* tmp, hipStream_t s) {
  return scan_impl<uint64_t>(in, n, out, tmp, s);
}

hipError_t launch_masks(const uint32_t* cnt, uint32_t N, uint32_t D1, uint64_t* mask, uint64_t* ngroups,
                        uint32_t* longest, hipStream_t s) {
  hipLaunchKernelGGL(k_masks, dim3((N + kB - 1) / kB), dim3(kB), 0, s, cnt, N, D1, mask, ngroups, longest);
  return hipGetLastError();
}

hipError_t launch_grp_off(const uint32_t* cnt, const uint64_t* off, const uint64_t* grp_ptr64, uint32_t N, uint32_t D1,
                          uint64_t* grp_off, uint32_t* grp_ptr32, hipStream_t s) {
  hipLaunchKernelGGL(k_grp_off, dim3((N + 1 + kB - 1) / kB), dim3(kB), 0, s, cnt, off, grp_ptr64, N, D1, grp_off,
                     grp_ptr32);
  return hipGetLastError();
}

size_t segsort_list(uint64_t n_syn, uint64_t n_groups) {
  return (size_t)std::min<uint64_t>(n_groups, n_syn / (kWaveSortMax + 1)) + 1;
}

bool row_sort_fits(const BinBuild& bb, uint32_t D1, uint32_t longest, uint64_t mean) {
  return bb.nbin && bb.words / D1 <= (uint32_t)kBT && longest <= 1024u * kRowSortRegs && mean >= kRowSortMean;
}

hipError_t launch_bin_rows(const BinBuild& bb, uint32_t D1, const uint64_t* off, uint32_t* payload, uint8_t* del,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_bin_rows, dim3(bb.nbin), dim3(kBT), kRowChunk * 7 + kBT * 12, s, bb, D1, off, payload, del);
  return hipGetLastError();
}

hipError_t launch_segsort(const uint64_t* grp_off, uint64_t n_groups, uint32_t* payload, uint64_t* longer,
                          uint32_t* n_longer, uint64_t list_cap, uint64_t* big, uint32_t* nbig, uint32_t big_cap,
                          const RowSort& rows, hipStream_t s) {
  if (n_groups == 0) return hipSuccess;
  if (rows.del) {
    uint32_t above = 0;  // a launch for each block size, over the rows that need it
    for (uint32_t th = 256; th <= 1024 && rows.longest > above; th *= 2) {
      auto k = th == 256 ? k_row_sort<256> : th == 512 ? k_row_sort<512> : k_row_sort<1024>;
      hipLaunchKernelGGL(k, dim3(rows.N), dim3(th), 0, s, rows.off, rows.grp_ptr, rows.D1, rows.del, payload, above,
                         (unsigned long long*)longer, n_longer, list_cap);
      above = th * kRowSortRegs;
    }
  } else {
    hipLaunchKernelGGL(k_segsort_wave, dim3(grid_for(n_groups, kB / 64, 1u << 20)), dim3(kB), 0, s, grp_off, n_groups,
                       payload, (unsigned long long*)longer, n_longer, list_cap);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_segsort_block, dim3(grid_for(list_cap, 1, 1024)), dim3(kSB), kBlockSortMax * sizeof(uint32_t), s,
                     grp_off, (const unsigned long long*)longer, n_longer, payload, (unsigned long long*)big, nbig,
                     big_cap);
  return hipGetLastError();
}

hipError_t launch_bin_gen(const ProjDev* projs, uint32_t nproj, uint64_t total_pairs, uint32_t dmax_cfg,
                          const uint16_t* cls_of, const ProjW* pw, const uint32_t* pop_first, uint32_t npop,
                          uint32_t cls_bits, const BinBuild& bb, hipStream_t s) {
  const uint64_t blocks = (total_pairs + (uint64_t)kBT * kBinItems - 1) / ((uint64_t)kBT * kBinItems);
  hipLaunchKernelGGL(k_bin_gen, dim3((uint32_t)blocks), dim3(kBT), 2 * bb.nbin * sizeof(uint32_t), s, projs, nproj,
                     total_pairs, dmax_cfg, cls_of, pw, pop_first, npop, cls_bits, bb);
  return hipGetLastError();
}

hipError_t launch_bin_count(const BinBuild& bb, uint32_t D1, uint32_t* cnt, hipStream_t s) {
  hipLaunchKernelGGL(k_bin_count, dim3(bb.nbin), dim3(kBT), bb.words * sizeof(uint32_t), s, bb, D1, cnt);
  return hipGetLastError();
}

hipError_t launch_bin_place(const BinBuild& bb, uint32_t D1, const uint64_t* off, uint32_t* payload, hipStream_t s) {
  hipLaunchKernelGGL(k_bin_place, dim3(bb.nbin), dim3(kBT), bb.words * sizeof(uint32_t), s, bb, D1, off, payload);
  return hipGetLastError();
}

hipError_t launch_runs(bool fill, const uint64_t* grp_off, uint64_t n_groups, const uint32_t* payload,
                       uint32_t cls_bits, uint32_t tsh, uint32_t* cnt, const uint64_t* grp_run, uint32_t* run_desc,
                       uint32_t* too_long, hipStream_t s) {
  if (n_groups == 0) return hipSuccess;
  const dim3 grid(grid_for(n_groups, kB / 64, 1u << 16));
  if (fill)
    hipLaunchKernelGGL(k_runs<true>, grid, dim3(kB), 0, s, grp_off, n_groups, payload, cls_bits, tsh, cnt, grp_run,
                       run_desc, too_long);
  else
    hipLaunchKernelGGL(k_runs<false>, grid, dim3(kB), 0, s, grp_off, n_groups, payload, cls_bits, tsh, cnt, grp_run,
                       run_desc, too_long);
  return hipGetLastError();
}

}  // namespace snn
