// bin_plan.h -- how the sources of a large network are cut into the bins that
// its synapses are drawn into (kernels_build.hip).  Host arithmetic only.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <map>
#include <vector>

namespace snn {

constexpr uint32_t kBinBuildMax = 4096;    // bins, at most
constexpr uint32_t kBinBuildWords = 24576; // (source, delay) counters of a bin, at most

struct BinPlan {
  std::vector<uint32_t> first, cap;  // bin b: sources [first[b], first[b + 1]), room for cap[b] synapses
  std::vector<uint64_t> off;         // ... from place off[b] on
  std::vector<uint16_t> of;          // bin of each source
  uint64_t places = 0;
};

// Bins of consecutive sources with about equal numbers of synapses, each with
// room for eight standard deviations more than are expected in it.  step: the
// changes of the expected synapses per source along the N gids; D1 counters a
// source.  False where more bins than kBinBuildMax would be needed.
inline bool plan_source_bins(uint32_t N, uint64_t total_syn, uint32_t D1, const std::map<uint32_t, double>& step,
                             BinPlan& p) {
  const uint32_t most = kBinBuildWords / D1;  // sources of a bin, at most
  const double want = std::max((double)total_syn / 1000.0, 8192.0);
  p = BinPlan();
  p.first.push_back(0);
  p.of.resize(N);
  double rate = 0.0, in_bin = 0.0;
  auto close = [&](uint32_t end) {
    const uint64_t c = (uint64_t)(in_bin + 8.0 * std::sqrt(in_bin) + 256.0);
    p.off.push_back(p.places);
    p.cap.push_back((uint32_t)std::min<uint64_t>(c, 0x7fffffffu));
    p.places += c;
    p.first.push_back(end);
    in_bin = 0.0;
  };
  auto next = step.begin();
  for (uint32_t i = 0; i < N; ++i) {
    // the changes need not cancel exactly: never below none
    while (next != step.end() && next->first <= i) { rate = std::max(0.0, rate + next->second); ++next; }
    if (i > p.first.back() && (i - p.first.back() >= most || in_bin + 0.5 * rate > want)) close(i);
    if (p.cap.size() >= kBinBuildMax) return false;
    p.of[i] = (uint16_t)p.cap.size();
    in_bin += rate;
  }
  close(N);
  return true;
}

}  // namespace snn
