"""The bins of sources that a large network is drawn into (csrc/bin_plan.h),
compiled for the host: every bin's room covers its share, and the places are no
more than the synapses and the bins' margins, also where populations with
different out-degrees precede neurons without synapses of their own (their
expected number is a difference of sums that do not cancel exactly)."""
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DRIVER = r"""
#include <cstdio>
#include "bin_plan.h"
// stdin, a plan a line: D1, then n (sources of a population) and s (synapses of it), pairs up to 0 0
int main() {
  unsigned D1, n;
  double s;
  while (scanf("%u", &D1) == 1) {
    std::map<uint32_t, double> step;
    uint32_t N = 0;
    double total = 0;
    while (scanf("%u %lf", &n, &s) == 2 && n) {
      step[N] += s / n;
      step[N + n] -= s / n;
      N += n;
      total += s;
    }
    snn::BinPlan p;
    const bool ok = snn::plan_source_bins(N, (uint64_t)total, D1, step, p);
    printf("%d %llu", ok, (unsigned long long)p.places);
    for (size_t b = 0; ok && b < p.cap.size(); ++b)
      printf(" %u %u %llu", p.first[b + 1], p.cap[b], (unsigned long long)p.off[b]);
    printf("\n");
  }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("bins")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2007_14236_amd", "csrc"),
                    str(d / "driver.cpp"), "-o", str(d / "driver")], check=True)

    def run(cases):
        text = "\n".join(f"{D1} " + " ".join(f"{n} {s}" for n, s in pops) + " 0 0" for D1, pops in cases)
        out = subprocess.run([str(d / "driver")], input=text, capture_output=True, text=True, check=True).stdout
        return [[int(x) for x in line.split()] for line in out.splitlines()]

    return run


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
@pytest.mark.parametrize("D1", [2, 26, 64])
def test_rooms_and_places(plan, D1):
    r = random.Random(D1)
    cases = [(D1, [(r.randint(1, 4000), r.randint(1, 1 << 22)) for _ in range(k)] + [(r.randint(1, 30000), 0)])
             for k in (1, 2, 2, 2, 3, 5) * 100]
    for (_, pops), (ok, places, *bins) in zip(cases, plan(cases)):
        if not ok:
            continue
        total, nbin, N = sum(s for _, s in pops), len(bins) // 3, sum(n for n, _ in pops)
        # room of all bins: x + 8 sqrt(x) + 256 of each bin's x, the square roots by Cauchy's inequality
        assert total <= places <= total + 8 * (total * nbin) ** 0.5 + 257 * nbin, pops
        first, at = 0, 0
        share = [s / n for n, s in pops for _ in range(n)]
        for end, cap, off in zip(bins[::3], bins[1::3], bins[2::3]):
            assert first < end <= N and off == at
            assert cap >= sum(share[first:end]) * (1 - 1e-9) + 255, pops
            first, at = end, at + cap
        assert first == N and at == places
