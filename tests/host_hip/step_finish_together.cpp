// k_step_finish of several populations of one system at the same time: each workgroup sees the
// counters as they were before any of them, a plain store of a later one covers an earlier one's,
// atomic additions add up.  Prints the five counters.
#include "common.hpp"
#include "k_step_finish.inc"

#include <cstdio>

int main() {
  std::vector<std::pair<unsigned long long*, unsigned long long>> adds;
  host_hip::deferred = &adds;
  unsigned long long counts[CAP_COUNT] = {100, 200, 300, 400, 500}, before[CAP_COUNT], after[CAP_COUNT];
  for (int i = 0; i < CAP_COUNT; ++i) before[i] = after[i] = counts[i];
  const int sizes[3] = {5, 300, 64};
  for (int k = 0; k < 3; ++k) {
    const int nw = sizes[k], threads = nw > 256 ? 1024 : 256;
    std::vector<double> weight(nw, 1.0), wold(nw, 1.0);
    std::vector<cd> e(nw, cd{-1.0, 0.0});
    std::vector<unsigned> stat(nw, 0u);
    stat[0] = 0x4u;            // one capped energy
    stat[1] = stat[2] = 0x8u;  // two capped weights
    wold[nw - 1] = 0.0;        // one walker lost before the step
    double g[GR_COUNT] = {};
    unsigned status = 0;
    int64_t dstep = 7;
    for (int i = 0; i < CAP_COUNT; ++i) counts[i] = before[i];
    host_hip::run_block(0, threads, threads / 64, [] {}, [&] {
      k_step_finish(nw, 0, 0, 0.01, weight.data(), e.data(), wold.data(), stat.data(), g, &status,
                    counts, &dstep, 1, 8);
    });
    for (int i = 0; i < CAP_COUNT; ++i)
      if (counts[i] != before[i]) after[i] = counts[i];
    if (status != 0xcu || dstep != 8) return 1;
  }
  for (auto& a : adds) after[a.first - counts] += a.second;
  for (int i = 0; i < CAP_COUNT; ++i) printf("%llu ", after[i]);
  return 0;
}
