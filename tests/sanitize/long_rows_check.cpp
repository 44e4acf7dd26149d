// long_rows (host_build.cpp) against a plain stable sort, on degree sequences
// whose longest rows, ties and bounds vary; built under AddressSanitizer and
// UndefinedBehaviorSanitizer by tests/test_long_rows.py. Exits with status 0
// only if all agree.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <random>
#include <vector>

#include "host_build.h"

int main() {
  int failures = 0, runs = 0;
  std::mt19937 rng(7);
  const std::vector<std::vector<int32_t>> fixed = {
      {}, {0}, {5}, {32}, {33}, {33, 33, 33}, {32, 33, 32, 34}, {0, 0, 4097, 0, 256, 257}, {70000, 33, 70000, 1}};
  std::vector<std::vector<int32_t>> all = fixed;
  for (int top : {1, 31, 40, 300, 5000})
    for (int n : {1, 7, 64, 3000}) {
      std::vector<int32_t> d(n);
      for (auto& x : d) x = static_cast<int32_t>(rng() % (top + 1));
      all.push_back(d);
    }
  for (const auto& d : all) {
    const int64_t n = static_cast<int64_t>(d.size());
    std::vector<int32_t> rp(n + 1, 0);
    for (int64_t u = 0; u < n; ++u) rp[u + 1] = rp[u] + d[u];
    for (int32_t least : {0, 1, 31, 32, 256}) {
      std::vector<int32_t> want;
      for (int64_t u = 0; u < n; ++u)
        if (d[u] > least) want.push_back(static_cast<int32_t>(u));
      std::stable_sort(want.begin(), want.end(), [&](int32_t a, int32_t b) { return d[a] > d[b]; });
      ++runs;
      if (blest::long_rows(n, rp.data(), least) != want) {
        std::printf("%zu rows above %d differ\n", d.size(), least);
        ++failures;
      }
    }
  }
  std::printf("long_rows_check: %d runs, %d failures\n", runs, failures);
  return failures == 0 ? 0 : 1;
}
