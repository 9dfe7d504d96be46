// Batches of one case in a launch, on the CPU: the home workgroups of
// spread_workgroups (ctd_schedule.h) and the claims the kernel's waves make with
// them.  Reads "seed grid waves n_0 ... n_{k-1}" lines (chunks per batch) from
// stdin; for each, lets the waves claim in a random order and prints "ok" or the
// first violation: home waves that do not add up to the grid, a workgroup
// outside its home range, a share of the grid off by more than a workgroup from
// the batch's share of the chunks, a chunk that does not run exactly once.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <sstream>
#include <string>
#include <vector>

#include "ctd_schedule.h"

namespace {

uint32_t next_random(uint64_t &s) {
  s = s * 6364136223846793005ull + 1442695040888963407ull;
  return (uint32_t)(s >> 33);
}

// A wave claims chunks of a batch until one is past the end, then of the next
// batch with chunks left, cyclically.
struct Wave {
  int batch = 0;
  uint64_t rank = 0;   // its first chunk at home
  bool home = true, exited = false;
};

std::string play(uint64_t seed, int grid, int waves, const std::vector<uint64_t> &n) {
  const int k = (int)n.size();
  std::vector<uint64_t> begin((size_t)k), counter((size_t)k, 0);
  uint64_t total = 0;
  for (int i = 0; i < k; ++i) {
    begin[i] = total;
    total += n[i];
  }
  std::vector<uint32_t> lo((size_t)k), hw((size_t)k);
  ctd::spread_workgroups(begin.data(), k, total, grid, waves, lo.data(), hw.data());
  uint64_t sum = 0;
  for (int i = 0; i < k; ++i) {
    sum += hw[i];
    const double share = total ? (double)grid * (double)n[i] / (double)total : 0.0;
    if (total && std::fabs((double)hw[i] / waves - share) > 1.0) return "share of the grid";
  }
  if (sum != (uint64_t)grid * (uint64_t)waves) return "home waves do not add up to the grid";
  std::vector<Wave> wave((size_t)grid * (size_t)waves);
  for (int g = 0; g < grid; ++g) {
    int c = 0;
    for (int i = 0; i < k; ++i)
      if (lo[i] <= (uint32_t)g) c = i;
    if ((uint32_t)g < lo[c] || (uint32_t)g >= (c + 1 < k ? lo[c + 1] : (uint32_t)grid))
      return "workgroup outside its home range";
    for (int w = 0; w < waves; ++w) {
      Wave &v = wave[(size_t)g * waves + w];
      v.batch = c;
      v.rank = (uint64_t)((uint32_t)g - lo[c]) * waves + w;
    }
  }
  std::vector<uint64_t> runs(total, 0);
  for (size_t live = wave.size(); live > 0;) {
    Wave &v = wave[next_random(seed) % wave.size()];
    if (v.exited) continue;
    const int c = v.batch;
    const uint64_t t = v.home ? v.rank : hw[c] + counter[c]++;
    v.home = false;
    if (t < n[c]) {
      runs[begin[c] + t] += 1;
      continue;
    }
    int nxt = -1;
    for (int i = 1; i <= k && nxt < 0; ++i)
      if (hw[(c + i) % k] + counter[(c + i) % k] < n[(c + i) % k]) nxt = (c + i) % k;
    if (nxt < 0) {
      v.exited = true;
      --live;
    }
    v.batch = nxt;
  }
  for (uint64_t r : runs)
    if (r != 1) return "a chunk ran " + std::to_string(r) + " times";
  return "ok";
}

}  // namespace

int main() {
  char line[1 << 16];
  while (std::fgets(line, sizeof line, stdin)) {
    std::istringstream in(line);
    uint64_t seed, x;
    int grid, waves;
    if (!(in >> seed >> grid >> waves)) continue;
    std::vector<uint64_t> n;
    while (in >> x) n.push_back(x);
    std::printf("%s\n", play(seed, grid, waves, n).c_str());
  }
  return 0;
}
