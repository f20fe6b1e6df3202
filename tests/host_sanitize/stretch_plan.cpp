// The rules of the kernels that deal rows by columns (csrc/stretch.h), on the host.
#include <hip/hip_runtime.h>
#include <stdio.h>

#include <vector>

#include "../../paper_2411_08446_amd/csrc/stretch.h"

using namespace lshmoe;

static int failures = 0, checks = 0;

static void expect(bool ok, const char* what, long long T, int k, int more) {
  ++checks;
  if (!ok && ++failures <= 20) printf("FAIL %s T=%lld k=%d %d\n", what, T, k, more);
}

// Cluster numbers of T tokens with k experts each: alone, every assignment has a cluster of its own, and the assignments that
// `shared` names are all in a few clusters that come first.
template <typename F>
static std::vector<int32_t> mostly_alone(uint32_t T, uint32_t k, F shared) {
  std::vector<int32_t> seg(T * k);
  int32_t next = (int32_t)k;
  for (uint32_t t = 0; t < T; ++t)
    for (uint32_t j = 0; j < k; ++j) seg[t * k + j] = shared(t, j) ? (int32_t)j : next++;
  return seg;
}

// The estimate of the number of clusters: not misled by what the tokens at one place of every sequence have in common, nor by
// one of a token's experts.
static void check_estimate() {
  for (uint32_t T : {4096u, 8192u, 16384u, 24576u, 30000u, 32768u, 49152u, 65536u, 65536u + 512u, 131072u, 262144u, 1048576u}) {
    for (uint32_t k = 1; k <= kStretchExperts; ++k) {
      for (uint32_t seq : {64u, 128u, 512u, 1000u, 1024u, 2048u, 4096u}) {
        std::vector<int32_t> seg = mostly_alone(T, k, [&](uint32_t t, uint32_t) { return t % seq == 0; });
        expect(!large_clusters(seg.data(), T, k, 25), "sequences that begin alike", T, (int)k, (int)seq);
        seg = mostly_alone(T, k, [&](uint32_t t, uint32_t) { return t % seq < seq / 4; });
        expect(!large_clusters(seg.data(), T, k, 25), "a quarter of padding in front", T, (int)k, (int)seq);
        seg = mostly_alone(T, k, [&](uint32_t t, uint32_t) { return t % seq >= seq - seq / 4; });
        expect(!large_clusters(seg.data(), T, k, 25), "a quarter of padding behind", T, (int)k, (int)seq);
      }
      for (uint32_t one = 0; one < k && k > 1; ++one) {
        const std::vector<int32_t> seg = mostly_alone(T, k, [&](uint32_t, uint32_t j) { return j == one; });
        expect(!large_clusters(seg.data(), T, k, 25), "one expert of a token shared by all", T, (int)k, (int)one);
      }
      for (int percent : {1, 10, 90}) {                        // clusters drawn uniformly: estimated from below, by about a ninth
        std::vector<int32_t> seg((size_t)T * k);
        uint64_t x = 88172645463325252ull + T + k;
        for (int32_t& s : seg) {
          x ^= x << 13; x ^= x >> 7; x ^= x << 17;
          s = (int32_t)(x % ((uint64_t)T * k * percent / 100));
        }
        expect(large_clusters(seg.data(), T, k, 25) == (percent < 25), "uniform clusters", T, (int)k, percent);
      }
      for (uint32_t i = 0; i < 8; ++i) expect(sample_place(i, T, k) < T * k, "place", T, (int)k, (int)i);
    }
  }
  for (uint32_t T : {1u, 2u, 3u, (1u << 30) - 1})
    for (uint32_t i = 0; i < 8; ++i) expect(sample_place(i, T, 1) < T, "place", T, 1, (int)i);
}

int main() {
  check_estimate();
  printf("%d checks, %d failures\n", checks, failures);
  return failures ? 1 : 0;
}
