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

// Whether a number of clusters is more than a quarter of the assignments.
static bool small(uint32_t clusters, uint32_t T, uint32_t k) { return (uint64_t)clusters * 4 > (uint64_t)T * k; }

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
        expect(small(estimate_clusters(seg.data(), T, k), T, k), "sequences that begin alike", T, (int)k, (int)seq);
        seg = mostly_alone(T, k, [&](uint32_t t, uint32_t) { return t % seq < seq / 4; });
        expect(small(estimate_clusters(seg.data(), T, k), T, k), "a quarter of padding in front", T, (int)k, (int)seq);
        seg = mostly_alone(T, k, [&](uint32_t t, uint32_t) { return t % seq >= seq - seq / 4; });
        expect(small(estimate_clusters(seg.data(), T, k), T, k), "a quarter of padding behind", T, (int)k, (int)seq);
      }
      for (uint32_t one = 0; one < k && k > 1; ++one) {
        const std::vector<int32_t> seg = mostly_alone(T, k, [&](uint32_t, uint32_t j) { return j == one; });
        expect(small(estimate_clusters(seg.data(), T, k), T, k), "one expert of a token shared by all", T, (int)k, (int)one);
      }
      for (int percent : {1, 10, 90}) {                        // clusters drawn uniformly: estimated from below, by about a ninth
        std::vector<int32_t> seg((size_t)T * k);
        uint64_t x = 88172645463325252ull + T + k;
        for (int32_t& s : seg) {
          x ^= x << 13; x ^= x >> 7; x ^= x << 17;
          s = (int32_t)(x % ((uint64_t)T * k * percent / 100));
        }
        expect(small(estimate_clusters(seg.data(), T, k), T, k) == (percent > 25), "uniform clusters", T, (int)k, percent);
      }
      for (uint32_t i = 0; i < 8; ++i) expect(sample_place(i, T, k) < T * k, "place", T, (int)k, (int)i);
    }
  }
  for (uint32_t T : {1u, 2u, 3u, (1u << 30) - 1})
    for (uint32_t i = 0; i < 8; ++i) expect(sample_place(i, T, 1) < T, "place", T, 1, (int)i);
}

// Every stretch of every token is somebody's, once, for any grid that has enough workgroups.
static void check_duties() {
  for (uint32_t cpr : {64u, 128u, 192u, 256u, 320u, 512u}) {
    for (uint32_t T : {1u, 2u, 31u, 33u, 4096u, 8192u + 13u, 30001u}) {
      const StretchPlan p = plan_stretches(T, 2, cpr, 0, 1);
      std::vector<uint8_t> done((size_t)T * p.stretches);
      for (uint64_t block = 0; block < p.workgroups() + 5000; ++block) {
        const StretchDuty d = stretch_duty(p, block, T);
        for (uint32_t t = d.first; t < d.end; ++t)
          if (d.at % (kStretchPieces * 16) == 0 && d.at < cpr * 16 && t < T) ++done[(size_t)t * p.stretches + d.at / (kStretchPieces * 16)];
      }
      bool ok = p.stretches * kStretchPieces == cpr;
      for (uint8_t n : done) ok = ok && n == 1;
      expect(ok, "duties", T, 2, (int)cpr);
    }
  }
  const uint32_t T = (1u << 27) + 6;                           // a grid of many rows of workgroups
  const StretchPlan p = plan_stretches(T, 1, 64, 0, 1);
  uint64_t done = 0, last = 0;
  for (uint64_t block = 0; block < p.workgroups(); ++block) {
    const StretchDuty d = stretch_duty(p, block, T);
    if (d.first < d.end) { done += d.end - d.first; if (d.end > last) last = d.end; }
  }
  expect(done == (uint64_t)T * p.stretches && last == T, "duties", T, 1, 64);
}

// Which calls go by columns.
static void check_rules() {
  const auto share = [](uint64_t T, uint64_t k, uint64_t percent) { return (uint32_t)(T * k * percent / 100); };
  struct { uint32_t T; int k; uint32_t cpr; bool bf16; int percent; bool combine, gradient; } cases[] = {
      {65536, 2, 128, true, 16, true, true},       // 2 KB rows, the method's rates
      {65536, 2, 128, true, 90, false, false},     // small clusters
      {32768, 2, 128, true, 1, false, false},      // cluster rows that an L2 holds
      {32768, 2, 128, true, 3, true, false},       // as they are; the token gradient passes more through it
      {32768, 1, 128, true, 12, true, true},
      {4096, 2, 128, true, 16, true, false},       // 16 MB of gradient rows
      {4095, 2, 128, true, 16, false, false},      // below 8 MB of tokens
      {262144, 2, 128, true, 10, true, true},
      {262144, 2, 128, true, 14, false, false},    // more clusters than an L2 has lines in use
      {65536, 2, 64, true, 20, true, true},        // 1 KB rows
      {65537, 2, 64, true, 20, false, false},
      {65536, 1, 64, true, 20, true, false},       // one expert
      {65537, 1, 64, true, 20, false, false},
      {32768, 1, 64, false, 13, false, false},
      {327680, 2, 128, true, 9, true, true},       // the bound on the clusters leaves a tenth
      {327681, 2, 128, true, 9, false, false},
      {32768, 2, 192, true, 16, true, true},
      {16384, 2, 256, true, 16, true, false},      // 4 KB rows
      {16384, 1, 256, true, 16, false, false},
      {16384, 4, 512, true, 16, true, false},
      {32768, 2, 256, false, 12, true, false},     // binary32
      {32768, 2, 256, false, 16, false, false},
      {65536, 2, 128, false, 14, true, true},
      {65536, 2, 128, false, 18, false, true},
      {65536, 1, 128, false, 14, true, false},
      {65536, 5, 128, true, 10, false, false},     // more experts than the lookups have room for
      {65536, 2, 96, true, 16, false, false},      // rows of six stretches
      // the shapes of tests/test_gpu_stretch.py: restore + combine
      {8192 + 13, 1, 64, true, 20, false, false}, {16384 + 13, 1, 64, true, 14, true, false}, {4096, 2, 128, true, 14, true, false},
      {8192 + 1, 3, 128, true, 10, true, false}, {4096 + 31, 2, 192, true, 10, true, false}, {4096 + 33, 4, 256, true, 10, true, false},
      {8192 + 7, 2, 64, false, 14, true, false}, {4096 + 65, 1, 256, false, 10, false, false}, {4096 + 65, 2, 256, false, 10, true, false},
      {4096 + 5, 5, 128, true, 10, false, false}, {8192 + 3, 2, 96, true, 10, false, false},
      // token gradient
      {32768 + 13, 2, 64, true, 12, true, true}, {32768 + 1, 1, 128, true, 12, true, true}, {16384 + 31, 2, 128, true, 12, true, true},
      {8192 + 7, 3, 192, true, 12, true, true}, {16384 + 33, 2, 256, false, 12, true, false}, {4096 + 5, 4, 256, true, 12, true, false},
      {8192 + 3, 5, 128, true, 12, false, false}, {32768 + 3, 1, 256, false, 12, false, false}, {32768 + 33, 2, 128, false, 12, true, true},
  };
  int i = 0;
  for (const auto& c : cases) {
    const uint32_t S = share(c.T, c.k, c.percent);
    expect(pays(plan_combine(c.T, c.k, c.cpr, c.bf16), S) == c.combine, "restore + combine", c.T, c.k, i);
    expect(pays(plan_grad_tokens(c.T, c.k, c.cpr, c.bf16), S) == c.gradient, "token gradient", c.T, c.k, i);
    ++i;
  }
  struct { uint32_t T; int k; uint32_t cpr; int percent; bool restore; } restores[] = {
      {32768, 2, 128, 14, true},     // 128 MB of output
      {32768, 2, 128, 15, false},
      {32768, 1, 128, 8, false},     // one expert
      {32768, 5, 128, 8, false},
      {16384, 2, 192, 8, false},     // rows wider than the XCDs take at once
      {32768 + 1, 2, 128, 9, false},
      {65536, 2, 128, 8, true},      // 256 MB
      {65536 + 1, 2, 128, 8, false},
      {6144, 2, 128, 8, true},       // 24 MB
      {6144 - 1, 2, 128, 8, false},
      {8192, 3, 128, 8, true},
      {43690, 3, 64, 8, false},      // rows that two groups of XCDs share
      // the shapes of tests/test_gpu_stretch.py
      {16384, 2, 128, 6, true}, {16384 + 13, 3, 128, 6, true}, {8192 + 1, 4, 128, 6, true}, {12288 + 5, 2, 64, 6, false},
      {16384, 2, 128, 10, true}, {65536 + 1, 2, 128, 6, false}, {6144 + 5, 2, 128, 6, true}, {6144 - 1, 2, 128, 6, false}, {8192 + 3, 2, 192, 6, false},
  };
  for (const auto& c : restores)
    expect(pays(plan_restore((int64_t)c.T * c.k, c.k, c.cpr), share(c.T, c.k, c.percent)) == c.restore, "restore", c.T, c.k, (int)c.cpr);
}

int main() {
  check_estimate();
  check_duties();
  check_rules();
  printf("%d checks, %d failures\n", checks, failures);
  return failures ? 1 : 0;
}
