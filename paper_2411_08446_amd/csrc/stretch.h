// Rows of clusters that every token reads, from an L2 instead of through it.  A cluster's members are spread over the tokens
// and so over the XCDs: a row of it crosses each of the eight L2s about once per member, and 7.1 TB/s of such traffic is what
// bounds the kernels that walk the tokens in their order.  Dealt by columns instead, an XCD takes one 256-byte stretch of
// the rows of all tokens at a time (workgroups go to the XCDs in turn, in the order of their numbers; if they did not, only
// time would be lost) and meets all members of a cluster: what is in use of the cluster rows at one time is 512 bytes per
// cluster.  65536 x 1024 bf16, two experts, 6.5 members per cluster: restore + combine 104 -> 81.5 us, token gradient 123 ->
// 104.5.  Stretches of 128 bytes make more lookups (95, 124 us), in stretches of 512 fewer members meet (87, 106).
#pragma once
#include "common.h"

namespace lshmoe {

__host__ __device__ inline uint64_t at_most(uint64_t a, uint64_t b) { return a < b ? a : b; }

constexpr uint32_t kXcdCount = 8;
constexpr uint32_t kStretchPieces = 16;    // 16-byte pieces of a stretch: a lane each
constexpr uint32_t kStretchTokens = 512 / kStretchPieces;   // tokens of a round of a workgroup of 256 threads, two per lane group
constexpr uint32_t kStretchExperts = 4;    // experts per token at most: the lookups of a round are kept in LDS

struct StretchPlan {
  uint32_t stretches;             // of a row; 0: the rows are not dealt by columns
  uint32_t parts, part_tokens;    // parts of the tokens, so that stretches x parts is a multiple of the XCDs; tokens of one
  uint32_t tokens, chunks;        // tokens of a workgroup; workgroups per stretch and part
  uint32_t low, high;             // it pays for low to high - 1 clusters
  uint64_t workgroups() const { return (uint64_t)stretches * parts * chunks; }
};

// Rows that split into eight stretches, or into four for each half of the tokens (with more parts a cluster's members are
// spread again).  A workgroup takes as many tokens as keep the grid to that of one wave per token.
inline StretchPlan plan_stretches(int64_t T, int k, uint32_t cpr, uint64_t low, uint64_t high) {
  StretchPlan p{};
  if (cpr % (4 * kStretchPieces) != 0 || k > (int)kStretchExperts || low >= high) return p;
  p.stretches = cpr / kStretchPieces;
  p.parts = p.stretches % kXcdCount == 0 ? 1 : 2;
  p.part_tokens = (uint32_t)((T + p.parts - 1) / p.parts);
  p.tokens = kStretchTokens * ((cpr + 127) / 128);
  p.chunks = (p.part_tokens + p.tokens - 1) / p.tokens;
  p.low = (uint32_t)low;
  p.high = (uint32_t)high;
  return p;
}

// Where it pays, for restore + combine and for the token gradient: rows of 1, 2, 3, 4 and 8 KB, 8 MB to 1 GB of them, one,
// two and four experts, 0.05 to 0.24 clusters per assignment were measured against the way round (us: way round -> columns).
//  * Two arrays of cluster rows that fit an XCD's L2 as they are need no columns.  Restore + combine, 32768 x 512 bf16, one
//    expert, 3.3 MB of them 15.8 -> 16.6; 65536, 6.7 MB 34.6 -> 31.2.  The token gradient, which has the rows of k experts pass
//    through the L2 as well, needs twice that: 16384 x 1024, two experts, 6.7 MB 25.9 -> 27.2; 32768, 13 MB 56.8 -> 51.2.
constexpr uint64_t kXcdL2 = 4ull << 20;
//  * 512 bytes of a cluster are in use at a time, and with too many of them the L2 does not hold what comes back.  Restore +
//    combine, N x 1024, two experts: 26 thousand clusters 110 -> 95, 31 217 -> 192, 63 431 -> 411, 105 438 -> 446, 126 889 -> 917.
//    Rows that are not eight or twelve stretches bear half of that: 131072 x 512, 31 thousand 107.5 -> 106.1, 52 109.4 ->
//    111.5; 131072 x 2048, 31 433 -> 391, 52 445 -> 453; and of four with one expert a quarter: 131072 x 512, 16 76.3 -> 75.4,
//    26 76.9 -> 78.5.
//  * To ask costs 0.4 us of a call that then goes the way round, and more where a wave has little else to do: restore + combine,
//    0.4 clusters per assignment, 65536 x 1024, two experts 107.8 -> 107.9; 16384 x 512, one expert 10.0 -> 10.7, 131072 of them
//    75.4 -> 77.9, 524288 x 256 binary32 306 -> 316.  So it is asked only where the bound on the clusters leaves a tenth of the
//    assignments, with rows of 1 KB the whole share for which columns pay.
inline uint64_t fewer_clusters_than(uint64_t N, int k, uint32_t cpr, uint64_t percent) {
  const bool narrow = cpr == 4 * kStretchPieces, eight_or_twelve = cpr == 8 * kStretchPieces || cpr == 12 * kStretchPieces;
  const uint64_t most = eight_or_twelve ? 65536 : narrow && k == 1 ? 16384 : 32768;
  if (most * 100 < N * (narrow ? percent : 10)) return 0;
  return at_most(N * percent / 100, most);
}

// Restore + combine: from rows of 8 MB in all on.  Measured with 10, 20, 30, 40 per cent of clusters per assignment, us: 4096 x
// 1024 bf16, two experts 8.8 -> 6.5, 9.0 -> 6.3, 9.0 -> 6.7, 9.1 -> 7.1; 32768 of them 53.6 -> 39.9, 56.1 -> 44.8, 57.0 -> 47.6,
// 56.9 -> 50.6; 65536 109 -> 84, 112 -> 99, 111 -> 107, 111 -> 110; one expert 75.6 -> 59.3 .. 76.3 -> 71.1.  Rows of binary32
// are twice as wide for the same L2: 32768 x 1024, two experts 110 -> 82, 114 -> 103, 114 -> 114, 114 -> 119.  One expert and rows
// of 4 KB and more lose (a row takes two turns of the XCDs): 8192, 32768, 65536 x 2048, 0.05: 15.6 -> 17.9, 67 -> 72, 142 -> 142;
// and so do rows of 1 KB of binary32, for which there is less to gain: 65536 x 256, 0.05 to 0.2: 1.04, 0.99, 0.96 times as fast.
inline StretchPlan plan_combine(int64_t T, int k, uint32_t cpr, bool bf16) {
  const uint64_t row = cpr * 16ull, N = (uint64_t)T * k;
  if (T * row < 8ull << 20) return StretchPlan{};
  if (k == 1 && (cpr > 12 * kStretchPieces || (!bf16 && cpr < 8 * kStretchPieces))) return StretchPlan{};
  return plan_stretches(T, k, cpr, kXcdL2 / (2 * row), fewer_clusters_than(N, k, cpr, bf16 ? 25 : 15));
}

// Restore knows the number of clusters and has another way round: in cluster order it reads a cluster's rows once and a token's
// once per expert, by columns the other way about, and writes the output in pieces of 256 bytes to all rows.  Measured as whole
// steps, rows of 1 to 4 KB, 4 to 512 MB of output, two to four experts, 0.03 to 0.15 clusters per assignment (us: cluster
// order -> columns).  It pays where each XCD has one stretch of all tokens: 128 MB of 2 KB rows, two experts, 0.05, 0.07, 0.09,
// 0.10, 0.14 clusters 115 -> 108, 111 -> 107, 112 -> 109, 112 -> 110, 106 -> 107.  Rows of 3 and 4 KB, 0.03 and 0.09, 137 -> 139,
// 114 -> 122 and 153 -> 152, 118 -> 125.  Rows of 1 KB, 0.05 and 0.09, 111 -> 106, 112 -> 110, but the call by itself, with its
// inputs in the last-level cache, 50 -> 50, 51 -> 53 (2 KB 49 -> 46, 49 -> 47) and with 256 MB 97 -> 108.  And it pays while the
// output stays in the last-level cache of 256 MB, up to more clusters if it takes no more than half of it: 0.14, 24, 48, 64, 96,
// 128 MB 44.0 -> 43.5, 58.3 -> 58.1, 65.9 -> 65.8, 87.3 -> 87.4, 108.3 -> 106.2 (10 hash functions 116.9 -> 115.4), with 0.2 three
// microseconds more; 256 MB, 0.05, 0.07, 0.09, 0.11 196 -> 177, 197 -> 185, 191 -> 185, 190 -> 190; 512 MB 360 -> 359, 359 -> 371,
// 358 -> 381.  From 24 MB on: 24 MB, 0.03 and 0.09, 72.4 -> 70.5, 49.6 -> 48.6; 16 MB, 0.06 and 0.08, 55.3 -> 54.8, 45.4 -> 45.9.
inline StretchPlan plan_restore(int64_t N, int k, uint32_t cpr) {
  const uint64_t bytes = (uint64_t)N * cpr * 16;
  if (k == 1 || cpr != kXcdCount * kStretchPieces || bytes < 24ull << 20 || bytes > 256ull << 20) return StretchPlan{};
  return plan_stretches(N / k, k, cpr, 0, (uint64_t)N * (bytes <= 128ull << 20 ? 15 : 9) / 100);
}

// Token gradient: from 64 MB of gradient rows on, of binary32 from 128 MB and two experts.  Measured with 10, 20, 30 per cent of
// clusters per assignment, us: 16384 x 1024 bf16, two experts 30.8 -> 28.7, 33.1 -> 29.3, 33.7 -> 29.8; 65536 of them 128 -> 107,
// 131 -> 119, 130 -> 126; one expert 71.4 -> 65.5, 73.6 -> 67.7, 73.4 -> 69.6; 8192, two experts 14.6 -> 15.4, 16.4 -> 15.8; binary32
// 32768 x 1024, two experts 128 -> 110, 130 -> 122, 130 -> 134; one 71.1 -> 73.9; 8192, two 29.5 -> 30.8.  Rows of 4 KB and more
// lose (16384 x 2048, two experts, 0.05, 0.12, 0.2: 52 -> 64, 59 -> 65, 63 -> 66) but for very many of them (131072: 506 -> 468, 514
// -> 492, 517 -> 552), and so do rows of 1 KB with one expert (131072 x 512, the same: 70 -> 74, 74 -> 77, 76 -> 80).
inline StretchPlan plan_grad_tokens(int64_t T, int k, uint32_t cpr, bool bf16) {
  const uint64_t row = cpr * 16ull, N = (uint64_t)T * k;
  if (N * row < (bf16 ? 64ull : 128ull) << 20 || cpr > 12 * kStretchPieces) return StretchPlan{};
  if (k == 1 && (!bf16 || cpr < 8 * kStretchPieces)) return StretchPlan{};
  return plan_stretches(T, k, cpr, 2 * kXcdL2 / (2 * row), fewer_clusters_than(N, k, cpr, bf16 ? 25 : 20));
}

// What a workgroup does: the stretch `at` bytes from a row's start of tokens first .. end - 1 (none, if first >= end).
struct StretchDuty {
  uint32_t at, first, end;
};
__host__ __device__ inline StretchDuty stretch_duty(const StretchPlan& p, uint64_t block, uint32_t T) {
  const uint64_t r = block / kXcdCount, turn = r / p.chunks;
  if (turn >= p.stretches * p.parts / kXcdCount) return StretchDuty{0, 0, 0};
  const uint32_t unit = (uint32_t)turn * kXcdCount + (uint32_t)(block % kXcdCount);
  const uint32_t part = unit % p.parts * p.part_tokens;
  StretchDuty d;
  d.at = unit / p.parts * kStretchPieces * 16;
  d.first = part + (uint32_t)(r % p.chunks) * p.tokens;
  d.end = (uint32_t)at_most(at_most(part + p.part_tokens, T), d.first + p.tokens);
  return d;
}

// Assignment number i of the eight that the number of clusters is estimated from.  Tokens at irregular fractions of T (multiples
// of the golden section): at even steps all eight were the first token of a sequence in a batch of 2^m sequences of equal
// length, which is one vector for all of them in a causal model, and so one cluster.  The experts take turns: a token's first
// one may be of a few for all tokens.  65536 x 1024 bf16, two experts, sequences of 512 that begin alike, 0.9 clusters per
// assignment, restore + combine and token gradient, us: even steps 90.8, 92.7; these 74.9, 73.9; without columns 74.2, 73.6.
__host__ __device__ inline uint32_t sample_place(uint32_t i, uint32_t T, uint32_t k) {
  return (uint32_t)(((uint64_t)T * (uint32_t)((i + 1) * 0x9e3779b9u)) >> 32) * k + (i * k >> 3);
}

// An estimate of the number of clusters that is the same in every workgroup: the largest of eight cluster numbers.  Scalar
// loads of eight fixed places, beside the loads of the way round: 0.4 us of 82; sixteen places by vector loads had cost 14 us.
__host__ __device__ inline uint32_t estimate_clusters(const int32_t* __restrict__ seg_of, uint32_t T, uint32_t k) {
  int32_t most = 0;
#pragma unroll
  for (uint32_t i = 0; i < 8; ++i) {
    const int32_t s = seg_of[sample_place(i, T, k)];
    most = s > most ? s : most;
  }
  return (uint32_t)most;
}

// Whether to go by columns for this number of clusters (none, if the rows are not dealt so at all: low == high == 0).
__host__ __device__ inline bool pays(const StretchPlan& p, uint32_t clusters) { return clusters - p.low < p.high - p.low; }

}  // namespace lshmoe
