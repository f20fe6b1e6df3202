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

constexpr uint32_t kXcdCount = 8;
constexpr uint32_t kStretchPieces = 16;    // 16-byte pieces of a stretch: a lane each
constexpr uint32_t kStretchTokens = 512 / kStretchPieces;   // tokens of a round of a workgroup of 256 threads, two per lane group
constexpr uint32_t kStretchExperts = 4;    // experts per token at most: the lookups of a round are kept in LDS

struct StretchPlan {
  uint32_t stretches;             // of a row; 0: the rows are not dealt by columns
  uint32_t parts, part_tokens;    // parts of the tokens, so that stretches x parts is a multiple of the XCDs; tokens of one
  uint32_t tokens, chunks;        // tokens of a workgroup; workgroups per stretch and part
  uint32_t percent;               // clusters per assignment below which it pays
  uint64_t workgroups() const { return (uint64_t)stretches * parts * chunks; }
};

// Rows that split into eight stretches, or into four for each half of the tokens (with more parts a cluster's members are
// spread again).  A workgroup takes as many tokens as keep the grid to that of one wave per token.
inline StretchPlan plan_stretches(int64_t T, int k, uint32_t cpr, uint32_t percent) {
  StretchPlan p{};
  if (cpr % (4 * kStretchPieces) != 0 || k > (int)kStretchExperts) return p;
  p.stretches = cpr / kStretchPieces;
  p.parts = p.stretches % kXcdCount == 0 ? 1 : 2;
  p.part_tokens = (uint32_t)((T + p.parts - 1) / p.parts);
  p.tokens = kStretchTokens * ((cpr + 127) / 128);
  p.chunks = (p.part_tokens + p.tokens - 1) / p.tokens;
  p.percent = percent;
  return p;
}

// What a workgroup does: the stretch `at` bytes from a row's start of tokens first .. end - 1 (none, if first >= end).
struct StretchDuty {
  uint32_t at, first, end;
};
__device__ __forceinline__ StretchDuty stretch_duty(const StretchPlan& p, uint64_t block, uint32_t T) {
  const uint64_t r = block / kXcdCount, turn = r / p.chunks;
  if (turn >= p.stretches * p.parts / kXcdCount) return StretchDuty{0, 0, 0};
  const uint32_t unit = (uint32_t)turn * kXcdCount + (uint32_t)(block % kXcdCount);
  const uint32_t part = unit % p.parts * p.part_tokens;
  StretchDuty d;
  d.at = unit / p.parts * kStretchPieces * 16;
  d.first = part + (uint32_t)(r % p.chunks) * p.tokens;
  d.end = min(min(part + p.part_tokens, T), d.first + p.tokens);
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

// Whether clusters are large enough for it, from an estimate of their number that is the same in every workgroup: the
// largest of eight cluster numbers.  Scalar loads of eight fixed places, beside the loads of the way round: 0.4 us of 82;
// sixteen places by vector loads had cost 14 us.
__host__ __device__ inline bool large_clusters(const int32_t* __restrict__ seg_of, uint32_t T, uint32_t k, uint32_t percent) {
  int32_t most = 0;
#pragma unroll
  for (uint32_t i = 0; i < 8; ++i) {
    const int32_t s = seg_of[sample_place(i, T, k)];
    most = s > most ? s : most;
  }
  return (uint64_t)(uint32_t)most * 100 < (uint64_t)T * k * percent;
}

}  // namespace lshmoe
