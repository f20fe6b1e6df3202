// Grouping of assignments by (expert, bucket) (Alg. 1: dispatch, then split
// each expert's tokens into clusters by bucket id).
//
// A stable sort of the packed key (expert << bbits | bucket) carrying the
// assignment index, then the numbering of the runs of equal keys.  Integer
// work only; every result is deterministic.  The arrays are a few MB at most,
// so the step is bound by launches and by dependent trips to memory, not by
// HBM: the design goal is few of both.  Three routes by size:
//
//  - up to kSmallMaxN assignments: everything in one workgroup and one launch
//    (bin_group_kernel on a single bin).
//  - up to kMaxTiles tiles of 2048 (every paper-shaped layer): two launches.
//    tile_bin_kernel sorts every tile of the input by the top 8 key bits and
//    leaves it in place, with a table of where its 256 bins start;
//    bin_group_kernel gives every bin one workgroup of 16 waves, which collects
//    the bin's keys from all tiles, sorts them in LDS, numbers their clusters
//    and writes every output.
//  - larger: least-significant-digit radix passes of histogram,
//    single-workgroup scan of the (bin, tile) table and scatter, then a
//    counting and a numbering launch.
//
// Ranks inside a group of 64 keys come from wave ballots: for every lane the
// lanes holding the same digit; group order equals element order, which keeps
// the sorts stable.
#include <atomic>

#include "kernels.h"

namespace lshmoe {

namespace {

constexpr int kSortThreads = 256;
// A radix tile of the large route holds kSortTile keys: 8 per thread, 32 wave-sized groups whose per-bin counts form
// a row of 33 words (padded against bank conflicts) in LDS.
constexpr int kSegThreads = 256;
constexpr int kSegItems = kSegTile / kSegThreads;     // 4

struct KeySource {
  // pass 0 builds keys from the inputs; later passes read the ping-pong buffers
  const int32_t* expert;
  const uint64_t* bucket;
  const uint64_t* key;
  const int32_t* idx;
  uint32_t k, E;
  int bbits;
};

template <bool FIRST>
__device__ __forceinline__ void load_item(const KeySource& src, uint32_t i, uint64_t& key, int32_t& idx) {
  if (FIRST) {
    uint32_t e = (uint32_t)src.expert[i];
    if (e >= src.E) e = src.E - 1;  // out-of-range ids violate the contract; stay in bounds
    // bbits <= 63; ids with bits above bbits violate the contract too and must not reach the expert field
    key = ((uint64_t)e << src.bbits) | (src.bucket[i / src.k] & ((1ull << src.bbits) - 1ull));
    idx = (int32_t)i;
  } else {
    key = src.key[i];
    idx = src.idx[i];
  }
}

// Lanes of the wave whose `bits`-bit digit equals this lane's, among the lanes with `valid` (bits <= kMaxDigitBits,
// wave-uniform).
__device__ __forceinline__ uint64_t same_digit_lanes(uint32_t digit, int bits, bool valid) {
  uint64_t same = __ballot(valid);
#pragma unroll
  for (int b = 0; b < kMaxDigitBits; ++b) {
    if (b < bits) {
      const bool bit = (digit >> b) & 1u;
      const uint64_t bal = __ballot(bit);
      same &= bit ? bal : ~bal;
    }
  }
  return same;
}

// Exclusive scan of one value per thread across a 256-thread block.
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* wave_sum /*[4]*/, uint32_t& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t t = __shfl_up(inc, o, 64);
    if (lane >= o) inc += t;
  }
  if (lane == 63) wave_sum[wave] = inc;
  __syncthreads();
  uint32_t before = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < 256 / kWave; ++w) {
    if (w < wave) before += wave_sum[w];
    total += wave_sum[w];
  }
  __syncthreads();
  return before + inc - v;
}

// Tile histogram of one pass: column `tile` of a bin-major table (scanned next).
template <bool FIRST>
__global__ __launch_bounds__(kSortThreads) void sort_hist_kernel(KeySource src, uint32_t N, int shift, uint32_t mask,
                                                                 uint32_t nblk, uint32_t* __restrict__ table) {
  constexpr int kSortItems = kSortTile / kSortThreads;
  __shared__ uint32_t h[kGroupBins];
  h[threadIdx.x] = 0;
  h[threadIdx.x + 256] = 0;
  __syncthreads();
  const uint32_t base = blockIdx.x * kSortTile;
  uint64_t key[kSortItems];
  int32_t idx[kSortItems];
#pragma unroll
  for (int it = 0; it < kSortItems; ++it)
    load_item<FIRST>(src, min(base + it * kSortThreads + threadIdx.x, N - 1), key[it], idx[it]);
#pragma unroll
  for (int it = 0; it < kSortItems; ++it)
    if (base + it * kSortThreads + threadIdx.x < N) atomicAdd(&h[(uint32_t)(key[it] >> shift) & mask], 1u);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const uint32_t bin = threadIdx.x + 256 * j;
    if (bin <= mask) table[bin * nblk + blockIdx.x] = h[bin];  // bin-major: a scan over the table orders by (bin, tile)
  }
}

// In-place exclusive scan of n 32-bit counters by one workgroup of 1024
// threads: the array is walked in slabs of 4096 counters (one coalesced
// 16-byte load per thread), carrying the running total from slab to slab.
__global__ __launch_bounds__(1024) void scan_kernel(uint32_t* __restrict__ data, uint32_t n) {
  __shared__ uint32_t wave_sum[16];
  __shared__ uint32_t carry_s;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t carry = 0;
  for (uint32_t base = 0; base < n; base += 4096) {
    const uint32_t i = base + threadIdx.x * 4;
    uint32_t v[4] = {0, 0, 0, 0};
    if (i + 4 <= n) {
      const uint4 q = *reinterpret_cast<const uint4*>(data + i);
      v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
    } else {
      for (int j = 0; j < 4; ++j)
        if (i + j < n) v[j] = data[i + j];
    }
    const uint32_t sum = v[0] + v[1] + v[2] + v[3];
    uint32_t inc = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t t = __shfl_up(inc, o, 64);
      if (lane >= o) inc += t;
    }
    if (lane == 63) wave_sum[wave] = inc;
    __syncthreads();
    uint32_t run = carry + inc - sum;
#pragma unroll
    for (int w = 0; w < 16; ++w)
      if (w < wave) run += wave_sum[w];
    if (threadIdx.x == 1023) carry_s = run + sum;
    uint32_t o[4];
    o[0] = run; o[1] = o[0] + v[0]; o[2] = o[1] + v[1]; o[3] = o[2] + v[2];
    if (i + 4 <= n) {
      *reinterpret_cast<uint4*>(data + i) = make_uint4(o[0], o[1], o[2], o[3]);
    } else {
      for (int j = 0; j < 4; ++j)
        if (i + j < n) data[i + j] = o[j];
    }
    __syncthreads();
    carry = carry_s;
  }
}

template <bool FIRST>
__global__ __launch_bounds__(kSortThreads) void sort_scatter_kernel(KeySource src, uint32_t N, int shift, uint32_t mask,
                                                                    uint32_t nblk, const uint32_t* __restrict__ table,
                                                                    uint64_t* __restrict__ dst_key,
                                                                    int32_t* __restrict__ dst_idx) {
  constexpr int kSortItems = kSortTile / kSortThreads, kGroupsPerTile = kSortTile / kWave, kGhStride = kGroupsPerTile + 1;
  extern __shared__ uint32_t gh[];  // [kGroupBins][kGhStride] per-bin counts of each 64-key group, then start offsets
  const uint32_t base = blockIdx.x * kSortTile;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  uint64_t key[kSortItems];
  int32_t idx[kSortItems];
  uint32_t rank[kSortItems];
  // all of the tile's loads are issued before the first use (positions past N re-read the last key and are
  // masked out below), so the tile costs one memory round trip
#pragma unroll
  for (int it = 0; it < kSortItems; ++it)
    load_item<FIRST>(src, min(base + it * kSortThreads + threadIdx.x, N - 1), key[it], idx[it]);
  static_assert((kGroupBins * kGhStride) % 4 == 0, "gh is cleared 16 bytes at a time");
  for (int i = threadIdx.x; i < kGroupBins * kGhStride / 4; i += kSortThreads)  // while the loads fly
    reinterpret_cast<uint4*>(gh)[i] = make_uint4(0, 0, 0, 0);
  __syncthreads();
#pragma unroll
  for (int it = 0; it < kSortItems; ++it) {
    const bool valid = base + it * kSortThreads + threadIdx.x < N;
    const uint32_t digit = (uint32_t)(key[it] >> shift) & mask;
    const uint64_t same = same_digit_lanes(digit, kMaxDigitBits, valid);
    rank[it] = (uint32_t)__popcll(same & lt_mask);
    if (valid && rank[it] == 0) gh[digit * kGhStride + it * (kSortThreads / kWave) + wave] = (uint32_t)__popcll(same);
  }
  uint32_t start[2];  // first output position of each bin for this tile
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const uint32_t bin = threadIdx.x + 256 * j;
    start[j] = bin <= mask ? table[bin * nblk + blockIdx.x] : 0;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 2; ++j) {  // counts -> start offsets along the bin's row (independent reads, then register adds)
    uint32_t* row = gh + (threadIdx.x + 256 * j) * kGhStride;
    uint32_t c[kGroupsPerTile];
#pragma unroll
    for (int g = 0; g < kGroupsPerTile; ++g) c[g] = row[g];
    uint32_t run = start[j];
#pragma unroll
    for (int g = 0; g < kGroupsPerTile; ++g) {
      row[g] = run;
      run += c[g];
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < kSortItems; ++it) {
    const uint32_t i = base + it * kSortThreads + threadIdx.x;
    if (i < N) {
      const uint32_t digit = (uint32_t)(key[it] >> shift) & mask;
      const uint32_t pos = gh[digit * kGhStride + it * (kSortThreads / kWave) + wave] + rank[it];
      dst_key[pos] = key[it];
      dst_idx[pos] = idx[it];
    }
  }
}

// Head flags of kSegItems consecutive sorted positions starting at `base`: position p starts a cluster when
// its key differs from the key before it.  The keys are fetched up front (indices clamped into range).
__device__ __forceinline__ void load_heads(const uint64_t* __restrict__ key, uint32_t base, uint32_t N,
                                           uint64_t (&kv)[kSegItems + 1], bool (&head)[kSegItems]) {
#pragma unroll
  for (int it = 0; it <= kSegItems; ++it) {
    const uint32_t p = base + it;  // kv[it] is the key at position p - 1
    kv[it] = key[min(p == 0 ? 0u : p - 1, N - 1)];
  }
#pragma unroll
  for (int it = 0; it < kSegItems; ++it) {
    const uint32_t p = base + it;
    head[it] = p < N && (p == 0 || kv[it + 1] != kv[it]);
  }
}

// Also clears the centroid step's window counters (each tile clears those of its own positions).
__global__ __launch_bounds__(kSegThreads) void seg_count_kernel(const uint64_t* __restrict__ key, uint32_t N,
                                                                uint32_t nblk, uint32_t* __restrict__ blocksum,
                                                                uint32_t* __restrict__ window_counters) {
  __shared__ uint32_t wave_sum[kSegThreads / kWave];
  constexpr uint32_t kCountersPerTile = 2 * kSegTile / kCentroidWindow;
  static_assert(kSegTile % kCentroidWindow == 0 && kCountersPerTile <= kSegThreads, "window counters per tile");
  if (threadIdx.x < kCountersPerTile) window_counters[blockIdx.x * kCountersPerTile + threadIdx.x] = 0;
  const uint32_t base = blockIdx.x * kSegTile + threadIdx.x * kSegItems;
  uint64_t kv[kSegItems + 1];
  bool head[kSegItems];
  load_heads(key, base, N, kv, head);
  uint32_t c = 0;
#pragma unroll
  for (int it = 0; it < kSegItems; ++it) c += head[it] ? 1u : 0u;
  uint32_t total;
  block_exclusive_scan(c, wave_sum, total);
  if (threadIdx.x == 0) {
    blocksum[blockIdx.x] = total;
    if (blockIdx.x == 0) blocksum[nblk] = 0;  // after a scan this slot holds the grand total
  }
}

// SELF_PREFIX: blocksum holds per-tile head counts and the block adds up the tiles before it itself;
// otherwise blocksum has been scanned.
template <bool SELF_PREFIX>
__global__ __launch_bounds__(kSegThreads) void seg_write_kernel(
    const uint64_t* __restrict__ key, const int32_t* __restrict__ perm, uint32_t N, uint32_t E, int bbits,
    const uint32_t* __restrict__ blocksum, int32_t* __restrict__ seg_offsets, int32_t* __restrict__ seg_expert,
    int32_t* __restrict__ expert_offsets, int32_t* __restrict__ seg_of, int32_t* __restrict__ num_segments) {
  __shared__ uint32_t wave_sum[kSegThreads / kWave];
  uint32_t tiles_before = 0;
  if (SELF_PREFIX) {
    uint32_t part = 0;
    for (uint32_t t = threadIdx.x; t < blockIdx.x; t += kSegThreads) part += blocksum[t];
    block_exclusive_scan(part, wave_sum, tiles_before);
  } else {
    tiles_before = blocksum[blockIdx.x];
  }
  const uint32_t base = blockIdx.x * kSegTile + threadIdx.x * kSegItems;
  uint64_t kv[kSegItems + 1];
  bool head[kSegItems];
  load_heads(key, base, N, kv, head);
  int32_t a[kSegItems];
#pragma unroll
  for (int it = 0; it < kSegItems; ++it) a[it] = perm[min(base + it, N - 1)];
  uint32_t c = 0;
#pragma unroll
  for (int it = 0; it < kSegItems; ++it) c += head[it] ? 1u : 0u;
  uint32_t total;
  uint32_t seg = tiles_before + block_exclusive_scan(c, wave_sum, total);  // heads before this thread
#pragma unroll
  for (int it = 0; it < kSegItems; ++it) {
    const uint32_t p = base + it;
    if (p >= N) break;
    const uint32_t e = (uint32_t)(kv[it + 1] >> bbits);
    if (head[it]) {
      seg_offsets[seg] = (int32_t)p;
      seg_expert[seg] = (int32_t)e;
      const uint32_t first = p == 0 ? 0u : (uint32_t)(kv[it] >> bbits) + 1u;
      for (uint32_t x = first; x <= e; ++x) expert_offsets[x] = (int32_t)seg;  // experts that start (or are empty) here
      ++seg;
    }
    seg_of[a[it]] = (int32_t)(seg - 1);
    if (p == N - 1) {
      for (uint32_t x = e + 1; x <= E; ++x) expert_offsets[x] = (int32_t)seg;
      seg_offsets[seg] = (int32_t)N;
      *num_segments = (int32_t)seg;
    }
  }
}

// ---------------------------------------------------------------------------------------------------
// Two-launch route.
//
// tile_bin_kernel.  A workgroup sorts its TILE keys by their top kBinBits bits (the bin), stably, writes them back to
// the tile's own positions and records for every bin where it starts in the tile and how many keys it has.  Nothing
// global is needed: a bin's first position in the final order is the sum over all tiles of the bin's start inside
// the tile, which the workgroup that owns the bin adds up from its column of the table.  So there is no histogram
// launch before the scatter, no scan, and no scattered write beyond the tile's own few KB.
constexpr int kBinBits = 8;
constexpr int kBins = 1 << kBinBits;
static_assert(kBins == kSortThreads, "one bin per thread of tile_bin_kernel");
constexpr uint32_t kClaimStride = 8;         // four claims to a 128-byte line: exchanges on one word or line queue up
constexpr uint32_t kSyncWords = kBins * (1 + kClaimStride);   // published head counts of the bins, then their claims

template <int TILE>
__global__ __launch_bounds__(kSortThreads) void tile_bin_kernel(KeySource src, uint32_t N, int shift,
                                                                uint32_t* __restrict__ table, uint64_t* __restrict__ dst_key,
                                                                int32_t* __restrict__ dst_idx, uint32_t* __restrict__ sync) {
  constexpr int kItems = TILE / kSortThreads, kGroups = TILE / kWave;
  static_assert(TILE <= 0xffff, "start and count of a bin in a tile share a word");
  __shared__ uint32_t cnt[kGroups][kBins];   // keys of a bin in a group of 64; then the group's first position of it
  __shared__ uint32_t wave_sum[kSortThreads / kWave];
  if (blockIdx.x == 0) {                     // what bin_group_kernel expects to find cleared
    sync[threadIdx.x] = 0;
    sync[kBins + threadIdx.x * kClaimStride] = 0;
  }
  const uint32_t base = blockIdx.x * TILE;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  uint64_t key[kItems];
  int32_t idx[kItems];
  uint32_t rank[kItems];
#pragma unroll
  for (int it = 0; it < kItems; ++it)        // positions past N re-read the last key and are masked out below
    load_item<true>(src, min(base + it * kSortThreads + threadIdx.x, N - 1), key[it], idx[it]);
#pragma unroll
  for (int g = 0; g < kGroups; ++g) cnt[g][threadIdx.x] = 0;   // while the loads fly
  __syncthreads();
#pragma unroll
  for (int it = 0; it < kItems; ++it) {
    const bool valid = base + it * kSortThreads + threadIdx.x < N;
    const uint32_t digit = (uint32_t)(key[it] >> shift) & (kBins - 1);
    const uint64_t same = same_digit_lanes(digit, kBinBits, valid);
    rank[it] = (uint32_t)__popcll(same & lt_mask);
    if (valid && rank[it] == 0) cnt[it * (kSortThreads / kWave) + wave][digit] = (uint32_t)__popcll(same);
  }
  __syncthreads();
  {
    uint32_t c[kGroups], total = 0;
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
      c[g] = cnt[g][threadIdx.x];
      total += c[g];
    }
    uint32_t unused;
    uint32_t run = block_exclusive_scan(total, wave_sum, unused);
    table[blockIdx.x * kBins + threadIdx.x] = run | (total << 16);
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
      cnt[g][threadIdx.x] = run;
      run += c[g];
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < kItems; ++it) {
    if (base + it * kSortThreads + threadIdx.x < N) {
      const uint32_t digit = (uint32_t)(key[it] >> shift) & (kBins - 1);
      const uint32_t pos = base + cnt[it * (kSortThreads / kWave) + wave][digit] + rank[it];
      dst_key[pos] = key[it];
      dst_idx[pos] = idx[it];
    }
  }
}

// bin_group_kernel.  One workgroup of 16 waves per bin.  It reads the bin's column of the table, collects the bin's
// keys from the tiles (element i of the bin is found by bisection over the tiles' running counts), sorts them in LDS,
// publishes the number of clusters it found, adds up the numbers of all bins before it and writes the outputs.
//
// What bounds it: dependent trips to memory that other XCDs wrote (table 1.8 us, keys 0.7, published counts 2.0) and
// the barriers of the sort (1.8 for 512 keys); all 256 bins run side by side, one to a compute unit.  16 waves: with
// 4 the sort took twice as long (LDS latency, not instructions).  Measured, both launches together, against the
// histogram, scatter, bin sort and numbering launches these two replace: 131072 assignments 16.4 us (30), 65536 with
// 50-bit ids 15.5 (30), 16384 12.4 (18); one workgroup alone, 2048 assignments: 9.7 (14.5), 74: 4.7 (8.0).
//
// The wait for the bins before.  A workgroup claims its bin with an exchange on the bin's claim word, publishes the
// bin's count before it waits for anything, and waits only for counts.  When one does not come it tries to claim the
// lowest bin that is still open: if that succeeds, the bin's own workgroup has not started (and will leave when it
// does), and the waiting workgroup does the bin itself - nothing before it is open, so without a wait - and then
// returns to its own; if not, the bin's owner is running and will publish.  So every wait ends, whatever else runs on
// the GPU and in whatever order workgroups are started.  (A ticket counter gives the same, but 256 workgroups adding
// to one word took 3.4 us.)  The counts and claims are the only data exchanged inside the launch, as relaxed
// device-scope accesses: no fence is needed.
//
// Sorting up to kBinCap keys, two ways:
//   sub-bins: the keys are thrown into 4096 sub-bins by their next 12 bits with LDS counters, in whatever order they
//     arrive; a key's rank is the start of its sub-bin plus the number of its keys that come before it, by key and,
//     among equal keys, by assignment.  Cost grows with the fullest sub-bin.
//   radix: least-significant-digit passes; each wave owns a slice of the bin, ranks inside a round of 64 keys come
//     from ballots.  Cost grows with the number of digits, whatever the data.
// A pass costs about as much as comparing with kCrowdPerPass keys, so the sub-bins are taken when no sub-bin holds
// more than that many keys per pass saved, and never for a single pass (25088 assignments of a Zipf gate: 14.2 us
// with sub-bins, 10.5 without).
// Larger bins: see sort_bin.  Everything must fit the 128 registers of a 1024-thread workgroup: a kernel that spills
// a few of them to scratch memory starts 3 to 8 us later, which is why kBinCap is not 8192.
//
// DIRECT: the whole input (up to kSmallMaxN assignments) is the one bin of a single workgroup.
constexpr int kXcds = 8;
constexpr int kBinWaves = 16;
constexpr int kBinThreads = kBinWaves * 64;
constexpr int kBinCap = 4096;                       // keys of a bin sorted in LDS
constexpr int kBinItems = kBinCap / kBinThreads;
constexpr int kSubBits = 12;
constexpr int kSubBins = 1 << kSubBits;
static_assert(kBinThreads >= kBins && kSubBins % kBinThreads == 0, "counters per thread");
constexpr uint32_t kCrowdPerPass = 32;
constexpr int kBigRounds = 4;                       // rounds of 64 keys a wave has in flight in a larger bin
static_assert(kSmallMaxN <= kBinCap, "a single workgroup sorts the smallest inputs in LDS");

struct BinLds {
  uint64_t key[kBinCap];
  int32_t idx[kBinCap];
  union {
    uint32_t cnt[kBinWaves][kGroupBins];              // radix: keys per (wave, digit)
    struct {
      uint32_t cnt[kSubBins], base[kSubBins];
    } sub;
  };
};
static_assert(sizeof(BinLds) <= 140 * 1024, "LDS of a compute unit, less the rest of the kernel");

struct BinArgs {
  KeySource src;              // DIRECT, and the keys of a bin of more than kBinCap keys
  const uint32_t* table;      // [tiles][kBins]: start of the bin inside the tile | keys << 16
  const uint64_t* tile_key;   // the tiles, each sorted by bin
  const int32_t* tile_idx;
  uint32_t tiles, tile_bits;
  uint32_t N, E;
  int bbits, top_shift;       // bin of a key is key >> top_shift
  int passes;                 // radix passes over the key bits below the bin
  int shift[8], width[8];
  int sub_shift;              // sub-bin of a key is (key >> sub_shift) & (kSubBins - 1)
  int32_t* big_idx;           // the ids of a bin of more than kBinCap keys go between here and perm
  int32_t *seg_offsets, *seg_expert, *expert_offsets, *perm, *seg_of, *num_segments;
  uint32_t* sync;             // kSyncWords, zero on entry (not used with DIRECT)
  uint32_t* window_counters;  // cleared here for the centroid step
  uint32_t n_counters;
  uint32_t first_bin;         // the workgroups of the bins before it leave at once (0; a test forces the takeover of bins with it)
  uint32_t spins;             // looks at the open counts before a workgroup tries to take one of them over
};

// Inclusive sum over the lanes of the wave, in the vector unit's cross-lane paths (no LDS).
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);   // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);   // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);   // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);   // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return v;
}

// Exclusive scan of one value per thread of the workgroup.  One barrier inside; the next one that the caller passes
// frees wave_sum.
__device__ __forceinline__ uint32_t bin_exclusive_scan(uint32_t v, uint32_t* wave_sum /*[kBinWaves]*/, uint32_t& total) {
  const int wave = threadIdx.x >> 6;
  const uint32_t inc = wave_inclusive_sum(v);
  if ((threadIdx.x & 63) == 63) wave_sum[wave] = inc;
  __syncthreads();
  uint32_t before = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < kBinWaves; ++w) {
    const uint32_t t = wave_sum[w];
    if (w < wave) before += t;
    total += t;
  }
  return before + inc - v;
}

// Digit counts per wave -> start offsets in (digit, wave) order.  Called by the whole workgroup between two barriers.
__device__ __forceinline__ void digit_starts(uint32_t (&cnt)[kBinWaves][kGroupBins], uint32_t* wave_sum) {
  constexpr int kPer = kGroupBins > kBinThreads ? kGroupBins / kBinThreads : 1;    // neighbouring digits of a thread
  const bool owner = threadIdx.x * kPer < kGroupBins;
  uint32_t c[kPer][kBinWaves], tot = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j)
#pragma unroll
    for (int w = 0; w < kBinWaves; ++w) {
      c[j][w] = owner ? cnt[w][threadIdx.x * kPer + j] : 0u;
      tot += c[j][w];
    }
  uint32_t unused;
  uint32_t run = bin_exclusive_scan(tot, wave_sum, unused);
#pragma unroll
  for (int j = 0; j < kPer; ++j)
#pragma unroll
    for (int w = 0; w < kBinWaves; ++w) {
      if (owner) cnt[w][threadIdx.x * kPer + j] = run;
      run += c[j][w];
    }
}

// Radix digits of a wave's keys, round q being positions lo + 64 q .. of its slice [lo, hi): place[q] is the number of
// keys of the same digit before the key in the slice; cnt ends as the slice's digit counts (zero on entry).
__device__ __forceinline__ void count_round_digits(uint32_t* cnt, const uint64_t (&key)[kBinItems], uint32_t (&place)[kBinItems],
                                                   int shift, int width, uint32_t lo, uint32_t hi) {
  const int lane = threadIdx.x & 63;
  const uint64_t lt_mask = (1ull << lane) - 1ull;
#pragma unroll
  for (int q = 0; q < kBinItems; ++q) {
    if (lo + q * 64 < hi) {                         // wave-uniform
      const bool valid = lo + q * 64 + lane < hi;
      const uint32_t digit = (uint32_t)(key[q] >> shift) & ((1u << width) - 1u);
      const uint64_t same = same_digit_lanes(digit, width, valid);
      const uint32_t rank = (uint32_t)__popcll(same & lt_mask);
      const uint32_t run = cnt[digit];
      place[q] = run + rank;
      if (valid && rank == 0) cnt[digit] = run + (uint32_t)__popcll(same);   // after every lane of the round has read
    }
  }
}

struct BinShared {
  uint32_t wave_sum[2][kBinWaves];
  uint32_t tile_before[kMaxTiles], tile_from[kMaxTiles];   // keys of the bin in earlier tiles; where the tile's begin
  uint32_t head_cnt[65];             // clusters in, then before, a round of one wave; [64]: ... before the common key
  uint32_t claimed, open_bin;
};

struct BinState {                    // a sorted bin
  uint32_t n, start, heads;          // keys, first position, clusters
  uint32_t x_lo, x_hi;               // experts whose first possible key lies in this bin: their offsets are written with it
  bool big;                          // the sorted ids are in perm; else keys and ids are in LDS
  uint32_t less, equal;              // in LDS: the first `less` keys come before `equal` ones that are `common`
  uint64_t common;
  uint32_t heads_before;             // big: clusters before the wave's slice
};

// Collects and sorts a bin and counts its clusters.  taken: not 0 in thread 0 when the bin belongs to another
// workgroup; the answer is false then.
template <bool DIRECT>
__device__ __forceinline__ bool sort_bin(const BinArgs& a, uint32_t bin, uint32_t taken, BinLds& m,
                                         BinShared& sh, BinState& st) {
  const uint32_t tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  uint32_t n = a.N, start = 0;
  if (!DIRECT) {
    static_assert(kMaxTiles == kBins && kMaxTiles % 64 == 0, "one tile per thread of the first waves");
    uint32_t keys = 0, first = 0;
    if (tid < a.tiles) {
      const uint32_t e = a.table[tid * kBins + bin];
      first = e & 0xffffu;
      keys = e >> 16;
    }
    const uint32_t inc = wave_inclusive_sum(keys), inc_first = wave_inclusive_sum(first);
    if (lane == 63) {
      sh.wave_sum[0][wave] = inc;
      sh.wave_sum[1][wave] = inc_first;
    }
    __syncthreads();
    uint32_t before = inc - keys;
    n = 0;
#pragma unroll
    for (int w = 0; w < kMaxTiles / 64; ++w) {      // later waves hold no tile
      const uint32_t c = sh.wave_sum[0][w];
      if (w < wave) before += c;
      n += c;
      start += sh.wave_sum[1][w];
    }
    if (tid < a.tiles) {
      sh.tile_before[tid] = before;
      sh.tile_from[tid] = (tid << a.tile_bits) + first - before;   // source of element i of the bin: tile_from + i
    }
    if (tid == 0) sh.claimed = taken == 0;
    __syncthreads();
    if (!sh.claimed) return false;                  // the bin is done by a workgroup that waited for it
  }
  // experts whose first possible key lies in this bin: their offsets are written here
  uint32_t x_lo = 0, x_hi = a.E;
  if (!DIRECT) {
    const int up = a.bbits - a.top_shift;
    x_lo = up >= 0 ? (bin + (1u << up) - 1u) >> up : bin << -up;
    x_hi = up >= 0 ? (bin + 1u + (1u << up) - 1u) >> up : (bin + 1u) << -up;
    x_lo = min(x_lo, a.E);
    x_hi = min(x_hi, a.E);
  }
  auto fetch = [&](uint32_t i, uint64_t& key, int32_t& idx) {   // element i < n of the bin, in assignment order
    if (DIRECT) {
      load_item<true>(a.src, i, key, idx);
    } else {
      uint32_t lo = 0, hi = a.tiles;                // last tile with tile_before <= i
      while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (sh.tile_before[mid] <= i) lo = mid; else hi = mid;
      }
      key = a.tile_key[sh.tile_from[lo] + i];
      idx = a.tile_idx[sh.tile_from[lo] + i];
    }
  };

  // A bin of more than kBinCap keys is hardly ever made of many clusters: it is the one key that a share of the tokens
  // has in common (padding).  If one key makes up most of the bin, its assignments go straight to their place in perm
  // (two walks over the bin, no sort) and the rest, if it is small enough, is sorted in LDS.  (26000 equal keys among
  // 131072, compress call at d = 8: 132 us, 361 with the passes below.)  Else the same radix passes as in LDS run
  // through global memory, by the one workgroup.  Only ids are moved: the keys are made from the inputs again in every
  // walk, so that the workspace holds no further key buffers.
  uint32_t less = n, equal = 0;                     // rest[0, less) comes before the common key, `equal` keys are it
  uint64_t common = 0;
  if (!DIRECT && n > (uint32_t)kBinCap) {
    uint64_t key;
    int32_t idx;
    fetch((uint32_t)(((uint64_t)n * (2u * lane + 1u)) >> 7), key, idx);   // 64 samples, the same in every wave
    uint32_t best = 0;
    for (int l = 0; l < 64; l += 4) {               // sixteen candidates
      const uint64_t o = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(key >> 32), l) << 32) |
                         (uint32_t)__builtin_amdgcn_readlane((int)key, l);
      const uint32_t same = (uint32_t)__popcll(__ballot(key == o));
      if (same > best) {
        best = same;
        common = o;
      }
    }
    // worth the walk when three quarters of the share that is needed shows up in the samples
    if (best > 1 && (uint64_t)best * n * 4u >= (uint64_t)(n - kBinCap) * (64u * 3u)) {
      const uint32_t hslice = ((n + kBinWaves - 1) / kBinWaves + 63u) & ~63u;
      const uint32_t hlo = min((uint32_t)wave * hslice, n), hhi = min(hlo + hslice, n);
      uint32_t eq = 0, lt = 0;
      auto walk = [&](auto&& f) {                   // f(valid, key, idx) for every round of the wave's slice
        for (uint32_t b = hlo; b < hhi; b += kBigRounds * 64) {
          uint64_t k[kBigRounds];
          int32_t id[kBigRounds];
#pragma unroll
          for (int q = 0; q < kBigRounds; ++q) fetch(min(b + q * 64 + lane, n - 1), k[q], id[q]);
#pragma unroll
          for (int q = 0; q < kBigRounds; ++q) f(b + q * 64 + lane < hhi, k[q], id[q]);
        }
      };
      walk([&](bool valid, uint64_t k, int32_t) {
        eq += (uint32_t)__popcll(__ballot(valid && k == common));
        lt += (uint32_t)__popcll(__ballot(valid && k < common));
      });
      uint32_t eq_all, lt_all;
      uint32_t eq_at = bin_exclusive_scan(lane == 0 ? eq : 0u, sh.wave_sum[0], eq_all);
      bin_exclusive_scan(lane == 0 ? lt : 0u, sh.wave_sum[1], lt_all);
      if (n - eq_all <= (uint32_t)kBinCap) {
        less = lt_all;
        equal = eq_all;
        eq_at = (uint32_t)__builtin_amdgcn_readfirstlane((int)eq_at);
        uint32_t rest_at = hlo - eq_at;             // keys of the rest before this wave's slice
        walk([&](bool valid, uint64_t k, int32_t id) {
          const uint64_t e = __ballot(valid && k == common), r = __ballot(valid && k != common);
          if (valid && k == common) a.perm[start + less + eq_at + (uint32_t)__popcll(e & lt_mask)] = id;
          if (valid && k != common) {
            m.key[rest_at + (uint32_t)__popcll(r & lt_mask)] = k;
            m.idx[rest_at + (uint32_t)__popcll(r & lt_mask)] = id;
          }
          eq_at += (uint32_t)__popcll(e);
          rest_at += (uint32_t)__popcll(r);
        });
      }
      __syncthreads();
    }
  }
  const uint32_t rest = n - equal;                  // keys to sort
  const bool big = !DIRECT && rest > (uint32_t)kBinCap;
  st.big = big;
  auto key_of = [&](int32_t id) {
    uint64_t key;
    int32_t unused;
    load_item<true>(a.src, (uint32_t)id, key, unused);
    return key;
  };
  const uint32_t slice = ((rest + kBinWaves - 1) / kBinWaves + 63u) & ~63u;   // keys per wave, whole rounds
  const uint32_t wlo = min((uint32_t)wave * slice, rest), whi = min(wlo + slice, rest);
  uint32_t heads = 0;

  if (!big) {
    uint64_t key[kBinItems];
    int32_t idx[kBinItems];
#pragma unroll
    for (int q = 0; q < kBinItems; ++q) {
      const uint32_t i = tid + q * kBinThreads;
      if (i < rest) {
        if (equal == 0) {
          fetch(i, key[q], idx[q]);
        } else {
          key[q] = m.key[i];
          idx[q] = m.idx[i];
        }
      }
    }
    if (equal != 0) __syncthreads();
    bool sorted = false;
    if (a.passes > 1) {
      constexpr int kPer = kSubBins / kBinThreads;    // neighbouring sub-bins of a thread
      static_assert(kPer == 4, "moved 16 bytes at a time");
      const int sub_shift = a.sub_shift;
      auto sub_of = [&](uint64_t k) { return (uint32_t)(k >> sub_shift) & (kSubBins - 1); };
      reinterpret_cast<uint4*>(m.sub.cnt)[tid] = make_uint4(0, 0, 0, 0);
      __syncthreads();
      uint32_t slot[kBinItems];
#pragma unroll
      for (int q = 0; q < kBinItems; ++q)
        if (tid + q * kBinThreads < rest) slot[q] = atomicAdd(&m.sub.cnt[sub_of(key[q])], 1u);
      __syncthreads();
      const uint4 c = reinterpret_cast<const uint4*>(m.sub.cnt)[tid];
      const uint32_t most = max(max(c.x, c.y), max(c.z, c.w));
      if (!__syncthreads_or(most > kCrowdPerPass * (uint32_t)a.passes)) {
        uint32_t unused;
        const uint32_t run = bin_exclusive_scan(c.x + c.y + c.z + c.w, sh.wave_sum[0], unused);
        reinterpret_cast<uint4*>(m.sub.base)[tid] = make_uint4(run, run + c.x, run + c.x + c.y, run + c.x + c.y + c.z);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kBinItems; ++q) {
          if (tid + q * kBinThreads < rest) {
            const uint32_t at = m.sub.base[sub_of(key[q])] + slot[q];
            m.key[at] = key[q];
            m.idx[at] = idx[q];
          }
        }
        __syncthreads();
        uint32_t rank[kBinItems];
#pragma unroll
        for (int q = 0; q < kBinItems; ++q) {
          if (tid + q * kBinThreads < rest) {
            const uint32_t sub = sub_of(key[q]);
            uint32_t t = m.sub.base[sub];
            const uint32_t end = t + m.sub.cnt[sub];
            rank[q] = t;
            auto before = [&](uint64_t k, int32_t i) { return k < key[q] || (k == key[q] && i < idx[q]) ? 1u : 0u; };
            for (; t + 4 <= end; t += 4) {            // crowded: four reads in flight
              uint64_t kj[4];
              int32_t ij[4];
#pragma unroll
              for (int u = 0; u < 4; ++u) {
                kj[u] = m.key[t + u];
                ij[u] = m.idx[t + u];
              }
#pragma unroll
              for (int u = 0; u < 4; ++u) rank[q] += before(kj[u], ij[u]);
            }
            for (; t < end; ++t) rank[q] += before(m.key[t], m.idx[t]);
          }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kBinItems; ++q) {
          if (tid + q * kBinThreads < rest) {
            m.key[rank[q]] = key[q];
            m.idx[rank[q]] = idx[q];
          }
        }
        sorted = true;
      }
    }
    if (!sorted) {
#pragma unroll
      for (int q = 0; q < kBinItems; ++q) {
        const uint32_t i = tid + q * kBinThreads;
        if (i < rest) {
          m.key[i] = key[q];
          m.idx[i] = idx[q];
        }
      }
      for (int p = 0; p < a.passes; ++p) {
        const int shift = a.shift[p], width = a.width[p];
        const uint32_t mask = (1u << width) - 1u;
        __syncthreads();                            // the counters are no longer read
        for (int i = tid; i < kBinWaves * kGroupBins / 4; i += kBinThreads)
          reinterpret_cast<uint4*>(&m.cnt[0][0])[i] = make_uint4(0, 0, 0, 0);
        __syncthreads();                            // also: the keys are in LDS
        uint32_t place[kBinItems];
#pragma unroll
        for (int q = 0; q < kBinItems; ++q) {
          if (wlo + q * 64 < whi) {                 // wave-uniform
            key[q] = m.key[min(wlo + q * 64 + lane, rest - 1)];
            idx[q] = m.idx[min(wlo + q * 64 + lane, rest - 1)];
          }
        }
        count_round_digits(m.cnt[wave], key, place, shift, width, wlo, whi);
        __syncthreads();                            // also: every key is in a register
        digit_starts(m.cnt, sh.wave_sum[p & 1]);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kBinItems; ++q) {
          if (wlo + q * 64 + lane < whi) {
            const uint32_t at = m.cnt[wave][(uint32_t)(key[q] >> shift) & mask] + place[q];
            m.key[at] = key[q];
            m.idx[at] = idx[q];
          }
        }
      }
    }
    __syncthreads();
    // heads: a key that differs from the one before it (the first key of a bin always starts a cluster)
#pragma unroll
    for (int q = 0; q < kBinItems; ++q) {
      const uint32_t i = tid + q * kBinThreads;
      const bool head = i < rest && (i == 0 || m.key[i] != m.key[i - 1]);
      const uint32_t c = (uint32_t)__popcll(__ballot(head));
      if (lane == 0) sh.head_cnt[q * kBinWaves + wave] = c;
    }
    __syncthreads();
    static_assert(kBinItems * kBinWaves == 64, "one round of one wave per lane");
    const uint32_t mine = sh.head_cnt[lane], inc = wave_inclusive_sum(mine);
    heads = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63) + (equal != 0 ? 1u : 0u);
    __syncthreads();
    if (wave == 0) sh.head_cnt[lane] = inc - mine;   // read after the barriers of the wait for the bins before
    if (DIRECT) __syncthreads();
  } else {
    // the ids are collected into one piece of global memory, then radix passes there; every wave walks its slice 64
    // keys at a time, twice per pass
    {
      int32_t* ids = ((a.passes & 1) ? a.big_idx : a.perm) + start;   // the last pass leaves the ids in perm
      for (uint32_t b = tid; b < n; b += kBigRounds * kBinThreads) {
        uint64_t key[kBigRounds];
        int32_t idx[kBigRounds];
#pragma unroll
        for (int q = 0; q < kBigRounds; ++q) fetch(min(b + q * kBinThreads, n - 1), key[q], idx[q]);
#pragma unroll
        for (int q = 0; q < kBigRounds; ++q) {
          if (b + q * kBinThreads < n) ids[b + q * kBinThreads] = idx[q];
        }
      }
      __syncthreads();
    }
    for (int p = 0; p < a.passes; ++p) {
      const int shift = a.shift[p], width = a.width[p];
      const uint32_t mask = (1u << width) - 1u;
      const bool to_perm = ((a.passes - 1 - p) & 1) == 0;
      const int32_t* sidx = (to_perm ? a.big_idx : a.perm) + start;
      int32_t* didx = (to_perm ? a.perm : a.big_idx) + start;
      for (int i = tid; i < kBinWaves * kGroupBins / 4; i += kBinThreads)
        reinterpret_cast<uint4*>(&m.cnt[0][0])[i] = make_uint4(0, 0, 0, 0);
      __syncthreads();
      for (uint32_t b = wlo; b < whi; b += kBigRounds * 64) {   // several rounds of loads in flight
        uint64_t key[kBigRounds];
#pragma unroll
        for (int q = 0; q < kBigRounds; ++q) key[q] = key_of(sidx[min(b + q * 64 + lane, n - 1)]);
#pragma unroll
        for (int q = 0; q < kBigRounds; ++q)
          if (b + q * 64 + lane < whi) atomicAdd(&m.cnt[wave][(uint32_t)(key[q] >> shift) & mask], 1u);
      }
      __syncthreads();
      digit_starts(m.cnt, sh.wave_sum[p & 1]);
      __syncthreads();
      for (uint32_t b = wlo; b < whi; b += kBigRounds * 64) {
        uint64_t key[kBigRounds];
        int32_t idx[kBigRounds];
#pragma unroll
        for (int q = 0; q < kBigRounds; ++q) {
          idx[q] = sidx[min(b + q * 64 + lane, n - 1)];
          key[q] = key_of(idx[q]);
        }
#pragma unroll
        for (int q = 0; q < kBigRounds; ++q) {
          if (b + q * 64 < whi) {                   // wave-uniform
            const bool valid = b + q * 64 + lane < whi;
            const uint32_t digit = (uint32_t)(key[q] >> shift) & mask;
            const uint64_t same = same_digit_lanes(digit, width, valid);
            const uint32_t rank = (uint32_t)__popcll(same & lt_mask);
            const uint32_t run = m.cnt[wave][digit];
            if (valid) {
              didx[run + rank] = idx[q];
              if (rank == 0) m.cnt[wave][digit] = run + (uint32_t)__popcll(same);   // after every lane of the round has read
            }
          }
        }
      }
      __syncthreads();   // the pass's global writes are visible to the whole workgroup (one compute unit, one L1)
    }
    const int32_t* ids = a.perm + start;
    uint32_t mine = 0;
    for (uint32_t b = wlo; b < whi; b += kBigRounds * 64) {
      uint64_t key[kBigRounds], prev[kBigRounds];
#pragma unroll
      for (int q = 0; q < kBigRounds; ++q) {
        const uint32_t i = min(b + q * 64 + lane, n - 1);
        key[q] = key_of(ids[i]);
        prev[q] = key_of(ids[i == 0 ? 0 : i - 1]);
      }
#pragma unroll
      for (int q = 0; q < kBigRounds; ++q) {
        const uint32_t i = b + q * 64 + lane;
        mine += (uint32_t)__popcll(__ballot(i < whi && (i == 0 || key[q] != prev[q])));
      }
    }
    st.heads_before = bin_exclusive_scan(lane == 0 ? mine : 0u, sh.wave_sum[0], heads);
    st.heads_before = (uint32_t)__shfl((int)st.heads_before, 0, 64);   // heads before this wave's slice
  }
  st.n = n;
  st.start = start;
  st.less = less;
  st.equal = equal;
  st.common = common;
  st.heads = heads;
  st.x_lo = x_lo;
  st.x_hi = x_hi;
  return true;
}

// Writes the outputs of a sorted bin; `base` clusters come before it.
template <bool DIRECT>
__device__ __forceinline__ void write_bin(const BinArgs& a, uint32_t bin, uint32_t base, const BinLds& m, BinShared& sh,
                                          const BinState& st) {
  const uint32_t tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const uint64_t le_mask = ((1ull << lane) - 1ull) | (1ull << lane);
  const uint32_t n = st.n;
  auto emit = [&](uint32_t i, uint64_t key, uint64_t prev, bool head, uint32_t seg, int32_t assignment) {
    if (head) {
      const uint32_t e = (uint32_t)(key >> a.bbits);
      a.seg_offsets[seg] = (int32_t)(st.start + i);
      a.seg_expert[seg] = (int32_t)e;
      // experts that start (or are empty) between the key before and this one
      for (uint32_t x = i == 0 ? st.x_lo : (uint32_t)(prev >> a.bbits) + 1u; x <= e; ++x) a.expert_offsets[x] = (int32_t)seg;
    }
    a.seg_of[assignment] = (int32_t)seg;
  };
  uint32_t x_tail = st.x_lo;                        // experts of this bin behind its last key
  if (!st.big) {
    const uint32_t rest = n - st.equal;
    if (st.equal != 0) {                            // the cluster of the common key
      if (tid == 0) sh.head_cnt[64] = st.heads - 1u;
      __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < kBinItems; ++q) {
      const uint32_t i = tid + q * kBinThreads;
      if (i < rest) {
        const uint64_t key = m.key[i], prev = m.key[i == 0 ? 0 : i - 1];
        const int32_t idx = m.idx[i];
        const bool head = i == 0 || key != prev;
        const uint64_t hmask = __ballot(head);
        uint32_t seg = base + sh.head_cnt[q * kBinWaves + wave] + (uint32_t)__popcll(hmask & le_mask) - 1u;
        if (i < st.less) {
          a.perm[st.start + i] = idx;
          emit(i, key, prev, head, seg, idx);
        } else {                                    // behind the common key
          if (i == st.less) sh.head_cnt[64] = seg - base;
          a.perm[st.start + st.equal + i] = idx;
          emit(st.equal + i, key, i == st.less ? st.common : prev, head, seg + 1u, idx);
        }
      }
    }
    if (st.equal != 0) {
      __syncthreads();
      const uint32_t seg = base + sh.head_cnt[64];
      if (tid == 0) emit(st.less, st.common, st.less == 0 ? st.common : m.key[st.less - 1], true, seg, a.perm[st.start + st.less]);
      for (uint32_t b = tid; b < st.equal; b += kBigRounds * kBinThreads) {
        int32_t idx[kBigRounds];
#pragma unroll
        for (int q = 0; q < kBigRounds; ++q) idx[q] = a.perm[st.start + st.less + min(b + q * kBinThreads, st.equal - 1)];
#pragma unroll
        for (int q = 0; q < kBigRounds; ++q)
          if (b + q * kBinThreads < st.equal) a.seg_of[idx[q]] = (int32_t)seg;
      }
      x_tail = max(x_tail, (uint32_t)(st.common >> a.bbits) + 1u);
    }
    if (rest > 0) x_tail = max(x_tail, (uint32_t)(m.key[rest - 1] >> a.bbits) + 1u);
  } else {
    auto key_of = [&](int32_t id) {
      uint64_t key;
      int32_t unused;
      load_item<true>(a.src, (uint32_t)id, key, unused);
      return key;
    };
    const uint32_t slice = ((n + kBinWaves - 1) / kBinWaves + 63u) & ~63u;
    const uint32_t wlo = min((uint32_t)wave * slice, n), whi = min(wlo + slice, n);
    uint32_t seg = base + st.heads_before;
    for (uint32_t b = wlo; b < whi; b += kBigRounds * 64) {
      uint64_t key[kBigRounds], prev[kBigRounds];
      int32_t idx[kBigRounds];
#pragma unroll
      for (int q = 0; q < kBigRounds; ++q) {
        const uint32_t i = min(b + q * 64 + lane, n - 1);
        idx[q] = a.perm[st.start + i];
        key[q] = key_of(idx[q]);
        prev[q] = key_of(a.perm[st.start + (i == 0 ? 0 : i - 1)]);
      }
#pragma unroll
      for (int q = 0; q < kBigRounds; ++q) {
        const uint32_t i = b + q * 64 + lane;
        const bool head = i < whi && (i == 0 || key[q] != prev[q]);
        const uint64_t hmask = __ballot(head);
        if (i < whi) emit(i, key[q], prev[q], head, seg + (uint32_t)__popcll(hmask & le_mask) - 1u, idx[q]);
        seg += (uint32_t)__popcll(hmask);
      }
    }
    x_tail = max(x_tail, (uint32_t)(key_of(a.perm[st.start + n - 1]) >> a.bbits) + 1u);
  }
  for (uint32_t x = x_tail + tid; x < st.x_hi; x += kBinThreads) a.expert_offsets[x] = (int32_t)(base + st.heads);
  if (tid == 0 && (DIRECT || bin == kBins - 1)) {
    a.expert_offsets[a.E] = (int32_t)(base + st.heads);
    a.seg_offsets[base + st.heads] = (int32_t)a.N;
    *a.num_segments = (int32_t)(base + st.heads);
  }
}

template <bool DIRECT>
__global__ __launch_bounds__(kBinThreads) void bin_group_kernel(BinArgs args) {
  extern __shared__ uint64_t bin_lds[];
  BinLds& m = *reinterpret_cast<BinLds*>(bin_lds);
  __shared__ BinShared sh;
  const uint32_t tid = threadIdx.x;
  for (uint32_t i = blockIdx.x * kBinThreads + tid; i < args.n_counters; i += gridDim.x * kBinThreads) args.window_counters[i] = 0;
  if (DIRECT) {
    BinState st;
    sort_bin<true>(args, 0, 0, m, sh, st);
    write_bin<true>(args, 0, 0, m, sh, st);
    return;
  }
  // consecutive workgroups sit on different XCDs; neighbouring bins, whose keys and table entries share cache lines,
  // go to the same one
  const uint32_t own = (blockIdx.x % kXcds) * (kBins / kXcds) + blockIdx.x / kXcds;
  if (own < args.first_bin) return;                 // never with first_bin = 0
  uint32_t taken = tid == 0 ? atomicExch(&args.sync[kBins + own * kClaimStride], 1u) : 0u;
  // One turn, unless a bin is taken over: that bin then, and after it the own one again (it was in LDS).  The
  // arguments are read through a pointer that the compiler must take for a new one in every turn; otherwise it keeps
  // all of them in scalar registers across the loop, and has to spill those.
  for (uint32_t bin = own;;) {
    auto ap = (const __attribute__((address_space(4))) BinArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(ap));
    const BinArgs& a = *(const BinArgs*)ap;
    BinState st;
    if (!sort_bin<false>(a, bin, taken, m, sh, st)) return;
    taken = 0;
    if (tid == 0) __hip_atomic_store(&a.sync[bin], st.heads + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // clusters before this bin: every published count is one more than the bin's clusters, 0 as long as there is none
    uint32_t v = 0;
    bool take_over = false;
    for (uint32_t spin = 1;; ++spin) {
      if (tid < bin && v == 0) v = __hip_atomic_load(&a.sync[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const bool open = tid < bin && v == 0;
      if (!__syncthreads_or(open)) break;
      if (spin < a.spins) continue;
      spin = 0;
      if (tid == 0) sh.open_bin = kBins;
      __syncthreads();
      if (open) atomicMin(&sh.open_bin, tid);
      __syncthreads();
      if (tid == 0) sh.claimed = atomicCAS(&a.sync[kBins + sh.open_bin * kClaimStride], 0u, 1u) == 0u;
      __syncthreads();
      if ((take_over = sh.claimed)) break;
    }
    if (take_over) {
      bin = sh.open_bin;
      __syncthreads();
      continue;
    }
    uint32_t base;
    bin_exclusive_scan(v == 0 ? 0u : v - 1u, sh.wave_sum[1], base);
    write_bin<false>(a, bin, base, m, sh, st);
    if (bin == own) return;
    bin = own;
    __syncthreads();
  }
}

int bits_for(uint64_t max_value) {  // number of bits needed to hold max_value
  int b = 0;
  while (max_value) {
    ++b;
    max_value >>= 1;
  }
  return b;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Raises the dynamic LDS limit of a kernel (once per kernel; repeating the call is harmless).
template <typename K> hipError_t raise_lds(K kern, size_t bytes, std::atomic<bool>& raised) {
  if (raised.load(std::memory_order_acquire)) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess) raised.store(true, std::memory_order_release);
  return e;
}

// A launch followed by a look at its status: a refused launch ends the call before anything else is enqueued.
#define LSHMOE_LAUNCH(...)                                                        \
  do {                                                                            \
    hipLaunchKernelGGL(__VA_ARGS__);                                              \
    if (hipError_t launch_err = hipGetLastError(); launch_err != hipSuccess) return launch_err; \
  } while (0)

template <bool FIRST>
hipError_t launch_scatter(const KeySource& src, uint32_t N, int shift, uint32_t mask, uint32_t nblk, const uint32_t* table,
                          uint64_t* dkey, int32_t* didx, hipStream_t stream) {
  constexpr size_t kScatterLds = (size_t)kGroupBins * (kSortTile / kWave + 1) * 4;  // 66 KB
  auto kern = sort_scatter_kernel<FIRST>;
  static std::atomic<bool> raised{false};
  if (hipError_t e = raise_lds(kern, kScatterLds, raised); e != hipSuccess) return e;
  LSHMOE_LAUNCH(kern, dim3(nblk), dim3(kSortThreads), kScatterLds, stream, src, N, shift, mask, nblk, table, dkey, didx);
  return hipSuccess;
}

template <bool DIRECT>
hipError_t launch_bins(const BinArgs& a, hipStream_t stream) {
  auto kern = bin_group_kernel<DIRECT>;
  static std::atomic<bool> raised{false};
  if (hipError_t e = raise_lds(kern, sizeof(BinLds), raised); e != hipSuccess) return e;
  LSHMOE_LAUNCH(kern, dim3(DIRECT ? 1 : kBins), dim3(kBinThreads), sizeof(BinLds), stream, a);
  return hipSuccess;
}

// Spreads `bits` key bits evenly over as few radix passes as possible; returns their number.
int plan_digits(int bits, int (&shift)[8], int (&width)[8]) {
  const int passes = (bits + kMaxDigitBits - 1) / kMaxDigitBits;
  for (int i = 0, at = 0; i < passes; ++i) {
    const int w = (bits - at + (passes - i) - 1) / (passes - i);
    shift[i] = at;
    width[i] = w;
    at += w;
  }
  return passes;
}

}  // namespace

bool plan_group(int64_t T, int d, int k, int E, int L, int r, GroupPlan* plan) {
  uint64_t nb = 1;  // (2r)^L, known to be < 2^63 by the caller's check
  for (int l = 0; l < L; ++l) nb *= (uint64_t)(2 * r);
  GroupPlan p{};
  p.N = T * k;
  p.ebits = bits_for((uint64_t)E - 1);
  p.bbits = bits_for(nb - 1);
  const int bits = p.ebits + p.bbits;
  if (bits > 64) return false;
  p.one_bin = p.N <= kSmallMaxN;
  p.tile = 256;                        // the smallest tile that keeps the table within kMaxTiles rows
  while (p.tile < kSortTile && (p.N + p.tile - 1) / p.tile > kMaxTiles) p.tile *= 2;
  p.tiles = (uint32_t)((p.N + p.tile - 1) / p.tile);
  p.bins = !p.one_bin && p.tiles <= (uint32_t)kMaxTiles;
  p.top_shift = p.bins ? (bits > kBinBits ? bits - kBinBits : 0) : bits;   // key bits below the bin
  p.passes = plan_digits(p.top_shift, p.shift, p.width);
  p.first_bin = 0;
  p.spins = 1u << 10;
  p.seg_blocks = (uint32_t)((p.N + kSegTile - 1) / kSegTile);
  size_t off = 0;
  if (!p.one_bin) {   // one workgroup keeps everything in LDS
    for (int i = 0; i < 2; ++i) {
      p.off_key[i] = off;
      off = align256(off + (size_t)p.N * 8);
    }
    for (int i = 0; i < 2; ++i) {
      p.off_idx[i] = off;
      off = align256(off + (size_t)p.N * 4);
    }
  }
  if (p.bins) {
    // The second key buffer is free.  The table (at most 4 N bytes + 1 KB) and behind it the bins' published counts and
    // claims lie there: the sizes that the built-in scratch holds do not shrink for the sake of this route.
    p.off_table = p.off_key[1];
    p.off_blocksum = align256(p.off_table + (size_t)kBins * p.tiles * 4);
    static_assert(4 * (size_t)kSmallMaxN >= 1024 + kSyncWords * 4, "room behind the table at every size of this route");
  } else if (!p.one_bin) {
    p.off_table = off;
    off = align256(off + (size_t)kGroupBins * p.tiles * 4);
    p.off_blocksum = off;   // head counts per numbering tile (+ 1)
    off = align256(off + ((size_t)p.seg_blocks + 1) * 4);
  }
  const size_t windows = 2 * (size_t)((p.N + kCentroidWindow - 1) / kCentroidWindow);
  p.off_partial = off;
  off = align256(off + windows * (size_t)d * 4);
  p.off_counters = off;
  // every numbering tile clears the counters of its whole tile, so the count is rounded up to whole tiles
  off = align256(off + (size_t)p.seg_blocks * (2 * kSegTile / kCentroidWindow) * 4);
  p.total_bytes = off;
  *plan = p;
  return true;
}

hipError_t launch_group(const GroupPlan& plan, const int32_t* expert, const uint64_t* bucket, int k, int E,
                        int32_t* seg_offsets, int32_t* seg_expert, int32_t* expert_offsets, int32_t* perm,
                        int32_t* seg_of, int32_t* num_segments, char* ws, hipStream_t stream) {
  const uint32_t N = (uint32_t)plan.N;
  uint64_t* keybuf[2] = {(uint64_t*)(ws + plan.off_key[0]), (uint64_t*)(ws + plan.off_key[1])};
  int32_t* idxbuf[2] = {(int32_t*)(ws + plan.off_idx[0]), (int32_t*)(ws + plan.off_idx[1])};
  uint32_t* table = (uint32_t*)(ws + plan.off_table);
  uint32_t* blocksum = (uint32_t*)(ws + plan.off_blocksum);
  KeySource src{expert, bucket, nullptr, nullptr, (uint32_t)k, (uint32_t)E, plan.bbits};

  if (plan.one_bin || plan.bins) {
    BinArgs a{};
    a.src = src;
    a.table = table;
    a.tile_key = keybuf[0];
    a.tile_idx = idxbuf[0];
    a.tiles = plan.tiles;
    a.tile_bits = bits_for((uint64_t)plan.tile - 1);
    a.N = N;
    a.E = (uint32_t)E;
    a.bbits = plan.bbits;
    a.top_shift = plan.top_shift;
    a.passes = plan.passes;
    for (int p = 0; p < plan.passes; ++p) {
      a.shift[p] = plan.shift[p];
      a.width[p] = plan.width[p];
    }
    a.sub_shift = plan.top_shift > kSubBits ? plan.top_shift - kSubBits : 0;
    a.big_idx = idxbuf[1];
    a.seg_offsets = seg_offsets; a.seg_expert = seg_expert; a.expert_offsets = expert_offsets;
    a.perm = perm; a.seg_of = seg_of; a.num_segments = num_segments;
    a.sync = blocksum;
    a.window_counters = (uint32_t*)(ws + plan.off_counters);
    a.first_bin = plan.first_bin;
    a.spins = plan.spins;
    a.n_counters = plan.seg_blocks * (uint32_t)(2 * kSegTile / kCentroidWindow);
    if (plan.one_bin) return launch_bins<true>(a, stream);
    const dim3 grid(plan.tiles), block(kSortThreads);
#define LSHMOE_TILES(TILE) \
    LSHMOE_LAUNCH((tile_bin_kernel<TILE>), grid, block, 0, stream, src, N, plan.top_shift, table, keybuf[0], idxbuf[0], a.sync)
    if (plan.tile == 256) LSHMOE_TILES(256);
    else if (plan.tile == 512) LSHMOE_TILES(512);
    else if (plan.tile == 1024) LSHMOE_TILES(1024);
    else LSHMOE_TILES(2048);
#undef LSHMOE_TILES
    return launch_bins<false>(a, stream);
  }

  const uint64_t* sorted_key = nullptr;
  const uint32_t nblk = plan.tiles;    // of kSortTile keys here
  for (int p = 0; p < plan.passes; ++p) {
    const bool last = p == plan.passes - 1;
    uint64_t* dkey = keybuf[p & 1];
    int32_t* didx = last ? perm : idxbuf[p & 1];
    const int shift = plan.shift[p];
    const uint32_t mask = (1u << plan.width[p]) - 1u;
    if (p == 0)
      LSHMOE_LAUNCH((sort_hist_kernel<true>), dim3(nblk), dim3(kSortThreads), 0, stream, src, N, shift, mask, nblk, table);
    else
      LSHMOE_LAUNCH((sort_hist_kernel<false>), dim3(nblk), dim3(kSortThreads), 0, stream, src, N, shift, mask, nblk, table);
    LSHMOE_LAUNCH(scan_kernel, dim3(1), dim3(1024), 0, stream, table, (mask + 1u) * nblk);
    const hipError_t e = p == 0 ? launch_scatter<true>(src, N, shift, mask, nblk, table, dkey, didx, stream)
                                : launch_scatter<false>(src, N, shift, mask, nblk, table, dkey, didx, stream);
    if (e != hipSuccess) return e;
    src.key = dkey;
    src.idx = didx;
    sorted_key = dkey;
  }
  const uint32_t sblk = plan.seg_blocks;
  LSHMOE_LAUNCH(seg_count_kernel, dim3(sblk), dim3(kSegThreads), 0, stream, sorted_key, N, sblk, blocksum,
                     (uint32_t*)(ws + plan.off_counters));
  if (sblk <= (uint32_t)kSelfPrefixMaxTiles) {
    LSHMOE_LAUNCH(seg_write_kernel<true>, dim3(sblk), dim3(kSegThreads), 0, stream, sorted_key, perm, N,
                       (uint32_t)E, plan.bbits, blocksum, seg_offsets, seg_expert, expert_offsets, seg_of,
                       num_segments);
  } else {
    LSHMOE_LAUNCH(scan_kernel, dim3(1), dim3(1024), 0, stream, blocksum, sblk + 1);
    LSHMOE_LAUNCH(seg_write_kernel<false>, dim3(sblk), dim3(kSegThreads), 0, stream, sorted_key, perm, N,
                       (uint32_t)E, plan.bbits, blocksum, seg_offsets, seg_expert, expert_offsets, seg_of,
                       num_segments);
  }
  return hipGetLastError();
}

#undef LSHMOE_LAUNCH

}  // namespace lshmoe
