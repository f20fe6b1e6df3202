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

__device__ __forceinline__ uint64_t key_of(const KeySource& src, int32_t id) {   // the key of an assignment
  uint64_t key;
  int32_t unused;
  load_item<true>(src, (uint32_t)id, key, unused);
  return key;
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
// Words that the workgroups of bin_group_kernel exchange, zero on entry.  parts: the most parts that large bins are cut
// into (max_parts).
constexpr uint32_t kClaimStride = 8;         // four claims to a 128-byte line: exchanges on one word or line queue up
constexpr uint32_t kCountAt = 0;             // published cluster counts: bins, then parts
constexpr uint32_t kArriveAt = 2 * kBins;    // parts of a bin that have their count, and the sum of the counts
constexpr uint32_t kTotalAt = 3 * kBins;     // keys of the bins (published when some bin may be large)
constexpr uint32_t kClaimAt = 4 * kBins;     // claims: bins, then parts
constexpr int kPeaks = kSortThreads / kWave;
__host__ __device__ constexpr uint32_t sync_words(uint32_t parts) { return kClaimAt + (kBins + parts) * kClaimStride; }

__device__ __forceinline__ uint32_t wave_max(uint32_t v) {   // in the last lane: the largest of the lanes
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));   // row_shr:1
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));   // row_shr:2
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));   // row_shr:4
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));   // row_shr:8
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));   // row_bcast:15 into rows 1 and 3
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));   // row_bcast:31 into rows 2 and 3
  return v;
}

template <int TILE>
__global__ __launch_bounds__(kSortThreads) void tile_bin_kernel(KeySource src, uint32_t N, int shift,
                                                                uint32_t* __restrict__ table, uint64_t* __restrict__ dst_key,
                                                                int32_t* __restrict__ dst_idx, uint32_t* __restrict__ sync,
                                                                uint32_t parts, uint32_t* __restrict__ peak) {
  constexpr int kItems = TILE / kSortThreads, kGroups = TILE / kWave;
  static_assert(TILE <= 0xffff, "start and count of a bin in a tile share a word");
  __shared__ uint32_t cnt[kGroups][kBins];   // keys of a bin in a group of 64; then the group's first position of it
  __shared__ uint32_t wave_sum[kSortThreads / kWave];
  if (blockIdx.x == 0) {                     // what bin_group_kernel expects to find cleared
    static_assert(kBins == kSortThreads, "a word of each kind per thread");
    sync[kCountAt + threadIdx.x] = 0;
    sync[kCountAt + kBins + threadIdx.x] = 0;
    sync[kArriveAt + threadIdx.x] = 0;
    sync[kTotalAt + threadIdx.x] = 0;
    sync[kClaimAt + threadIdx.x * kClaimStride] = 0;
    if (threadIdx.x < parts) sync[kClaimAt + (kBins + threadIdx.x) * kClaimStride] = 0;
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
    const uint32_t most = wave_max(total);   // of this wave's quarter of the bins
    if (lane == 63) peak[blockIdx.x * kPeaks + wave] = most;
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
// lowest bin that is still open: if that succeeds, the bin's own workgroup has not started (and will leave it alone when
// it does), and the waiting workgroup does the bin itself - nothing before it is open, so without a wait - and then
// returns to its own; if not, the bin's owner is running and will publish.  So every wait ends, whatever else runs on
// the GPU and in whatever order workgroups are started.  (A ticket counter gives the same, but 256 workgroups adding
// to one word took 3.4 us.)  Counts, claims and sizes of bins are the only data exchanged inside the launch, as relaxed
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
// with sub-bins, 10.5 without).  Everything must fit the 128 registers of a 1024-thread workgroup: a kernel that spills
// a few of them to scratch memory starts 3 to 8 us later, which is why kBinCap is not 8192.
//
// Large bins, of more than kBinCap keys.  There is none when the largest counts that the tiles have of any bin add up to no
// more than that; this costs a few words per tile and is so on balanced inputs.  Otherwise every workgroup publishes the
// size of its bin, and all of them learn which bins are large.
//   One key makes up most of the bin (padding; 1024 samples say so): its assignments go straight to their place in perm
//     without a sort and the rest is sorted in LDS, by the bin's own workgroup.
//   Else the bin is cut into parts of about 1024 keys (up to 2048 on the largest inputs: there are no more parts than
//     workgroups) by key ranges, at equal steps of a sorted sample of its keys.  The bin's workgroup does the first part,
//     workgroups of small bins the others, after they have published their own bin's count and before they write that bin,
//     whose sorted ids are set aside in perm.  For a part the sample is sorted and the bin walked to pick out the part's
//     keys; then the part is like a bin, with a count and a claim of its own; the last part of a bin to be counted
//     publishes the bin's count.  A key that is frequent itself begins a part (the sample has it at a step) and takes the
//     way of the padding there.
// A part that is large all the same (the sample missed it) is radix sorted through global memory by its workgroup.
// Measured, compress call at d = 8, against one workgroup per bin, whatever its size, and (in brackets) the four launches
// before: 65536 and 131072 assignments of a Zipf gate over 64 experts, whose first holds a quarter, 54 -> 44 us (48) and
// 64 -> 50 us (56); 131072 of one expert of 64 243 -> 60 us (174); half of 131072 with one expert of 256 488 -> 93 us (255).
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
constexpr int kBigRounds = 4;                       // rounds of 64 keys a wave has in flight on a walk
constexpr uint32_t kSampleOnceMax = 1u << 16;       // keys of a bin up to which a sample of 1024 cuts it into parts; else 4096
constexpr int kTotalLooks = 64;                     // looks at the sizes of the bins before they are added up from the table
constexpr uint32_t kPartKeys = 1024;                // keys of a part, at least
constexpr uint32_t kWaveSlot = kBinCap / kBinWaves; // LDS places of a wave on a walk
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

struct BinArgs {               // what is needed first comes first: the fields arrive by cache lines
  uint32_t* sync;             // sync_words(), zero on entry (not used with DIRECT)
  const uint32_t* table;      // [tiles][kBins]: start of the bin inside the tile | keys << 16
  const uint4* peak;          // [tiles]: the largest count in each quarter of the bins
  uint32_t tiles, tile_bits;
  const uint64_t* tile_key;   // the tiles, each sorted by bin
  const int32_t* tile_idx;
  int passes;                 // radix passes over the key bits below the bin
  int sub_shift;              // sub-bin of a key is (key >> sub_shift) & (kSubBins - 1)
  uint32_t spins;             // looks at the open counts before a workgroup tries to take one of them over
  uint32_t N, E;
  int bbits, top_shift;       // bin of a key is key >> top_shift
  int32_t *seg_offsets, *seg_expert, *expert_offsets, *perm, *seg_of, *num_segments;
  uint32_t* window_counters;  // cleared here for the centroid step
  uint32_t n_counters;
  uint32_t first_bin;         // SKIP: see bin_group_kernel
  int shift[8], width[8];
  uint32_t part_keys;         // keys of a part, on average
  int32_t* big_idx;           // the ids of a part that is sorted through global memory go between here and perm
  KeySource src;              // DIRECT, and keys that are made again
};

// A value that all lanes have in common, kept in scalar registers: what comes out of LDS would sit in vector ones.
__device__ __forceinline__ uint32_t scalar(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ uint64_t scalar(uint64_t v) {
  return (uint64_t)scalar((uint32_t)(v >> 32)) << 32 | scalar((uint32_t)v);
}

// Code that balanced inputs do not need goes behind the rest: what they run is read into the instruction cache in one piece.
__device__ __forceinline__ bool seldom(bool v) { return __builtin_expect(v, false); }

// threadIdx.x, as a value that the compiler must take for a new one: what it computes from it would otherwise be moved out of
// the loop over a workgroup's turns, and has to be spilled there.
__device__ __forceinline__ uint32_t own_thread() {
  uint32_t tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  __builtin_assume(tid < (uint32_t)kBinThreads);
  return tid;
}

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
  const uint32_t tid = own_thread(), wave = tid >> 6;
  const uint32_t inc = wave_inclusive_sum(v);
  if ((tid & 63) == 63) wave_sum[wave] = inc;
  __syncthreads();
  uint32_t before = 0;
  total = 0;
#pragma unroll
  for (uint32_t w = 0; w < (uint32_t)kBinWaves; ++w) {
    const uint32_t t = wave_sum[w];
    if (w < wave) before += t;
    total += t;
  }
  total = scalar(total);
  return before + inc - v;
}

// Whether any thread of the workgroup says so.  One barrier inside; said may be used again behind the next one.
__device__ __forceinline__ bool workgroup_any(bool v, uint32_t* said /*[kBinWaves], 16-byte aligned*/) {
  const uint32_t tid = own_thread();
  const bool any = __any(v);
  if ((tid & 63) == 0) said[tid >> 6] = any ? 1u : 0u;
  __syncthreads();
  uint32_t all = 0;
#pragma unroll
  for (int w = 0; w < kBinWaves; w += 4) {
    const uint4 q = *reinterpret_cast<const uint4*>(said + w);
    all |= q.x | q.y | q.z | q.w;
  }
  return scalar(all) != 0u;
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

// What a workgroup works on: a whole bin, item i for bin i, or a part, item kBins + i for part i of all.
constexpr uint32_t kNoItem = ~0u;

struct BinState {                    // a sorted bin or part; in LDS, so that it takes no registers while others are sorted
  uint32_t n, start;                 // keys, first position
  uint32_t less, equal;              // in LDS: the first `less` keys come before `equal` ones that are `common`
  uint64_t common;
};

struct BinShared {
  uint32_t wave_sum[3][kBinWaves];
  __align__(16) uint32_t said[3][kBinWaves];
  uint32_t tile_before[kMaxTiles], tile_from[kMaxTiles];   // keys of the bin in earlier tiles; where the tile's begin
  uint4 wave_four[kBinWaves];
  uint32_t head_cnt[65];             // clusters in, then before, a round of one wave (big: its slice); [64]: ... before the common key
  uint32_t claimed, open, my_part, my_bin, interrupted, interrupted_bin;
  uint32_t total[kBins], first_part[kBins];                // when some bin may be large: keys, number of the first part
  BinState state[2];                 // of a bin, of a part
  uint32_t column_n, column_start;   // of the own bin, when some bin may be large
  uint64_t range_lo, range_hi;       // the part's keys: from range_lo on (but for the first part), below range_hi (but for the last)
  uint64_t sub_base;                 // its sub-bins: (key - sub_base) >> sub_shift
  int sub_shift;
  uint32_t aside, aside_heads[kBinWaves];   // clusters of the own bin (top bit: in perm) and its head_cnt, set aside
};

__device__ __forceinline__ uint32_t parts_of(const BinArgs& a, uint32_t n) { return n > (uint32_t)kBinCap ? n / a.part_keys : 0u; }

// Learns the sizes of all bins (from their workgroups; from the table if one does not come) and numbers the parts of the
// large ones.  sh.my_part: the part that falls to this workgroup, or kNoItem, and its bin.
__device__ __forceinline__ void number_parts(const BinArgs& a, uint32_t own, BinShared& sh) {
  const uint32_t tid = own_thread();
  uint32_t v = 0;
  bool all = false;
  for (int look = 0; look < kTotalLooks && !all; ++look) {
    if (tid < kBins && v == 0) v = __hip_atomic_load(&a.sync[kTotalAt + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    all = !workgroup_any(tid < kBins && v == 0, sh.said[look & 1]);
  }
  if (tid < kBins) sh.total[tid] = all ? v - 1u : 0u;
  if (tid == 0) sh.my_part = kNoItem;
  __syncthreads();
  if (!all) {
    constexpr uint32_t kRows = kBinThreads / kBins, kBatch = 8;   // rows of the table side by side, loads in flight
    const uint32_t bin = tid % kBins;
    uint32_t sum = 0;
    for (uint32_t t0 = tid / kBins; t0 < a.tiles; t0 += kRows * kBatch) {
      uint32_t e[kBatch];
#pragma unroll
      for (uint32_t q = 0; q < kBatch; ++q) {
        const uint32_t t = t0 + q * kRows;
        e[q] = t < a.tiles ? a.table[t * kBins + bin] : 0u;
      }
#pragma unroll
      for (uint32_t q = 0; q < kBatch; ++q) sum += e[q] >> 16;
    }
    atomicAdd(&sh.total[bin], sum);
    __syncthreads();
  }
  // Numbers of the parts, and of the workgroups for them: part 0 of a bin is its own workgroup's, the others fall to those
  // whose bins are not large (there are no more than 256 parts in all, so they are enough), of at most average size first.
  const uint32_t n = tid < kBins ? sh.total[tid] : 0u, parts = parts_of(a, n);
  const bool average = tid < kBins && parts == 0 && n <= min(a.N / kBins, (uint32_t)kBinThreads);
  const bool more = tid < kBins && parts == 0 && !average;
  uint32_t all_of;
  const uint32_t at = bin_exclusive_scan(parts << 20 | (average ? 1u << 10 : 0u) | (more ? 1u : 0u), sh.wave_sum[0], all_of);
  const uint32_t first = at >> 20, averages = (at >> 10) & 1023u, mores = at & 1023u;
  if (tid < kBins) sh.first_part[tid] = first;
  if (tid == own) sh.open = average ? averages : more ? ((all_of >> 10) & 1023u) + mores : kNoItem;   // which of them this is
  __syncthreads();
  const uint32_t me = sh.open, first_other = first - (tid - averages - mores);   // large bins before: one part each is not for others
  if (tid < kBins && parts != 0) {
    const uint32_t q = tid == own ? 0u : 1u + (me - first_other);
    if (tid == own || (me != kNoItem && me >= first_other && q < parts)) {
      sh.my_part = kBins + first + q;
      sh.my_bin = tid;
    }
  }
  __syncthreads();
}

// The code of a workgroup: the whole input; a bin, none being large; anything when some bin may be large.  The second is
// what balanced inputs run: with the third's code in between it took 1 us more to arrive.
enum { kDirect, kBalanced, kCrowded };

// Collects and sorts a bin or part and counts its clusters.  taken: not 0 in thread 0 when it belongs to another
// workgroup.  own: the item is the workgroup's own bin and this the first turn.
// False: the item is another's, or the bin is done in parts, or the part's bin as a whole (LDS still holds what was sorted
// before then), or some bin may be large, which kBalanced finds on the first turn (crowded).  True: heads are its clusters;
// big: the sorted ids are in perm, else keys and ids are in LDS.  With kCrowded the workgroup's own bin, if it is large and
// done in parts, becomes its first part.
template <int MODE>
__device__ __forceinline__ bool sort_item(const BinArgs& a, uint32_t& item, uint32_t bin, uint32_t taken, bool own,
                                          bool& crowded, uint32_t& heads, bool& big, BinLds& m, BinShared& sh) {
  constexpr bool DIRECT = MODE == kDirect, CROWDED = MODE == kCrowded;
  uint32_t tid = own_thread();
  int lane = tid & 63, wave = tid >> 6;
  bool part = CROWDED && item >= kBins;
  uint32_t n = a.N, start = 0;
  if (CROWDED && own) {                             // kBalanced has been here
    n = scalar(sh.column_n);
    start = scalar(sh.column_start);
  } else if (!DIRECT) {
    static_assert(kMaxTiles == kBins && kMaxTiles % 64 == 0, "one tile per thread of the first waves");
    uint32_t keys = 0, first = 0, most = 0;
    if (tid < a.tiles) {
      const uint32_t e = a.table[tid * kBins + bin];
      if (own) {
        const uint4 p = a.peak[tid];
        most = max(max(p.x, p.y), max(p.z, p.w));
      }
      first = e & 0xffffu;
      keys = e >> 16;
    }
    const uint32_t inc_most = wave_inclusive_sum(most);
    const uint32_t inc = wave_inclusive_sum(keys), inc_first = wave_inclusive_sum(first);
    if (lane == 63) {
      sh.wave_sum[0][wave] = inc;
      sh.wave_sum[1][wave] = inc_first;
      sh.wave_sum[2][wave] = inc_most;
    }
    __syncthreads();
    uint32_t before = inc - keys, bound = 0;
    n = 0;
#pragma unroll
    for (int w = 0; w < kMaxTiles / 64; ++w) {      // later waves hold no tile
      const uint32_t c = sh.wave_sum[0][w];
      if (w < wave) before += c;
      n += c;
      start += sh.wave_sum[1][w];
      bound += sh.wave_sum[2][w];
    }
    n = scalar(n);
    start = scalar(start);
    if (tid < a.tiles) {
      sh.tile_before[tid] = before;
      sh.tile_from[tid] = (tid << a.tile_bits) + first - before;   // source of element i of the bin: tile_from + i
    }
    if (tid == 0) sh.claimed = taken == 0;
    if (MODE == kBalanced && own) {
      crowded = scalar(bound) > (uint32_t)kBinCap;
      if (seldom(crowded) && tid == 0) {
        sh.column_n = n;
        sh.column_start = start;
        __hip_atomic_store(&a.sync[kTotalAt + bin], n + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    __syncthreads();
  }
  if (MODE == kBalanced && seldom(crowded)) return false;
  if (!DIRECT && seldom(scalar(sh.claimed) == 0u)) return false;   // done by a workgroup that waited for it
  auto tile_of = [&](uint32_t i, uint32_t lo, uint32_t hi) {    // last tile with tile_before <= i, of those from lo on before hi
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (sh.tile_before[mid] <= i) lo = mid; else hi = mid;
    }
    return lo;
  };
  // element i < n of the bin, in assignment order
  auto fetch = [&](uint32_t i, uint32_t tile_lo, uint32_t tile_hi, uint64_t& key, int32_t& idx) {
    if (DIRECT) {
      load_item<true>(a.src, i, key, idx);
    } else {
      const uint32_t lo = tile_of(i, tile_lo, tile_hi);
      key = a.tile_key[sh.tile_from[lo] + i];
      idx = a.tile_idx[sh.tile_from[lo] + i];
    }
  };

  enum { kSample, kPick, kSort };
  int step = kSort;
  bool picked = false;                              // the keys to sort are in LDS
  uint32_t common_heads = 0;
  big = false;
  uint64_t common = 0;
  if (CROWDED && n > (uint32_t)kBinCap) {
    uint64_t key, own_key;
    int32_t idx;
    fetch((uint32_t)(((uint64_t)n * (2u * lane + 1u)) >> 7), 0, a.tiles, key, idx);         // 64 samples, the same in every wave
    fetch((uint32_t)(((uint64_t)n * (2u * tid + 1u)) >> 11), 0, a.tiles, own_key, idx);     // 1024, one per thread
    static_assert(kBinThreads == 1 << 10, "samples per workgroup");
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
    uint32_t hits;
    bin_exclusive_scan(own_key == common ? 1u : 0u, sh.wave_sum[0], hits);
    __syncthreads();
    // the other keys, by the sample, fill half of LDS at most: twice as many still fit
    if ((uint64_t)(kBinThreads - hits) * n <= (uint64_t)kBinThreads * (kBinCap / 2)) {
      if (part) return false;
      step = kPick;
    } else {
      if (!part && !own) return false;
      if (n <= kSampleOnceMax) {                    // the sample in hand will do: 16 keys and more per part
        m.key[tid] = own_key;
        m.idx[tid] = (int32_t)tid;
        picked = true;
      }
      if (!part) {
        number_parts(a, bin, sh);
        item = scalar(sh.my_part);
        part = true;
        if (tid == 0) sh.claimed = atomicExch(&a.sync[kClaimAt + item * kClaimStride], 1u) == 0u;
        __syncthreads();
        if (!sh.claimed) return false;
      }
      step = kSample;
    }
  }

  BinState& st = sh.state[part ? 1 : 0];
  if (tid == 0) {
    st.n = n;
    st.start = start;
    st.less = n;
    st.equal = 0;
    st.common = common;
  }
  // the places of the sample are computed from st.n (kPick has a barrier of its own before it reads st)
  if (CROWDED && step == kSample) __syncthreads();
  uint32_t rest = n;                                // keys to sort
  for (;;) {
    const uint32_t tid = own_thread();
    const int lane = tid & 63, wave = tid >> 6;
    const uint64_t lt_mask = (1ull << lane) - 1ull;
    if (CROWDED && step == kPick) {
      // the keys of a part, or of a bin that is mostly one key
      __syncthreads();
      const uint32_t n = scalar(st.n), bin_start = scalar(st.start);
      bool has_lo = false, has_hi = false;
      uint64_t range_lo = 0, range_hi = 0;
      if (part) {
        const uint32_t q = item - kBins - scalar(sh.first_part[bin]);
        has_lo = q > 0;
        has_hi = q + 1 < parts_of(a, n);
        range_lo = scalar(sh.range_lo);
        range_hi = scalar(sh.range_hi);
      }
      const uint64_t common = part ? range_lo : scalar(st.common);
      const uint32_t hslice = ((n + kBinWaves - 1) / kBinWaves + 63u) & ~63u;
      const uint32_t hlo = scalar(min((uint32_t)wave * hslice, n)), hhi = min(hlo + hslice, n);
      uint32_t tile_lo = 0, tile_hi = a.tiles;      // tiles of the slice; finding them takes longer than a short walk gains
      if (n > 4u * kBinCap) {
        tile_lo = scalar(tile_of(min(hlo, n - 1), 0, a.tiles));
        tile_hi = scalar(tile_of(max(hhi, 1u) - 1, 0, a.tiles)) + 1;
      }
      auto walk = [&](auto&& f) {                   // f(valid, key, idx) for every round of the wave's slice
        for (uint32_t b = hlo; b < hhi; b += kBigRounds * 64) {
          uint64_t k[kBigRounds];
          int32_t id[kBigRounds];
#pragma unroll
          for (int q = 0; q < kBigRounds; ++q) fetch(min(b + q * 64 + lane, hhi - 1), tile_lo, tile_hi, k[q], id[q]);
#pragma unroll
          for (int q = 0; q < kBigRounds; ++q) f(b + q * 64 + lane < hhi, k[q], id[q]);
        }
      };
      // Keys before the part, of it, of the common key, of the part before that.  What is to be sorted goes to the wave's
      // places in LDS as long as there are any left; the ids of a bin's common key, if the bin is not too large, go to
      // those of the wave's slice where the counters of the sort will be.
      uint32_t below = 0, in = 0, eq = 0, lt = 0;
      constexpr uint32_t kWaveIds = sizeof(m.cnt) / sizeof(int32_t) / kBinWaves;
      const bool ids_kept = !part && n <= kWaveIds * kBinWaves;
      int32_t* wave_ids = reinterpret_cast<int32_t*>(&m.cnt[0][0]) + wave * kWaveIds;
      walk([&](bool valid, uint64_t k, int32_t id) {
        const bool low = has_lo && k < range_lo, inside = valid && !low && !(has_hi && k >= range_hi);
        const uint64_t r = __ballot(inside), e = __ballot(inside && k == common), sort = part ? r : r & ~e;
        const uint32_t at = (part ? in : in - eq) + (uint32_t)__popcll(sort & lt_mask);
        if ((sort >> lane & 1ull) != 0 && at < kWaveSlot) {
          m.key[wave * kWaveSlot + at] = k;
          m.idx[wave * kWaveSlot + at] = id;
        }
        if (ids_kept && inside && k == common) wave_ids[eq + (uint32_t)__popcll(e & lt_mask)] = id;
        below += (uint32_t)__popcll(__ballot(valid && low));
        in += (uint32_t)__popcll(r);
        eq += (uint32_t)__popcll(e);
        lt += (uint32_t)__popcll(__ballot(inside && k < common));
      });
      if (lane == 0) sh.wave_four[wave] = make_uint4(in, eq, lt, below);
      __syncthreads();
      uint32_t rest_at = 0, eq_at = 0, in_all = 0, eq_all = 0, lt_all = 0, below_all = 0, in_most = 0;
#pragma unroll
      for (int w = 0; w < kBinWaves; ++w) {
        const uint4 c = sh.wave_four[w];
        if (w < wave) {
          rest_at += c.x;
          eq_at += c.y;
        }
        in_all += c.x;
        eq_all += c.y;
        lt_all += c.z;
        below_all += c.w;
        in_most = max(in_most, part ? c.x : c.x - c.y);
      }
      in_all = scalar(in_all);
      eq_all = scalar(eq_all);
      rest_at = scalar(rest_at);
      eq_at = scalar(eq_at);
      const uint32_t start = bin_start + scalar(below_all);
      uint32_t less = in_all, equal = 0;            // rest[0, less) comes before the common key, `equal` keys are it
      if (in_all > (uint32_t)kBinCap) {
        if (in_all - eq_all <= (uint32_t)kBinCap) {
          less = scalar(lt_all);
          equal = eq_all;
          rest_at -= eq_at;
        } else {
          big = true;
        }
      }
      if ((part || ids_kept) && !big && scalar(in_most) <= kWaveSlot) {   // all of them are there: closed up
        static_assert(kWaveSlot == kBinItems * 64, "a wave's places in its registers");
        uint64_t k[kBinItems];
        int32_t id[kBinItems];
#pragma unroll
        for (int q = 0; q < kBinItems; ++q) {
          k[q] = m.key[wave * kWaveSlot + q * 64 + lane];
          id[q] = m.idx[wave * kWaveSlot + q * 64 + lane];
        }
        if (!part)
          for (uint32_t i = lane; i < eq; i += 64) a.perm[start + less + eq_at + i] = wave_ids[i];
        __syncthreads();
        const uint32_t here = part ? in : in - eq;
#pragma unroll
        for (int q = 0; q < kBinItems; ++q) {
          if (q * 64 + (uint32_t)lane < here) {
            m.key[rest_at + q * 64 + lane] = k[q];
            m.idx[rest_at + q * 64 + lane] = id[q];
          }
        }
      } else {                                      // another walk, that knows the places
        int32_t* ids = ((a.passes & 1) ? a.big_idx : a.perm) + start;   // big: the last pass leaves the ids in perm
        walk([&](bool valid, uint64_t k, int32_t id) {
          const bool inside = valid && !(has_lo && k < range_lo) && !(has_hi && k >= range_hi);
          const bool same = equal != 0 && k == common;
          const uint64_t e = __ballot(inside && same), r = __ballot(inside && !same);
          if (inside && same) a.perm[start + less + eq_at + (uint32_t)__popcll(e & lt_mask)] = id;
          if (inside && !same) {
            const uint32_t at = rest_at + (uint32_t)__popcll(r & lt_mask);
            if (big) {
              ids[at] = id;
            } else {
              m.key[at] = k;
              m.idx[at] = id;
            }
          }
          eq_at += (uint32_t)__popcll(e);
          rest_at += (uint32_t)__popcll(r);
        });
      }
      rest = in_all - equal;
      common_heads = equal != 0 ? 1u : 0u;
      picked = true;
      step = kSort;
      if (tid == 0) {                               // every thread has read the bin's
        st.n = in_all;
        st.start = start;
        st.less = less;
        st.equal = equal;
        st.common = common;
      }
      __syncthreads();
      if (big) break;
    }
    uint64_t key[kBinItems];
    int32_t idx[kBinItems];
    uint32_t zero = 0;                              // not a constant that sits in registers through the turns
    asm volatile("" : "+v"(zero));
    if (CROWDED && step == kSample) rest = picked ? (uint32_t)kBinThreads : (uint32_t)kBinCap;
#pragma unroll
    for (int q = 0; q < kBinItems; ++q) {
      const uint32_t i = tid + q * kBinThreads;
      if (i < rest) {
        if (CROWDED && picked) {
          key[q] = m.key[i];
          idx[q] = m.idx[i];
        } else {
          fetch(CROWDED && step == kSample ? (uint32_t)(((uint64_t)i * st.n) / kBinCap) : i, 0, a.tiles, key[q], idx[q]);
        }
      }
    }
    if (CROWDED && picked) __syncthreads();
    const uint32_t slice = ((rest + kBinWaves - 1) / kBinWaves + 63u) & ~63u;   // keys per wave, whole rounds
    const uint32_t wlo = min((uint32_t)wave * slice, rest), whi = min(wlo + slice, rest);
    bool sorted = false;
    if (a.passes > 1) {
      constexpr int kPer = kSubBins / kBinThreads;    // neighbouring sub-bins of a thread
      static_assert(kPer == 4, "moved 16 bytes at a time");
      const bool ranged = CROWDED && part && step == kSort;    // of a part's range
      const uint64_t sub_base = ranged ? scalar(sh.sub_base) : 0;
      const int sub_shift = ranged ? (int)scalar((uint32_t)sh.sub_shift) : a.sub_shift;
      auto sub_of = [&](uint64_t k) { return (uint32_t)((k - sub_base) >> sub_shift) & (kSubBins - 1); };
      reinterpret_cast<uint4*>(m.sub.cnt)[tid] = make_uint4(zero, zero, zero, zero);
      __syncthreads();
      uint32_t slot[kBinItems];                       // sub-bin << 16 | arrival
#pragma unroll
      for (int q = 0; q < kBinItems; ++q)
        if (tid + q * kBinThreads < rest) {
          const uint32_t sub = sub_of(key[q]);
          slot[q] = atomicAdd(&m.sub.cnt[sub], 1u) | sub << 16;
        }
      __syncthreads();
      const uint4 c = reinterpret_cast<const uint4*>(m.sub.cnt)[tid];
      const uint32_t most = max(max(c.x, c.y), max(c.z, c.w));
      if (!workgroup_any(most > kCrowdPerPass * (uint32_t)a.passes, sh.said[2])) {
        uint32_t unused;
        const uint32_t run = bin_exclusive_scan(c.x + c.y + c.z + c.w, sh.wave_sum[0], unused);
        reinterpret_cast<uint4*>(m.sub.base)[tid] = make_uint4(run, run + c.x, run + c.x + c.y, run + c.x + c.y + c.z);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kBinItems; ++q) {
          if (tid + q * kBinThreads < rest) {
            const uint32_t at = m.sub.base[slot[q] >> 16] + (slot[q] & 0xffffu);
            m.key[at] = key[q];
            m.idx[at] = idx[q];
          }
        }
        __syncthreads();
        uint32_t rank[kBinItems];
#pragma unroll
        for (int q = 0; q < kBinItems; ++q) {
          if (tid + q * kBinThreads < rest) {
            const uint32_t sub = slot[q] >> 16;
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
          reinterpret_cast<uint4*>(&m.cnt[0][0])[i] = make_uint4(zero, zero, zero, zero);
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
    if (!CROWDED || step == kSort) break;
    // the range of the part: steps of the sorted sample
    if (tid == 0) {
      const uint32_t parts = parts_of(a, st.n), q = item - kBins - sh.first_part[bin];
      uint64_t lo = (uint64_t)bin << a.top_shift, hi = lo + (1ull << a.top_shift);   // hi: 0 at the end of 64 bits
      if (q > 0) sh.range_lo = lo = m.key[q * rest / parts];
      if (q + 1 < parts) sh.range_hi = hi = m.key[(q + 1) * rest / parts];
      sh.sub_base = lo;
      const uint64_t span = hi - lo - 1;            // an empty part has no use for it
      sh.sub_shift = max(64 - kSubBits - (int)__clzll((long long)span), 0);
    }
    step = kPick;
  }
  tid = own_thread();
  lane = tid & 63;
  wave = tid >> 6;
  if (!CROWDED || !big) {
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
    heads = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63) + common_heads;
    __syncthreads();
    if (wave == 0) sh.head_cnt[lane] = inc - mine;   // read after the barriers of the wait for the bins before
  } else {
    // radix passes through global memory, of ids alone: the keys are made from the inputs again on every walk, so that
    // the workspace holds no further key buffers.  Every wave walks its slice 64 keys at a time, twice per pass.
    const uint32_t n = scalar(st.n), start = scalar(st.start), zero = 0;
    const uint64_t lt_mask = (1ull << lane) - 1ull;
    const uint32_t slice = ((n + kBinWaves - 1) / kBinWaves + 63u) & ~63u;
    const uint32_t wlo = min((uint32_t)wave * slice, n), whi = min(wlo + slice, n);
    for (int p = 0; p < a.passes; ++p) {
      const int shift = a.shift[p], width = a.width[p];
      const uint32_t mask = (1u << width) - 1u;
      const bool to_perm = ((a.passes - 1 - p) & 1) == 0;
      const int32_t* sidx = (to_perm ? a.big_idx : a.perm) + start;
      int32_t* didx = (to_perm ? a.perm : a.big_idx) + start;
      for (int i = tid; i < kBinWaves * kGroupBins / 4; i += kBinThreads)
        reinterpret_cast<uint4*>(&m.cnt[0][0])[i] = make_uint4(zero, zero, zero, zero);
      __syncthreads();
      for (uint32_t b = wlo; b < whi; b += kBigRounds * 64) {   // several rounds of loads in flight
        uint64_t key[kBigRounds];
#pragma unroll
        for (int q = 0; q < kBigRounds; ++q) key[q] = key_of(a.src, sidx[min(b + q * 64 + lane, n - 1)]);
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
          key[q] = key_of(a.src, idx[q]);
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
        key[q] = key_of(a.src, ids[i]);
        prev[q] = key_of(a.src, ids[i == 0 ? 0 : i - 1]);
      }
#pragma unroll
      for (int q = 0; q < kBigRounds; ++q) {
        const uint32_t i = b + q * 64 + lane;
        mine += (uint32_t)__popcll(__ballot(i < whi && (i == 0 || key[q] != prev[q])));
      }
    }
    const uint32_t heads_before = bin_exclusive_scan(lane == 0 ? mine : 0u, sh.wave_sum[0], heads);
    if (lane == 0) sh.head_cnt[wave] = heads_before;   // before this wave's slice
  }
  if (DIRECT) __syncthreads();
  return true;
}

// Writes the outputs of a sorted bin or part; `base` clusters come before it.
template <int MODE>
__device__ __forceinline__ void write_item(const BinArgs& a, uint32_t item, uint32_t bin, uint32_t n, uint32_t start,
                                           uint32_t heads, uint32_t equal, bool big, uint32_t base, const BinLds& m,
                                           BinShared& sh, const BinState& st) {
  const uint32_t tid = own_thread();
  const int lane = tid & 63, wave = tid >> 6;
  const uint64_t le_mask = ((1ull << lane) - 1ull) | (1ull << lane);
  constexpr bool DIRECT = MODE == kDirect, CROWDED = MODE == kCrowded;
  const uint32_t less = CROWDED && equal != 0 ? scalar(st.less) : n;
  // experts whose first possible key lies in the range: their offsets are written here
  uint32_t x_lo = 0, x_hi = a.E;
  bool last = true;
  if (!DIRECT) {
    const int up = a.bbits - a.top_shift;
    x_lo = up >= 0 ? (bin + (1u << up) - 1u) >> up : bin << -up;
    x_hi = up >= 0 ? (bin + 1u + (1u << up) - 1u) >> up : (bin + 1u) << -up;
    last = bin == kBins - 1;
    if (CROWDED && item >= kBins) {
      auto first_expert = [&](uint64_t k) {         // the first expert whose possible keys begin at k or later
        return (uint32_t)(k >> a.bbits) + ((k & ((1ull << a.bbits) - 1ull)) != 0 ? 1u : 0u);
      };
      const uint32_t q = item - kBins - scalar(sh.first_part[bin]);
      if (q > 0) x_lo = first_expert(scalar(sh.range_lo));
      if (q + 1 < parts_of(a, scalar(sh.total[bin]))) {
        x_hi = first_expert(scalar(sh.range_hi));
        last = false;
      }
    }
    x_lo = min(x_lo, a.E);
    x_hi = min(x_hi, a.E);
  }
  auto emit = [&](uint32_t i, uint64_t key, uint64_t prev, bool head, uint32_t seg, int32_t assignment) {
    if (head) {
      const uint32_t e = (uint32_t)(key >> a.bbits);
      a.seg_offsets[seg] = (int32_t)(start + i);
      a.seg_expert[seg] = (int32_t)e;
      // experts that start (or are empty) between the key before and this one
      for (uint32_t x = i == 0 ? x_lo : (uint32_t)(prev >> a.bbits) + 1u; x <= e; ++x) a.expert_offsets[x] = (int32_t)seg;
    }
    a.seg_of[assignment] = (int32_t)seg;
  };
  uint32_t x_tail = x_lo;                        // experts of this bin behind its last key
  if (!CROWDED || !big) {
    const uint32_t rest = n - equal;
    if (CROWDED && equal != 0) {                            // the cluster of the common key
      if (tid == 0) sh.head_cnt[64] = heads - 1u;
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
        if (!CROWDED || i < less) {
          a.perm[start + i] = idx;
          emit(i, key, prev, head, seg, idx);
        } else {                                    // behind the common key
          if (i == less) sh.head_cnt[64] = seg - base;
          a.perm[start + equal + i] = idx;
          emit(equal + i, key, i == less ? st.common : prev, head, seg + 1u, idx);
        }
      }
    }
    if (CROWDED && equal != 0) {
      __syncthreads();
      const uint32_t seg = base + sh.head_cnt[64];
      if (tid == 0) emit(less, st.common, less == 0 ? st.common : m.key[less - 1], true, seg, a.perm[start + less]);
      for (uint32_t b = tid; b < equal; b += kBigRounds * kBinThreads) {
        int32_t idx[kBigRounds];
#pragma unroll
        for (int q = 0; q < kBigRounds; ++q) idx[q] = a.perm[start + less + min(b + q * kBinThreads, equal - 1)];
#pragma unroll
        for (int q = 0; q < kBigRounds; ++q)
          if (b + q * kBinThreads < equal) a.seg_of[idx[q]] = (int32_t)seg;
      }
      x_tail = max(x_tail, (uint32_t)(st.common >> a.bbits) + 1u);
    }
    if (rest > 0) x_tail = max(x_tail, (uint32_t)(m.key[rest - 1] >> a.bbits) + 1u);
  } else {
    const uint32_t slice = ((n + kBinWaves - 1) / kBinWaves + 63u) & ~63u;
    const uint32_t wlo = min((uint32_t)wave * slice, n), whi = min(wlo + slice, n);
    uint32_t seg = base + sh.head_cnt[wave];
    for (uint32_t b = wlo; b < whi; b += kBigRounds * 64) {
      uint64_t key[kBigRounds], prev[kBigRounds];
      int32_t idx[kBigRounds];
#pragma unroll
      for (int q = 0; q < kBigRounds; ++q) {
        const uint32_t i = min(b + q * 64 + lane, n - 1);
        idx[q] = a.perm[start + i];
        key[q] = key_of(a.src, idx[q]);
        prev[q] = key_of(a.src, a.perm[start + (i == 0 ? 0 : i - 1)]);
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
    x_tail = max(x_tail, (uint32_t)(key_of(a.src, a.perm[start + n - 1]) >> a.bbits) + 1u);
  }
  for (uint32_t x = x_tail + tid; x < x_hi; x += kBinThreads) a.expert_offsets[x] = (int32_t)(base + heads);
  if (tid == 0 && last) {
    a.expert_offsets[a.E] = (int32_t)(base + heads);
    a.seg_offsets[base + heads] = (int32_t)a.N;
    *a.num_segments = (int32_t)(base + heads);
  }
}

// Called by one thread: claims what keeps count number `open` from being published, if nobody has: the bin or part itself,
// or a part of the bin when that is large.
template <int MODE>
__device__ __forceinline__ uint32_t claim_open(const BinArgs& a, const BinShared& sh, uint32_t open) {
  uint32_t* claim = a.sync + kClaimAt;
  if (MODE == kCrowded && open < kBins && sh.total[open] > (uint32_t)kBinCap) {
    const uint32_t first = kBins + sh.first_part[open], parts = parts_of(a, sh.total[open]);
    for (uint32_t i = first; i < first + parts; ++i)
      if (atomicCAS(&claim[i * kClaimStride], 0u, 1u) == 0u) return i;
  }
  return atomicCAS(&claim[open * kClaimStride], 0u, 1u) == 0u ? open : kNoItem;
}

// Waits for the counts that the threads with `watch` look at and adds them up: base are the clusters before the item.
// kNoItem: done; else something was open for long and is claimed now, to be done first (sh.open: the count it keeps back).
// patient: nothing is taken over.
template <int MODE>
__device__ __forceinline__ uint32_t wait_for_counts(const BinArgs& a, BinShared& sh, uint32_t own, bool watch, bool patient,
                                                    bool& numbered, uint32_t& base) {
  const uint32_t tid = own_thread();
  uint32_t v = 0;                                   // one more than the clusters, 0 as long as there is no count
  for (uint32_t spin = 1;; ++spin) {
    if (watch && v == 0) v = __hip_atomic_load(&a.sync[kCountAt + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool open = watch && v == 0;
    if (!workgroup_any(open, sh.said[spin & 1])) break;
    if (!seldom(!patient && spin >= a.spins)) continue;
    spin = 0;
    if (MODE == kCrowded && !numbered) {
      __syncthreads();
      number_parts(a, own, sh);
      numbered = true;
    }
    if (tid == 0) sh.open = kNoItem;
    __syncthreads();
    if (open) atomicMin(&sh.open, tid);             // a bin before a part
    __syncthreads();
    if (tid == 0) sh.claimed = claim_open<MODE>(a, sh, sh.open);
    __syncthreads();
    if (sh.claimed != kNoItem) return scalar(sh.claimed);
  }
  bin_exclusive_scan(v == 0 ? 0u : v - 1u, sh.wave_sum[1], base);
  return kNoItem;
}

// The turns of a workgroup when some bin may be large.  Its own bin is sorted and counted first; a part that falls to the
// workgroup comes next, between the sorting and the writing of the own bin: no workgroup waits for anything while it
// has not published what it has claimed, or has a part still to claim.  What it takes over while it waits needs no takeover
// itself: that waits for workgroups that run.
__device__ __forceinline__ void crowded_turns(uint32_t own, BinLds& m, BinShared& sh) {
  enum : uint32_t {
    kFirstTurn = 1,
    kNumbered = 2,      // the parts are numbered
    kAnnounced = 4,     // the item's count is published
    kOwnLeft = 8,       // the own bin is still to be written
    kAside = 16,        // ... and its ids are in perm
    kRestore = 32,      // ... and need not be sorted again
    kTakenOver = 64     // the item was open; sh.interrupted waits
  };
  uint32_t item = own, bin = own, taken = 0, state = kFirstTurn;
  for (;;) {
    auto ap = (const __attribute__((address_space(4))) BinArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(ap));
    const BinArgs& a = *(const BinArgs*)ap;
    const uint32_t tid = own_thread();
    bool sorted = true, big = false;
    uint32_t heads = 0;
    if (state & kRestore) {
      state &= ~kRestore;
      heads = scalar(sh.aside);
      big = (heads >> 31) != 0;
      heads &= 0x7fffffffu;
    } else {
      bool unused;
      sorted = sort_item<kCrowded>(a, item, bin, taken, (state & kFirstTurn) != 0, unused, heads, big, m, sh);
      if (item >= kBins) state |= kNumbered;
    }
    const BinState& st = sh.state[item >= kBins ? 1 : 0];
    taken = 0;
    if (sorted && !(state & kAnnounced) && tid == 0) {
      __hip_atomic_store(&a.sync[kCountAt + item], heads + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (item >= kBins) {
        constexpr uint32_t kOne = 1u << 22;         // parts above, clusters (2^19 at most) below
        const uint32_t now = atomicAdd(&a.sync[kArriveAt + bin], heads + kOne) + heads + kOne;
        if (now / kOne == parts_of(a, sh.total[bin]))
          __hip_atomic_store(&a.sync[kCountAt + bin], now % kOne + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    // (a bin that is large and not done in parts leaves its workgroup no time for others)
    if ((state & (kFirstTurn | kNumbered)) == kFirstTurn && !(sorted && scalar(st.n) > (uint32_t)kBinCap)) {
      number_parts(a, own, sh);
      state |= kNumbered;
      if (sh.my_part != kNoItem) {
        if (sorted) {
          state |= kOwnLeft;
          const uint32_t n = scalar(st.n);
          if (n <= (uint32_t)kBinThreads) {
            // its ids go to their place already; it is written like a bin that was sorted through global memory (of so
            // few keys a wave's first round is its whole slice there)
            state |= kAside;
            if (tid < n) a.perm[scalar(st.start) + tid] = m.idx[tid];
            if (tid < (uint32_t)kBinWaves) sh.aside_heads[tid] = sh.head_cnt[tid];
            big = n != 0;
          }
          if (tid == 0) sh.aside = heads | (big ? 0x80000000u : 0u);
        }
        item = scalar(sh.my_part);
        bin = scalar(sh.my_bin);
        state &= ~(kFirstTurn | kAnnounced);
        taken = tid == 0 ? atomicExch(&a.sync[kClaimAt + item * kClaimStride], 1u) : 0u;
        continue;
      }
    }
    state &= ~kFirstTurn;
    if (sorted) {
      const uint32_t n = scalar(st.n), start = scalar(st.start), equal = scalar(st.equal);
      // the counts of the bins before, and of the parts of the same bin before
      const bool watch = tid < bin || (item >= kBins && tid < item && tid >= kBins + sh.first_part[bin]);
      bool numbered = (state & kNumbered) != 0;
      uint32_t base;
      const uint32_t other = wait_for_counts<kCrowded>(a, sh, own, watch, (state & kTakenOver) != 0, numbered, base);
      if (numbered) state |= kNumbered;
      if (other != kNoItem) {
        if (tid == 0) {
          sh.interrupted = item;
          sh.interrupted_bin = bin;
        }
        item = other;
        if (scalar(sh.open) < kBins) bin = scalar(sh.open);
        state = (state & ~kAnnounced) | kTakenOver;
        __syncthreads();
        continue;
      }
      write_item<kCrowded>(a, item, bin, n, start, heads, equal, big, base, m, sh, st);
    }
    if (state & kTakenOver) {
      item = scalar(sh.interrupted);
      bin = scalar(sh.interrupted_bin);
      state &= ~kTakenOver;
    } else if (state & kOwnLeft) {                  // after the part
      item = bin = own;
      if (state & kAside) {
        __syncthreads();
        if (tid < (uint32_t)kBinWaves) sh.head_cnt[tid] = sh.aside_heads[tid];
      }
      if (!sorted || (state & kAside)) state |= kRestore;
      state &= ~(kOwnLeft | kAside);
    } else {
      return;
    }
    state |= kAnnounced;
    __syncthreads();
  }
}

// SKIP: the workgroups of the bins before first_bin leave at once, for a test of the takeover.
template <bool DIRECT, bool SKIP = false>
__global__ __launch_bounds__(kBinThreads) void bin_group_kernel(BinArgs args) {
  extern __shared__ uint64_t bin_lds[];
  BinLds& m = *reinterpret_cast<BinLds*>(bin_lds);
  __shared__ BinShared sh;
  const uint32_t tid = threadIdx.x;
  for (uint32_t i = blockIdx.x * kBinThreads + tid; i < args.n_counters; i += gridDim.x * kBinThreads) args.window_counters[i] = 0;
  bool crowded = false, big = false;
  uint32_t heads = 0;
  if (DIRECT) {
    uint32_t item = 0;
    sort_item<kDirect>(args, item, 0, 0, true, crowded, heads, big, m, sh);
    write_item<kDirect>(args, 0, 0, args.N, 0, heads, 0, false, 0, m, sh, sh.state[0]);
    return;
  }
  // consecutive workgroups sit on different XCDs; neighbouring bins, whose keys and table entries share cache lines,
  // go to the same one
  const uint32_t own = (blockIdx.x % kXcds) * (kBins / kXcds) + blockIdx.x / kXcds;
  if (SKIP && own < args.first_bin) return;
  uint32_t taken = tid == 0 ? atomicExch(&args.sync[kClaimAt + own * kClaimStride], 1u) : 0u;
  // One turn, unless a bin is taken over: that bin then, and after it the own one again (it was in LDS).  The
  // arguments are read through a pointer that the compiler must take for a new one in every turn; otherwise it keeps
  // all of them in scalar registers across the loop, and has to spill those.
  bool first_turn = true;
  for (uint32_t bin = own;;) {
    auto ap = (const __attribute__((address_space(4))) BinArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(ap));
    const BinArgs& a = *(const BinArgs*)ap;
    const uint32_t tid = own_thread();
    uint32_t item = bin;
    const bool sorted = sort_item<kBalanced>(a, item, bin, taken, first_turn, crowded, heads, big, m, sh);
    if (seldom(crowded)) break;                     // (on the first turn)
    if (seldom(!sorted)) return;                    // (on the first turn) the bin is done by a workgroup that waited for it
    taken = 0;
    first_turn = false;
    if (tid == 0) __hip_atomic_store(&a.sync[kCountAt + bin], heads + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t n = scalar(sh.state[0].n), start = scalar(sh.state[0].start);
    bool numbered = false;
    uint32_t base;
    const uint32_t other = wait_for_counts<kBalanced>(a, sh, own, tid < bin, false, numbered, base);
    if (seldom(other != kNoItem)) {
      bin = other;
      __syncthreads();
      continue;
    }
    write_item<kBalanced>(a, bin, bin, n, start, heads, 0, false, base, m, sh, sh.state[0]);
    if (bin == own) return;
    bin = own;
    __syncthreads();
  }
  crowded_turns(own, m, sh);
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

template <bool DIRECT, bool SKIP = false>
hipError_t launch_bins(const BinArgs& a, hipStream_t stream) {
  auto kern = bin_group_kernel<DIRECT, SKIP>;
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
    // The second key buffer is free.  The table (at most 4 N bytes + 1 KB) and behind it the largest counts per tile (16
    // bytes per 256 keys) and the words of the bins and parts lie there: the sizes that the built-in scratch holds do not shrink for
    // the sake of this route.
    p.part_keys = max(kPartKeys, (uint32_t)(p.N / kBins));    // no more parts than workgroups
    p.parts = (uint32_t)(p.N / p.part_keys);
    p.off_table = p.off_key[1];
    p.off_peak = align256(p.off_table + (size_t)kBins * p.tiles * 4);
    p.off_blocksum = align256(p.off_peak + (size_t)p.tiles * kPeaks * 4);
    static_assert((4 - 1.0 / 16 - 1.0 / 32) * kSmallMaxN >= 1024 + 16 + 3 * 256 + sync_words(0) * 4,
                  "room behind the table at every size of this route");
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
    a.part_keys = plan.part_keys;
    a.peak = (const uint4*)(ws + plan.off_peak);
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
    LSHMOE_LAUNCH((tile_bin_kernel<TILE>), grid, block, 0, stream, src, N, plan.top_shift, table, keybuf[0], idxbuf[0], a.sync, \
                  plan.parts, (uint32_t*)a.peak)
    if (plan.tile == 256) LSHMOE_TILES(256);
    else if (plan.tile == 512) LSHMOE_TILES(512);
    else if (plan.tile == 1024) LSHMOE_TILES(1024);
    else LSHMOE_TILES(2048);
#undef LSHMOE_TILES
    return plan.first_bin == 0 ? launch_bins<false>(a, stream) : launch_bins<false, true>(a, stream);
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
