// Cluster centroids (Section 2.3 centroid formula with 1/n_j; Alg. 1 "Mean"):
// c_s = (1/n_s) * sum of the member rows, members taken in perm order,
// binary32 accumulation, one rounding to the storage type.
//
// HBM-bound gather: reads N token rows (T of them distinct), writes S rows.
// A group of LPR lanes owns one cluster and strides over the 16-byte pieces of
// the row; with rows of 1 KB and more that is a whole wave per cluster, and
// the cluster's offsets and member ids are wave-uniform scalars.  A one-member
// cluster is a plain row copy.  Centroid rows are written with streaming
// stores: nothing in this kernel reads them again.  By size: up to 16 members a
// plain sum, up to 32 a compensated one, up to kWindowMin the four waves of
// the workgroup share the cluster through LDS, beyond that the cluster is cut
// into blocks of positions that many workgroups (or waves) sum side by side;
// the one that finishes last adds the block sums in position order.
#include "kernels.h"

namespace lshmoe {

namespace {

constexpr int kPlainSumMax = 16;  // members summed without compensation
constexpr int kCoopMin = 32;      // clusters with more members (up to kWindowMin) are shared by the workgroup's waves
// Clusters with more members are cut into windows of positions.  The fewest that the windows' slots allow (see
// long_cluster_wg_window): one workgroup walks 1024 rows of 1536 bytes in 32 rounds per wave and pass, six workgroups and
// more the same cluster in four.  Measured against 1024, kernels whose
// largest clusters have hundreds of members: 67.6 -> 24.5 us, 44.2 -> 13.8 us, 57.8 -> 28.8 us.
constexpr int kWindowMin = 256;
static_assert(kWindowMin >= kCentroidWindow, "a window meets at most two windowed clusters only if they are longer than it");
constexpr size_t kCoopMaxLds = 32 * 1024;  // more LDS per workgroup would cut the occupancy of the common path

template <int LPR> __device__ __forceinline__ int32_t uniform(int32_t v) {
  return LPR == 64 ? __builtin_amdgcn_readfirstlane(v) : v;  // a whole wave shares the value: keep it scalar
}

// a + b without loss: a becomes the rounded sum, its rounding error is added to err (Knuth's two-sum; Kahan's shorter step
// needs the larger operand first, which holds for a long sum's next row but not where sums of the same size meet).
__device__ __forceinline__ void two_sum(float& a, float b, float& err) {
  const float t = a + b, bb = t - a;
  err += (a - (t - bb)) + (b - bb);
  a = t;
}

// Compensated sum of the token rows at sorted positions [a, b), wave-wide: lanes stride over the 16-byte pieces
// c_lo .. c_hi - 1 of the row, eight rows in flight (a walk by one wave is bound by memory latency).  emit(c, acc, comp)
// receives the sums of piece c and their compensations (the sum is acc - comp).  Kept small in registers on purpose: the kernel's occupancy is set by its largest path.
template <typename DT, typename Emit>
__device__ __forceinline__ void row_sum_kahan(const char* __restrict__ tokens, const int32_t* __restrict__ perm,
                                              int32_t a, int32_t b, uint32_t k, uint32_t c_lo, uint32_t c_hi,
                                              size_t row_bytes, Emit emit) {
  constexpr int E = Piece<DT>::kElems;
  constexpr int kRows = 8;
  const uint32_t lane = threadIdx.x & 63;
  // every lane of the wave walks every pass, also lanes past the end of the row (they hold member ids, see
  // below, and only skip the row loads): the loop bounds are wave-uniform
  for (uint32_t c0 = c_lo; c0 < c_hi; c0 += 64) {
    const uint32_t c = c0 + lane;
    const bool on = c < c_hi;
    float acc[E], comp[E];
#pragma unroll
    for (int i = 0; i < E; ++i) acc[i] = comp[i] = 0.0f;
    // the member ids come 64 at a time, one coalesced load per block (lane l holds the id of row p0 + l), so
    // that a round of row loads does not wait for an id load first; the next block is fetched a block ahead
    int32_t ids = perm[min(a + (int32_t)lane, b - 1)];
    for (int32_t p0 = a; p0 < b; p0 += 64) {
      const int32_t ids_now = ids;
      if (p0 + 64 < b) ids = perm[min(p0 + 64 + (int32_t)lane, b - 1)];
      const int32_t rows_here = min(64, b - p0);
      for (int32_t j = 0; j < rows_here; j += kRows) {
        uint4 q[kRows];
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
          const int32_t jj = min(j + u, rows_here - 1);  // the surplus rows of the last round are loaded and not added
          const uint32_t id = (uint32_t)__builtin_amdgcn_readlane(ids_now, jj);
          q[u] = on ? load16(tokens + (size_t)(id / k) * row_bytes + c * 16) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
          if (j + u < rows_here) {
            float x[E];
            Piece<DT>::widen(q[u], x);
#pragma unroll
            for (int i = 0; i < E; ++i) {
              const float y = x[i] - comp[i];
              const float t = acc[i] + y;
              comp[i] = (t - acc[i]) - y;
              acc[i] = t;
            }
          }
        }
      }
    }
    if (on) emit(c, acc, comp);
  }
}

// Data that workgroups of one launch hand to each other, whatever XCD they run on: eight bytes at a time past the XCD's own
// L2 (relaxed device-scope accesses).  Such a store is in memory once it is counted off (vmcnt), so "written before the
// counter moves" is a wait and not a device-scope fence, which writes back all that the L2 holds.  The compress call of 65536 x
// 1024 bf16, two experts, with 64 clusters of 1024 members, 200 of 300 and one of 65536, with two fences per block: 206, 270,
// 282 us; without 139, 171, 178.
__device__ __forceinline__ void store_shared8(void* p, uint32_t lo, uint32_t hi) {
  __hip_atomic_store((uint64_t*)p, (uint64_t)hi << 32 | lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint2 load_shared8(const void* p) {
  const uint64_t v = __hip_atomic_load((const uint64_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_uint2((uint32_t)v, (uint32_t)(v >> 32));
}
__device__ __forceinline__ void store_shared_row(float* p, float4 v) {
  store_shared8(p, __float_as_uint(v.x), __float_as_uint(v.y));
  store_shared8(p + 2, __float_as_uint(v.z), __float_as_uint(v.w));
}
__device__ __forceinline__ float4 load_shared_row(const float* p) {
  const uint2 a = load_shared8(p), b = load_shared8(p + 2);
  return make_float4(__uint_as_float(a.x), __uint_as_float(a.y), __uint_as_float(b.x), __uint_as_float(b.y));
}
__device__ __forceinline__ void wait_for_stores() {
  asm volatile("" ::: "memory");               // the stores stay in front of it, the counter's increment behind
  __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0)
  asm volatile("" ::: "memory");
}

// A cluster with more than kWindowMin members is summed by many waves: the sorted positions are cut into
// aligned blocks of kCentroidWindow; the wave that owns block m sums the part of the block that belongs to the
// long cluster containing the block's first position (slot 2m) and the part that belongs to a long cluster
// starting inside the block (slot 2m + 1; there is at most one, since a long cluster is longer than a block).
// Every window bumps its cluster's counter; the wave that brings it to the cluster's window count adds the
// partial sums in position order, so the result does not depend on which wave came last.
//
// The compensation of a window's sum is kept beside it, or a cluster of 257 to 1024 members would lose up to 0.4 times
// the error of one wave's sum over all its rows (rms against binary64, Gaussian rows, 1024 members: one wave 1.07e-9,
// windows without 1.48e-9, with 1.06e-9).  A block that lies in the cluster as a whole has its other slot free for it.  The
// two ends of the cluster put theirs into the cluster's own centroid row, which is written last: rounded to bfloat16 (eight
// bits of a correction will do) those of both ends fit a binary32 row, each 16-byte piece's into the piece itself.  Rows of
// bfloat16 are rounded far above that; there the ends are added to their sums.
template <typename DT>
__device__ __forceinline__ void long_cluster_window(
    const char* __restrict__ tokens, const int32_t* __restrict__ perm, const int32_t* __restrict__ seg_offsets,
    char* __restrict__ centroids, float* partial, uint32_t* counters, int32_t s, int32_t a, int32_t b, uint32_t slot,
    uint32_t k, uint32_t cpr, uint32_t d, uint32_t mean) {
  constexpr int E = Piece<DT>::kElems;
  constexpr bool kEndRows = std::is_same<DT, F32>::value;
  const size_t row_bytes = (size_t)cpr * 16;
  const uint32_t lane = threadIdx.x & 63;
  const int32_t lo = __builtin_amdgcn_readfirstlane(seg_offsets[s]);
  const int32_t hi = __builtin_amdgcn_readfirstlane(seg_offsets[s + 1]);
  const uint32_t m0 = (uint32_t)lo / kCentroidWindow, m1 = (uint32_t)(hi - 1) / kCentroidWindow;
  const uint32_t first_slot = 2 * m0 + ((uint32_t)lo % kCentroidWindow != 0 ? 1u : 0u);
  char* dst = centroids + (size_t)s * row_bytes;
  const bool whole = b - a == kCentroidWindow;      // blocks are aligned: the cluster covers this one
  float* out_row = partial + (size_t)slot * d;
  char* end_half = dst + (a == lo ? 0 : 8);         // the first end's corrections are the first half of each piece
  row_sum_kahan<DT>(tokens, perm, a, b, k, 0, cpr, row_bytes, [&](uint32_t c, float (&acc)[E], const float (&comp)[E]) {
    if (!kEndRows && !whole) {
#pragma unroll
      for (int i = 0; i < E; ++i) acc[i] -= comp[i];
    }
#pragma unroll
    for (int i = 0; i < E; i += 4) {
      store_shared_row(out_row + (size_t)c * E + i, make_float4(acc[i], acc[i + 1], acc[i + 2], acc[i + 3]));
      if (whole)
        store_shared_row(out_row + d + (size_t)c * E + i, make_float4(comp[i], comp[i + 1], comp[i + 2], comp[i + 3]));
      else if (kEndRows)
        store_shared8(end_half + c * 16, f32_to_bf16_pair(comp[i], comp[i + 1]), f32_to_bf16_pair(comp[i + 2], comp[i + 3]));
    }
  });
  wait_for_stores();  // the partial row is in memory before the counter moves
  uint32_t old = 0;
  if (lane == 0) old = atomicAdd(&counters[first_slot], 1u);
  old = __builtin_amdgcn_readfirstlane(old);
  if (old != m1 - m0) return;
  // The last window of the cluster: every other partial row is in memory, and what this XCD's caches may hold of them from
  // before is dropped once, so that they can be read as any other rows.  One wave reads them all, one pair behind the other, and
  // with every load past the L2 that took longer than the fences had: segment sums, one cluster of 65536 rows of 128 bytes
  // 236 -> 188 us, of 4608 bytes 1286 -> 968 (two fences per window 186, 970); 1024 x 256 of 256 bytes 38.3, 38.6 (86).
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  const uint32_t nwin = m1 - m0 + 1;
  const bool whole0 = (uint32_t)lo % kCentroidWindow == 0, whole1 = (uint32_t)hi % kCentroidWindow == 0;
  const float fn = (float)(hi - lo), inv = 1.0f / fn;
  constexpr int kRows = 2;
  for (uint32_t c = lane; c < cpr; c += 64) {
    float acc[E], err[E];
#pragma unroll
    for (int i = 0; i < E; ++i) acc[i] = err[i] = 0.0f;
    if (kEndRows) {
#pragma unroll
      for (int end = 0; end < 2; ++end) {
        if (end == 0 ? whole0 : whole1) continue;
        const uint2 w = *(const uint2*)(dst + c * 16 + end * 8);
        err[0] -= __uint_as_float(w.x << 16); err[1] -= __uint_as_float(w.x & 0xffff0000u);
        err[2] -= __uint_as_float(w.y << 16); err[3] -= __uint_as_float(w.y & 0xffff0000u);
      }
    }
    for (uint32_t j = 0; j < nwin; j += kRows) {
      float x[kRows][E], comp[kRows][E];
#pragma unroll
      for (int u = 0; u < kRows; ++u) {
        const uint32_t jj = min(j + u, nwin - 1);
        const float* src = partial + (size_t)(jj == 0 ? first_slot : 2 * (m0 + jj)) * d + (size_t)c * E;
        const bool whole_j = (jj != 0 || whole0) && (jj != nwin - 1 || whole1);
#pragma unroll
        for (int i = 0; i < E; i += 4) {
          const float4 v = *(const float4*)(src + i);
          const float4 w = whole_j ? *(const float4*)(src + d + i) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
          x[u][i] = v.x; x[u][i + 1] = v.y; x[u][i + 2] = v.z; x[u][i + 3] = v.w;
          comp[u][i] = w.x; comp[u][i + 1] = w.y; comp[u][i + 2] = w.z; comp[u][i + 3] = w.w;
        }
      }
#pragma unroll
      for (int u = 0; u < kRows; ++u) {
        if (j + u < nwin) {
#pragma unroll
          for (int i = 0; i < E; ++i) {
            two_sum(acc[i], x[u][i], err[i]);
            err[i] -= comp[u][i];
          }
        }
      }
    }
#pragma unroll
    for (int i = 0; i < E; ++i) acc[i] += err[i];
    if (mean) div_count<DT>(acc, fn, inv);
    store16_stream(dst + c * 16, Piece<DT>::narrow(acc));
  }
}

// The same with workgroups (needs the LDS of the shared sums).  The sorted positions are cut into aligned blocks of W and
// two workgroups take a block, each one half of the columns: every wave sums its quarter of the block's part of the
// cluster into LDS, wave 0 adds the four in wave order, writes half a partial row and bumps the half's counter (that of the
// cluster's first slot, or the one of its next block's, which counts for nobody else: the cluster covers that block's first
// position).  The workgroup that brings the counter to the cluster's block count adds its half of the partial
// rows in position order, again a quarter per wave joined through LDS in wave order, so the result does not depend on
// which workgroup came last.  Every join is by two-sums, and the first takes the waves' compensations with it (in LDS, in
// the columns of the other half): with plain sums the error was a third larger than that of four waves that share the
// whole cluster (rms against binary64, Gaussian rows, 600 / 1024 members: 2.41 / 1.66e-9 for four waves, 3.00 / 2.21e-9
// with plain joins, 2.28 / 1.57e-9 so; without the compensations 2.54 / 1.76e-9, far below the rounding of bfloat16 rows,
// which do without them).
// Called by all four waves of the workgroup with the same arguments (barriers inside).
//
// W: a wave is bound by memory latency, about 1.8 us per round of eight rows and 64 pieces, and the partial rows are read
// in rounds of four by the last workgroup alone.  Blocks of 128 positions halve the first part for clusters of up to
// kSmallWindowMax members; beyond that the second part would outweigh it and blocks are of 256 (with one huge cluster
// 128 and 512 were both slower).  One cluster of 4362 rows of 1536 bytes among 12022 others: the whole kernel
// 39.3 -> 25.1 us (with blocks of 256 by one workgroup each before; 14.3 now, see below).
// A cluster's blocks of either size use slots of their own: block m of 256 positions holds the slots of block 2m of 128,
// and at most one cluster beyond kWindowMin covers a block's first position and one starts inside it - of both sizes
// together, since no two clusters of 256 members and more start within 256 positions.
constexpr int kSmallWindowMax = 8192;
// The blocks are looked after by workgroups of their own, the first of the grid: with the long clusters' blocks behind the
// clusters that a workgroup has itself (up to 32 rows one after the other), the kernel waited for them (16384 rows of 1536
// bytes, one cluster of 4362: the step 66.4 -> 55.1 us; without fences, see store_shared8, 53.7; this kernel 26.9 -> 14.3).
// A workgroup asks for up to 16 of its (block, half) duties with one chain of three loads.  No more than 1024, or their
// looking around delays inputs that have no long cluster (65536 rows of 2048 bytes, two experts each: 2048 of them + 1 us);
// with 256, inputs of long clusters alone wait for them (64 clusters of 1024: 215 us for the call, with 1024 202, fences in
// both).
constexpr uint32_t kDutyWorkgroups = 1024, kDutiesAtOnce = 16;
__host__ __device__ inline uint32_t duty_workgroups(uint32_t N) {
  return N <= (uint32_t)kWindowMin ? 0u : min(2 * ((N + kCentroidWindow - 1) / kCentroidWindow), kDutyWorkgroups);
}
constexpr uint32_t kSmallWindow = kCentroidWindow, kLargeWindow = 2 * kCentroidWindow;
static_assert(kLargeWindow <= (uint32_t)kWindowMin, "a block meets at most two clusters that are cut into blocks");

template <typename DT>
__device__ __forceinline__ void long_cluster_wg_window(
    const char* __restrict__ tokens, const int32_t* __restrict__ perm, const int32_t* __restrict__ seg_offsets,
    char* __restrict__ centroids, float* partial, uint32_t* counters, float* coop_sum, int32_t s, uint32_t block_p0,
    uint32_t W, int32_t a, int32_t b, uint32_t slot, uint32_t half, uint32_t k, uint32_t cpr, uint32_t d, uint32_t mean) {
  constexpr int E = Piece<DT>::kElems;
  constexpr bool kComp = std::is_same<DT, F32>::value;   // the compensations are taken along
  const size_t row_bytes = (size_t)cpr * 16;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t w4 = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t stride = d + E;   // a row in LDS: one piece more, for the compensations of the longer half
  uint32_t* last_flag = reinterpret_cast<uint32_t*>(coop_sum + (size_t)4 * stride);   // one word behind the four rows
  const uint32_t middle = (cpr + 1) / 2;
  const uint32_t c_lo = half == 0 ? 0 : middle, c_hi = half == 0 ? middle : cpr;
  const uint32_t to_comp = (half == 0 ? middle : 0u - middle) * E;   // from a column's sum to its compensation
  const int32_t qa = max(a, (int32_t)(block_p0 + w4 * (W / 4)));
  const int32_t qb = min(b, (int32_t)(block_p0 + (w4 + 1) * (W / 4)));
  float* mine = coop_sum + (size_t)w4 * stride;
  if (qa < qb) {
    row_sum_kahan<DT>(tokens, perm, qa, qb, k, c_lo, c_hi, row_bytes,
                      [&](uint32_t c, const float (&acc)[E], const float (&comp)[E]) {
#pragma unroll
      for (int i = 0; i < E; i += 4) {
        *(float4*)(mine + c * E + i) = make_float4(acc[i], acc[i + 1], acc[i + 2], acc[i + 3]);
        if (kComp) *(float4*)(mine + (c * E + to_comp) + i) = make_float4(comp[i], comp[i + 1], comp[i + 2], comp[i + 3]);
      }
    });
  } else {
    for (uint32_t i = c_lo * E + lane; i < c_hi * E; i += 64) {
      mine[i] = 0.0f;
      if (kComp) mine[i + to_comp] = 0.0f;
    }
  }
  const int32_t lo = __builtin_amdgcn_readfirstlane(seg_offsets[s]);
  const int32_t hi = __builtin_amdgcn_readfirstlane(seg_offsets[s + 1]);
  const uint32_t m0 = (uint32_t)lo / W, m1 = (uint32_t)(hi - 1) / W;
  const uint32_t step = 2 * (W / (uint32_t)kCentroidWindow);   // slots per block
  const uint32_t first_slot = step * m0 + ((uint32_t)lo % W != 0 ? 1u : 0u);
  __syncthreads();
  if (w4 == 0) {
    float* out_row = partial + (size_t)slot * d;
    for (uint32_t i = c_lo * E + lane * 4; i < c_hi * E; i += 256) {   // E is a multiple of 4
      float4 v = *(const float4*)(coop_sum + i), e = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const float4 u = *(const float4*)(coop_sum + w * stride + i);
        if (w > 0) {
          two_sum(v.x, u.x, e.x); two_sum(v.y, u.y, e.y); two_sum(v.z, u.z, e.z); two_sum(v.w, u.w, e.w);
        }
        if (kComp) {
          const float4 q = *(const float4*)(coop_sum + w * stride + (i + to_comp));
          e.x -= q.x; e.y -= q.y; e.z -= q.z; e.w -= q.w;
        }
      }
      store_shared_row(out_row + i, make_float4(v.x + e.x, v.y + e.y, v.z + e.z, v.w + e.w));
    }
    wait_for_stores();  // the partial row is in memory before the counter moves
    if (lane == 0) *last_flag = atomicAdd(&counters[half == 0 ? first_slot : step * (m0 + 1)], 1u) == m1 - m0 ? 1u : 0u;
  }
  __syncthreads();    // the flag is set; the four LDS rows are free again
  if (*last_flag == 0u) return;   // the same for all four waves
  const uint32_t nwin = m1 - m0 + 1;
  const uint32_t per = (nwin + 3) / 4;
  const uint32_t j0 = min(w4 * per, nwin), j1 = min(j0 + per, nwin);
  constexpr int kRows = 4;
  for (uint32_t c = c_lo + lane; c < c_hi; c += 64) {
    float acc[E], err[E];
#pragma unroll
    for (int i = 0; i < E; ++i) acc[i] = err[i] = 0.0f;
    for (uint32_t j = j0; j < j1; j += kRows) {
      float x[kRows][E];
#pragma unroll
      for (int u = 0; u < kRows; ++u) {
        const uint32_t jj = min(j + u, j1 - 1);
        const float* src = partial + (size_t)(jj == 0 ? first_slot : step * (m0 + jj)) * d + (size_t)c * E;
#pragma unroll
        for (int i = 0; i < E; i += 4) {
          const float4 v = load_shared_row(src + i);
          x[u][i] = v.x; x[u][i + 1] = v.y; x[u][i + 2] = v.z; x[u][i + 3] = v.w;
        }
      }
#pragma unroll
      for (int u = 0; u < kRows; ++u) {
        if (j + u < j1) {
#pragma unroll
          for (int i = 0; i < E; ++i) two_sum(acc[i], x[u][i], err[i]);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < E; i += 4)
      *(float4*)(mine + c * E + i) =
          make_float4(acc[i] + err[i], acc[i + 1] + err[i + 1], acc[i + 2] + err[i + 2], acc[i + 3] + err[i + 3]);
  }
  __syncthreads();
  const float fn = (float)(hi - lo), inv = 1.0f / fn;
  char* dst = centroids + (size_t)s * row_bytes;
  for (uint32_t c = c_lo + threadIdx.x; c < c_hi; c += 256) {
    float acc[E];
#pragma unroll
    for (int i = 0; i < E; ++i) {
      float err = 0.0f;
      acc[i] = coop_sum[c * E + i];
#pragma unroll
      for (int w = 1; w < 4; ++w) two_sum(acc[i], coop_sum[w * stride + c * E + i], err);
      acc[i] += err;
    }
    if (mean) div_count<DT>(acc, fn, inv);
    store16_stream(dst + c * 16, Piece<DT>::narrow(acc));
  }
  __syncthreads();  // before the LDS rows are used again
}

// ALL: seg_offsets has N + 1 entries that may be read; otherwise it may end at entry S.
// Seven waves per SIMD are stated for bfloat16: left to itself the compiler takes 75 registers, three too many for it.
template <typename DT, int LPR, bool ALL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(std::is_same<DT, BF16>::value ? 7 : 1))) void centroid_kernel(
    const char* __restrict__ tokens, const int32_t* __restrict__ perm, const int32_t* __restrict__ seg_offsets,
    const int32_t* __restrict__ seg_of, const int32_t* __restrict__ num_segments, char* __restrict__ centroids,
    float* partial, uint32_t* counters, uint32_t N, uint32_t k, uint32_t cpr, uint32_t mean, uint32_t coop) {
  constexpr int G = 64 / LPR;  // clusters handled side by side by one wave
  constexpr int E = Piece<DT>::kElems;
  // coop: [4 waves][cpr * E] partial sums of a cluster the workgroup shares, or [4 waves][(cpr + 1) * E] and a flag
  extern __shared__ float coop_sum[];
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t block64 = linear_block();
  const bool shares = LPR == 64 && coop != 0;
  const uint32_t duty_wgs = shares ? duty_workgroups(N) : 0;
  // surplus workgroups of a folded grid (whole workgroups: no barrier is skipped by part of one)
  if (block64 >= duty_wgs + ((uint64_t)N + 3) / 4) return;
  const bool on_duty = block64 < duty_wgs;
  const uint32_t block = (uint32_t)(on_duty ? block64 : block64 - duty_wgs);
  const uint32_t wave = block * 4u + (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t s = wave * G + lane / LPR;
  const size_t row_bytes = (size_t)cpr * 16;
  // Whole-wave rows: the offsets of the workgroup's four clusters, in lanes 0 to 4, with ALL asked for together with the number
  // of clusters (those behind the last cluster mean nothing and are not used).  One after the other, and a wave's own offsets
  // once more behind them, these loads were two of the five trips to memory of a one-member cluster's wave.
  int32_t offsets = 0;
  if constexpr (LPR == 64 && ALL) {
    if (!on_duty) offsets = seg_offsets[min(block * 4u + min(lane, 4u), N)];
  }
  const uint32_t S = (uint32_t)*num_segments;
  if constexpr (LPR == 64 && !ALL) {
    if (!on_duty) offsets = seg_offsets[min(block * 4u + min(lane, 4u), S)];
  }
  // Clusters of kCoopMin+1 .. kWindowMin members (whole-wave rows only): a single wave walking such a
  // cluster is bound by memory latency (one round of 8 rows per ~2 us), and when a few hundred of them hold
  // most of the assignments the kernel waits for them.  The four waves of the workgroup therefore share each
  // such cluster among the workgroup's four: a quarter of the members each, joined through LDS in wave order.
  auto shared_size = [&](int32_t n) { return shares && n > kCoopMin && n <= kWindowMin; };
  if constexpr (LPR == 64) {
    if (on_duty) {
      // window duty with the workgroup's LDS rows.  Duty 2 m + half: one half of the columns of block m of kSmallWindow positions
      // and, with m even, of the block of kLargeWindow positions that starts there.
      const uint32_t duties = 2 * ((N + kSmallWindow - 1) / kSmallWindow), d = cpr * E;
      // (a turn by two from one round to the next: the wide blocks fall to other workgroups then)
      auto duty_of = [&](uint32_t q) { return (block + 2 * q) % duty_wgs + q * duty_wgs; };
      for (uint32_t q0 = 0; q0 * duty_wgs < duties; q0 += kDutiesAtOnce) {
        // lanes 3 j .. 3 j + 2: the clusters of the j-th duty's first position and of the two block sizes' last ones
        const uint32_t mine = duty_of(q0 + lane / 3);
        bool cut = false;
        int32_t cluster = 0;
        if (lane < 3 * kDutiesAtOnce && mine < duties) {
          const uint32_t m = mine >> 1, p0 = m * kSmallWindow;
          const uint32_t p = lane % 3 == 0 ? p0 : min(p0 + (lane % 3 == 1 || m % 2 != 0 ? kSmallWindow : kLargeWindow), N) - 1;
          cluster = seg_of[perm[p]];
          cut = seg_offsets[cluster + 1] - seg_offsets[cluster] > kWindowMin;
        }
        for (uint64_t left = __builtin_amdgcn_ballot_w64(cut); left != 0;) {   // the same in all four waves
          const uint32_t j = (uint32_t)__builtin_ctzll(left) / 3;
          left = left >> (3 * j + 3) << (3 * j + 3);
          const uint32_t at = duty_of(q0 + j), m = at >> 1, half = at & 1, p0 = m * kSmallWindow;
          int32_t of[3];
#pragma unroll
          for (int i = 0; i < 3; ++i) of[i] = __builtin_amdgcn_readlane(cluster, (int)(3 * j) + i);
          auto duty = [&](int32_t sc, uint32_t W, uint32_t slot) {
            const int32_t lo = __builtin_amdgcn_readfirstlane(seg_offsets[sc]);
            const int32_t hi = __builtin_amdgcn_readfirstlane(seg_offsets[sc + 1]);
            if (hi - lo <= kWindowMin || (hi - lo <= kSmallWindowMax) != (W == kSmallWindow)) return;
            long_cluster_wg_window<DT>(tokens, perm, seg_offsets, centroids, partial, counters, coop_sum, sc, p0, W,
                                       max(lo, (int32_t)p0), min(hi, (int32_t)min(p0 + W, N)), slot, half, k, cpr, d, mean);
          };
          // both block sizes meet the cluster of the first position; it is of one size class
          duty(of[0], kSmallWindow, 2 * m);
          if (of[1] != of[0]) duty(of[1], kSmallWindow, 2 * m + 1);
          if (m % 2 == 0) {
            duty(of[0], kLargeWindow, 2 * m);
            if (of[2] != of[0]) duty(of[2], kLargeWindow, 2 * m + 1);
          }
        }
      }
      return;
    }
  }
  // the sharing pass comes first: after its own cluster's stores a wave should have nothing left to wait for.  One vote over
  // the four sizes skips it: looking at them one by one cost the common case 1.4 us of 75 (65536 x 1024 bf16, 2 experts).
  bool any_shared = false;
  if constexpr (LPR == 64) {
    const int32_t next = __builtin_amdgcn_update_dpp(0, offsets, 0x101, 0xf, 0xf, false);   // row_shl:1, the next lane's
    any_shared = __builtin_amdgcn_ballot_w64(lane < 4 && block * 4u + lane < S && shared_size(next - offsets)) != 0;
  }
  if (__builtin_expect(any_shared, false)) {   // the same for every wave of the workgroup
    const uint32_t s0 = block * 4u, w4 = threadIdx.x >> 6;
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      const uint32_t sj = s0 + j;
      if (sj >= S) break;  // the same for every wave of the workgroup
      const int32_t lo = __builtin_amdgcn_readlane(offsets, j), hi = __builtin_amdgcn_readlane(offsets, j + 1);
      const int32_t n = hi - lo;
      if (!shared_size(n)) continue;
      const int32_t quarter = (n + 3) / 4;
      const int32_t a = min(lo + (int32_t)w4 * quarter, hi), b = min(a + quarter, hi);
      float* mine = coop_sum + (size_t)w4 * cpr * E;
      if (a < b) {
        row_sum_kahan<DT>(tokens, perm, a, b, k, 0, cpr, row_bytes, [&](uint32_t c, const float (&acc)[E], const float (&)[E]) {
#pragma unroll
          for (int i = 0; i < E; i += 4)
            *(float4*)(mine + (size_t)c * E + i) = make_float4(acc[i], acc[i + 1], acc[i + 2], acc[i + 3]);
        });
      } else {
        for (uint32_t i = lane; i < cpr * E; i += 64) mine[i] = 0.0f;
      }
      __syncthreads();
      char* dst = centroids + (size_t)sj * row_bytes;
      const float fn = (float)n, inv = 1.0f / fn;
      for (uint32_t c = threadIdx.x; c < cpr; c += 256) {
        float acc[E];
#pragma unroll
        for (int i = 0; i < E; ++i) {
          acc[i] = coop_sum[(size_t)c * E + i];
#pragma unroll
          for (int w = 1; w < 4; ++w) acc[i] += coop_sum[((size_t)w * cpr + c) * E + i];
        }
        if (mean) div_count<DT>(acc, fn, inv);
        store16_stream(dst + c * 16, Piece<DT>::narrow(acc));
      }
      __syncthreads();  // before the partial sums are overwritten
    }
  }
  if (s < S) {
    int32_t lo, hi;
    if constexpr (LPR == 64) {
      const int32_t w4 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
      lo = __builtin_amdgcn_readlane(offsets, w4);
      hi = __builtin_amdgcn_readlane(offsets, w4 + 1);
    } else {
      lo = seg_offsets[s];
      hi = seg_offsets[s + 1];
    }
    const int32_t n = hi - lo;
    if (shared_size(n)) {
      // done by the workgroup, above
    } else if (LPR == 64 && n > kPlainSumMax && n <= kWindowMin) {
      // a whole wave on a cluster of more than 16 members: compensated sum, eight rows in flight
      char* dst = centroids + (size_t)s * row_bytes;
      const float fn = (float)n, inv = 1.0f / fn;
      row_sum_kahan<DT>(tokens, perm, lo, hi, k, 0, cpr, row_bytes, [&](uint32_t c, float (&acc)[E], const float (&)[E]) {
        if (mean) div_count<DT>(acc, fn, inv);
        store16_stream(dst + c * 16, Piece<DT>::narrow(acc));
      });
    } else if (n <= kWindowMin) {
      const char* first = tokens + (size_t)((uint32_t)uniform<LPR>(perm[lo]) / k) * row_bytes;
      char* dst = centroids + (size_t)s * row_bytes;
      for (uint32_t c = lane % LPR; c < cpr; c += LPR) {
        const uint4 v0 = load16(first + c * 16);
        if (n == 1) {  // the mean of one row is the row
          store16_stream(dst + c * 16, v0);
          continue;
        }
        float acc[E], x[E];
        Piece<DT>::widen(v0, acc);
        int32_t p = lo + 1;
        if (n <= kPlainSumMax) {
          for (; p + 4 <= hi; p += 4) {
            uint4 q[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
              q[u] = load16(tokens + (size_t)((uint32_t)uniform<LPR>(perm[p + u]) / k) * row_bytes + c * 16);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              Piece<DT>::widen(q[u], x);
#pragma unroll
              for (int i = 0; i < E; ++i) acc[i] += x[i];
            }
          }
          for (; p < hi; ++p) {
            Piece<DT>::widen(load16(tokens + (size_t)((uint32_t)uniform<LPR>(perm[p]) / k) * row_bytes + c * 16), x);
#pragma unroll
            for (int i = 0; i < E; ++i) acc[i] += x[i];
          }
        } else {
          // longer cluster: compensated (Kahan) summation keeps the binary32 sum within
          // a couple of ulps of the exact one however many members there are
          float comp[E];
#pragma unroll
          for (int i = 0; i < E; ++i) comp[i] = 0.0f;
          for (; p < hi; p += 4) {
            uint4 q[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
              if (p + u < hi)
                q[u] = load16(tokens + (size_t)((uint32_t)uniform<LPR>(perm[p + u]) / k) * row_bytes + c * 16);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              if (p + u >= hi) break;
              Piece<DT>::widen(q[u], x);
#pragma unroll
              for (int i = 0; i < E; ++i) {
                const float y = x[i] - comp[i];
                const float t = acc[i] + y;
                comp[i] = (t - acc[i]) - y;
                acc[i] = t;
              }
            }
          }
        }
        if (mean) {
          const float fn = (float)n, inv = 1.0f / fn;
          div_count<DT>(acc, fn, inv);
        }
        store16_stream(dst + c * 16, Piece<DT>::narrow(acc));
      }
    }
  }
  if (shares) return;
  // window duty: wave m looks after block m of the sorted positions
  if ((uint64_t)wave * kCentroidWindow >= N) return;
  const uint32_t p0 = wave * (uint32_t)kCentroidWindow;
  const uint32_t p1 = min(p0 + (uint32_t)kCentroidWindow, N);
  const uint32_t d = cpr * E;
  const int32_t sf = __builtin_amdgcn_readfirstlane(seg_of[perm[p0]]);
  const int32_t sl = __builtin_amdgcn_readfirstlane(seg_of[perm[p1 - 1]]);
  {
    const int32_t lo = __builtin_amdgcn_readfirstlane(seg_offsets[sf]);
    const int32_t hi = __builtin_amdgcn_readfirstlane(seg_offsets[sf + 1]);
    if (hi - lo > kWindowMin)
      long_cluster_window<DT>(tokens, perm, seg_offsets, centroids, partial, counters, sf, (int32_t)p0,
                              min(hi, (int32_t)p1), 2 * wave, k, cpr, d, mean);
  }
  if (sl != sf) {
    const int32_t lo = __builtin_amdgcn_readfirstlane(seg_offsets[sl]);
    const int32_t hi = __builtin_amdgcn_readfirstlane(seg_offsets[sl + 1]);
    if (hi - lo > kWindowMin)
      long_cluster_window<DT>(tokens, perm, seg_offsets, centroids, partial, counters, sl, lo, (int32_t)p1,
                              2 * wave + 1, k, cpr, d, mean);
  }
}

template <typename DT, int LPR>
void launch_lpr(const void* tokens, const int32_t* perm, const int32_t* seg_offsets, const int32_t* seg_of,
                const int32_t* num_segments, void* centroids, float* partial, uint32_t* counters, int64_t N, int k,
                uint32_t cpr, bool mean, bool all_offsets, hipStream_t stream) {
  constexpr int G = 64 / LPR;
  const uint64_t waves = ((uint64_t)N + G - 1) / G;  // worst case S == N; surplus waves leave at once
  const uint32_t blocks = (uint32_t)((waves + 3) / 4);
  const size_t coop_bytes = (size_t)4 * cpr * Piece<DT>::kElems * sizeof(float);  // four partial rows in binary32
  const bool coop = LPR == 64 && coop_bytes <= kCoopMaxLds;
  constexpr size_t kCoopMore = 4 * Piece<DT>::kElems * sizeof(float) + 16;   // a piece more per row, the flag
  const dim3 grid = grid_of_blocks((uint64_t)blocks + (coop ? duty_workgroups((uint32_t)N) : 0u));
  // the instances differ for whole-wave rows only, and a choice inside the kernel costs the compress call: 65536 x 1024 bf16,
  // 0.16 clusters per assignment, this kernel 53.7 -> 55.4 us
  auto kern = all_offsets || LPR != 64 ? centroid_kernel<DT, LPR, true> : centroid_kernel<DT, LPR, LPR != 64>;
  hipLaunchKernelGGL(kern, grid, dim3(256), coop ? coop_bytes + kCoopMore : 0, stream, (const char*)tokens, perm, seg_offsets,
                     seg_of, num_segments, (char*)centroids, partial, counters, (uint32_t)N, (uint32_t)k, cpr, mean ? 1u : 0u,
                     coop ? 1u : 0u);
}

template <typename DT>
void launch_typed(const void* tokens, const int32_t* perm, const int32_t* seg_offsets, const int32_t* seg_of,
                  const int32_t* num_segments, void* centroids, float* partial, uint32_t* counters, int64_t N, int k,
                  uint32_t cpr, bool mean, bool all_offsets, hipStream_t stream) {
  if (cpr > 16)
    launch_lpr<DT, 64>(tokens, perm, seg_offsets, seg_of, num_segments, centroids, partial, counters, N, k, cpr, mean, all_offsets,
                       stream);
  else if (cpr > 4)
    launch_lpr<DT, 16>(tokens, perm, seg_offsets, seg_of, num_segments, centroids, partial, counters, N, k, cpr, mean, all_offsets,
                       stream);
  else
    launch_lpr<DT, 4>(tokens, perm, seg_offsets, seg_of, num_segments, centroids, partial, counters, N, k, cpr, mean, all_offsets,
                      stream);
}

}  // namespace

hipError_t launch_centroid(const void* tokens, const int32_t* perm, const int32_t* seg_offsets, const int32_t* seg_of,
                           const int32_t* num_segments, void* centroids, float* partial, uint32_t* counters, int64_t N,
                           int k, int d, bool bf16, bool mean, bool all_offsets, hipStream_t stream) {
  const uint32_t cpr = (uint32_t)((size_t)d * (bf16 ? 2 : 4) / 16);
  if (bf16)
    launch_typed<BF16>(tokens, perm, seg_offsets, seg_of, num_segments, centroids, partial, counters, N, k, cpr, mean, all_offsets,
                       stream);
  else
    launch_typed<F32>(tokens, perm, seg_offsets, seg_of, num_segments, centroids, partial, counters, N, k, cpr, mean, all_offsets,
                      stream);
  return hipGetLastError();
}

}  // namespace lshmoe
