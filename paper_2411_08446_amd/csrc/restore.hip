// Restore with residual compensation (Eq. 4 and Eq. 5):
//     out[a] = expert_out[s] + (tokens[a / k] - centroids[s]),   s = seg_of[a].
//
// HBM-bound gather: per output row it reads the expert-output row and, for
// members of clusters with more than one member, the token row and the
// centroid row; it writes one row.  A group of LPR lanes owns kRows
// consecutive output rows (the k assignments of a token are consecutive, so
// they share the token row) and strides over the 16-byte pieces; with rows of
// 1 KB and more that is a whole wave, and the cluster lookups are wave-uniform
// scalars.  Output rows are written with streaming stores.  With large clusters the
// rows are dealt to the XCDs by columns instead (stretch.h, plan_restore, plan_combine).
#include "kernels.h"
#include "stretch.h"

namespace lshmoe {

namespace {

constexpr int kRows = 2;  // output rows a lane group works on at once

template <int LPR> __device__ __forceinline__ int32_t uniform(int32_t v) {
  return LPR == 64 ? __builtin_amdgcn_readfirstlane(v) : v;
}

// With perm and num_segments given, the lane groups walk the rows in cluster order (row a = perm[p]) when the
// clusters are long on average (S / N below kClusterOrderBelow): the members of a cluster are then restored
// side by side and its expert-output and centroid rows are fetched from memory once instead of once per
// member.  With mostly one-member clusters the assignment order is faster (measured at T5: S/N 0.92:
// 101 against 106 us; S/N 0.38: 124 against 104 us).
constexpr uint32_t kClusterOrderBelowNum = 13, kClusterOrderBelowDen = 20;  // S / N < 0.65

// The rows of whole tokens for one stretch (stretch.h): sixteen lanes to a token.
template <typename DT>
__device__ __forceinline__ void restore_stretch(const char* __restrict__ tokens, const char* __restrict__ centroids,
                                                const char* __restrict__ expert_out, const int32_t* __restrict__ seg_of,
                                                const int32_t* __restrict__ seg_offsets, char* __restrict__ out, uint32_t k,
                                                size_t row_bytes, bool no_res, const StretchDuty& duty, uint32_t* look) {
  constexpr int E = Piece<DT>::kElems, Q = 2;
  constexpr uint32_t kGroups = 256 / kStretchPieces;
  static_assert(kGroups * Q == kStretchTokens, "two tokens per lane group");
  const uint32_t at = duty.at + threadIdx.x % kStretchPieces * 16;
  for (uint32_t first = duty.first; first < duty.end; first += kStretchTokens) {
    const uint32_t here = min(kStretchTokens, duty.end - first);
    uint32_t i_of[Q];                     // lane groups past the end do the last token once more
    uint4 x[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      i_of[q] = min(q * kGroups + threadIdx.x / kStretchPieces, here - 1);
      x[q] = no_res ? make_uint4(0, 0, 0, 0) : load16_stream(tokens + (first + i_of[q]) * row_bytes + at);
    }
    __builtin_amdgcn_sched_barrier(0);
    for (uint32_t i = threadIdx.x; i < here * k; i += 256) {
      const uint32_t s = (uint32_t)seg_of[first * k + i];
      bool full = !no_res;
      if (full && seg_offsets != nullptr) full = seg_offsets[s + 1] - seg_offsets[s] != 1;
      look[i] = s | (full ? 0x80000000u : 0u);
    }
    __syncthreads();
    for (uint32_t j = 0; j < k; ++j) {
      uint4 ec[Q], cc[Q];
      uint32_t l[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        l[q] = look[i_of[q] * k + j];
        const size_t row = (l[q] & 0x7fffffffu) * row_bytes + at;
        ec[q] = load16(expert_out + row);
        cc[q] = make_uint4(0, 0, 0, 0);
        if (l[q] >> 31) cc[q] = load16(centroids + row);
      }
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        uint4 y = ec[q];
        if (!no_res) {
          float e[E];
          Piece<DT>::widen(ec[q], e);
          if (l[q] >> 31) {
            float xv[E], cv[E];
            Piece<DT>::widen(x[q], xv);
            Piece<DT>::widen(cc[q], cv);
#pragma unroll
            for (int i = 0; i < E; ++i) e[i] += xv[i] - cv[i];
          } else {
#pragma unroll
            for (int i = 0; i < E; ++i) e[i] += 0.0f;   // as the full formula would, -0 into +0
          }
          y = Piece<DT>::narrow(e);
        }
        store16_stream(out + ((size_t)(first + i_of[q]) * k + j) * row_bytes + at, y);
      }
    }
    if (first + kStretchTokens < duty.end) __syncthreads();   // before the lookups are overwritten
  }
}

template <typename DT, int LPR>
__global__ __launch_bounds__(256) void restore_kernel(
    const char* __restrict__ tokens, const char* __restrict__ centroids, const char* __restrict__ expert_out,
    const int32_t* __restrict__ seg_of, const int32_t* __restrict__ seg_offsets, const int32_t* __restrict__ perm,
    const int32_t* __restrict__ num_segments, char* __restrict__ out, uint32_t N, uint32_t k, uint32_t cpr,
    uint32_t flags, StretchPlan plan) {
  constexpr int G = 64 / LPR;
  constexpr int E = Piece<DT>::kElems;
  const uint32_t lane = threadIdx.x & 63;
  // a folded grid can pass 2^32 threads: the workgroup's first row is checked in 64 bits, the rest fits 32.
  // The row index is left in a vector register on purpose: with a scalar index the cluster lookups below
  // become scalar-cache loads, and this kernel then runs 3 us slower at the T5 shape (the gate-weighted
  // variant and the token-gradient kernel, which have one more lookup per row, gain from the scalar form).
  const uint64_t block64 = linear_block();
  if constexpr (LPR == 64) {
    if (plan.stretches != 0 && pays(plan, (uint32_t)*num_segments)) {
      __shared__ uint32_t look[kStretchTokens * kStretchExperts];
      restore_stretch<DT>(tokens, centroids, expert_out, seg_of, seg_offsets, out, k, (size_t)cpr * 16, (flags & 1u) != 0,
                          stretch_duty(plan, block64, N / k), look);
      return;
    }
  }
  if (block64 * (4u * G * kRows) >= N) return;
  const uint32_t a0 = (((uint32_t)block64 * 4u + (threadIdx.x >> 6)) * G + lane / LPR) * kRows;
  if (a0 >= N) return;
  const size_t row_bytes = (size_t)cpr * 16;
  const bool no_res = (flags & 1u) != 0;

  // what either order needs first is asked for together with the number of clusters that decides between them
  bool by_cluster = false;
  int32_t member[kRows], s[kRows];
#pragma unroll
  for (int u = 0; u < kRows; ++u) s[u] = seg_of[min(a0 + u, N - 1)];
  if (perm != nullptr && num_segments != nullptr) {
#pragma unroll
    for (int u = 0; u < kRows; ++u) member[u] = perm[min(a0 + u, N - 1)];
    by_cluster = (uint64_t)(uint32_t)*num_segments * kClusterOrderBelowDen < (uint64_t)N * kClusterOrderBelowNum;
  }
  uint32_t a[kRows];   // the rows this lane group restores
  bool live[kRows], full[kRows];
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    live[u] = a0 + u < N;
    a[u] = a0 + u;
    if (by_cluster) {
      a[u] = (uint32_t)uniform<LPR>(member[u]);
      s[u] = seg_of[a[u]];
    }
    s[u] = uniform<LPR>(s[u]);
  }
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    full[u] = live[u] && !no_res;
    // a one-member cluster's centroid is its token bit for bit: the residual is exactly zero
    if (full[u] && seg_offsets != nullptr)
      full[u] = uniform<LPR>(seg_offsets[s[u] + 1]) - uniform<LPR>(seg_offsets[s[u]]) != 1;
  }
  for (uint32_t c = lane % LPR; c < cpr; c += LPR) {
    uint4 ec[kRows], x[kRows], cc[kRows];
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
      if (live[u]) ec[u] = load16(expert_out + (size_t)s[u] * row_bytes + c * 16);
      if (full[u]) {
        x[u] = load16(tokens + (size_t)(a[u] / k) * row_bytes + c * 16);
        cc[u] = load16(centroids + (size_t)s[u] * row_bytes + c * 16);
      }
    }
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
      if (!live[u]) continue;
      uint4 y = ec[u];
      if (!no_res) {
        float e[E], xv[E], cv[E];
        Piece<DT>::widen(ec[u], e);
        if (full[u]) {
          Piece<DT>::widen(x[u], xv);
          Piece<DT>::widen(cc[u], cv);
#pragma unroll
          for (int i = 0; i < E; ++i) e[i] += xv[i] - cv[i];
        } else {
#pragma unroll
          for (int i = 0; i < E; ++i) e[i] += 0.0f;  // e + (+0): only turns -0 into +0, as the full formula would
        }
        y = Piece<DT>::narrow(e);
      }
      store16_stream(out + (size_t)a[u] * row_bytes + c * 16, y);
    }
  }
}

// The combine (restore_combine_kernel) of whole tokens for one stretch (stretch.h): sixteen lanes to a token.  The tokens' own
// loads go out first, the lookups of all tokens and experts are made once per workgroup and not once per lane group.
template <typename DT>
__device__ __forceinline__ void combine_stretch(const char* __restrict__ tokens, const char* __restrict__ centroids,
                                                const char* __restrict__ expert_out, const int32_t* __restrict__ seg_of,
                                                const int32_t* __restrict__ seg_offsets, const float* __restrict__ gate_weight,
                                                char* __restrict__ out, uint32_t k, size_t row_bytes, bool no_res,
                                                const StretchDuty& duty, uint2* look) {
  constexpr int E = Piece<DT>::kElems, Q = 2;
  constexpr uint32_t kGroups = 256 / kStretchPieces;
  static_assert(kGroups * Q == kStretchTokens, "two tokens per lane group");
  const uint32_t at = duty.at + threadIdx.x % kStretchPieces * 16;
  for (uint32_t first = duty.first; first < duty.end; first += kStretchTokens) {
    const uint32_t here = min(kStretchTokens, duty.end - first);
    uint32_t i_of[Q];                     // lane groups past the end do the last token once more
    uint4 x[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      i_of[q] = min(q * kGroups + threadIdx.x / kStretchPieces, here - 1);
      x[q] = no_res ? make_uint4(0, 0, 0, 0) : load16_stream(tokens + (first + i_of[q]) * row_bytes + at);
    }
    __builtin_amdgcn_sched_barrier(0);
    for (uint32_t i = threadIdx.x; i < here * k; i += 256) {
      const uint32_t a = first * k + i, s = (uint32_t)seg_of[a];
      bool full = !no_res;
      if (full && seg_offsets != nullptr) full = seg_offsets[s + 1] - seg_offsets[s] != 1;
      look[i] = make_uint2(s | (full ? 0x80000000u : 0u), __float_as_uint(gate_weight[a]));
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      float acc[E];
#pragma unroll
      for (int i = 0; i < E; ++i) acc[i] = 0.0f;
      for (uint32_t j = 0; j < k; ++j) {
        const uint2 l = look[i_of[q] * k + j];
        const bool full = l.x >> 31;
        const size_t row = (l.x & 0x7fffffffu) * row_bytes + at;
        const uint4 ec = load16(expert_out + row);
        uint4 cc = make_uint4(0, 0, 0, 0);
        if (full) cc = load16(centroids + row);
        float e[E];
        Piece<DT>::widen(ec, e);
        if (full) {
          float xv[E], cv[E];
          Piece<DT>::widen(x[q], xv);
          Piece<DT>::widen(cc, cv);
#pragma unroll
          for (int i = 0; i < E; ++i) e[i] += xv[i] - cv[i];
        }
        const float w = __uint_as_float(l.y);
#pragma unroll
        for (int i = 0; i < E; ++i) acc[i] = fmaf(w, e[i], acc[i]);
      }
      store16_stream(out + (first + i_of[q]) * row_bytes + at, Piece<DT>::narrow(acc));
    }
    if (first + kStretchTokens < duty.end) __syncthreads();   // before the lookups are overwritten
  }
}

// Restore fused with the gate-weighted combine of the k expert outputs of a token (Eq. 2 with gate weights):
//     out[t] = sum_j w[t][j] * (expert_out[s_j] + (tokens[t] - centroids[s_j])),   s_j = seg_of[t*k + j],
// accumulated in binary32 in the order j = 0..k-1 and rounded once.  One lane group per token, or sixteen lanes for each of its
// stretches: the token row is read once, and one row is written instead of k.
template <typename DT, int LPR>
__global__ __launch_bounds__(256) void restore_combine_kernel(
    const char* __restrict__ tokens, const char* __restrict__ centroids, const char* __restrict__ expert_out,
    const int32_t* __restrict__ seg_of, const int32_t* __restrict__ seg_offsets, const float* __restrict__ gate_weight,
    char* __restrict__ out, uint32_t T, uint32_t k, uint32_t cpr, uint32_t flags, StretchPlan plan) {
  constexpr int G = 64 / LPR;
  constexpr int E = Piece<DT>::kElems;
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t wave64 = linear_block() * 4u + (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if constexpr (LPR == 64) {
    if (plan.stretches != 0 && pays(plan, estimate_clusters(seg_of, T, k))) {   // the same for every workgroup
      __shared__ uint2 look[kStretchTokens * kStretchExperts];
      combine_stretch<DT>(tokens, centroids, expert_out, seg_of, seg_offsets, gate_weight, out, k, (size_t)cpr * 16,
                          (flags & 1u) != 0, stretch_duty(plan, linear_block(), T), look);
      return;
    }
  }
  if (wave64 * G >= T) return;
  const uint32_t t = (uint32_t)(wave64 * G) + lane / LPR;   // below T + 64: 32 bits are enough
  if (t >= T) return;
  const size_t row_bytes = (size_t)cpr * 16;
  const bool no_res = (flags & 1u) != 0;
  for (uint32_t c = lane % LPR; c < cpr; c += LPR) {
    float acc[E], xv[E];
#pragma unroll
    for (int i = 0; i < E; ++i) acc[i] = 0.0f;
    bool have_x = false;
    for (uint32_t j = 0; j < k; ++j) {
      const int32_t s = uniform<LPR>(seg_of[t * k + j]);
      const float w = __int_as_float(uniform<LPR>(__float_as_int(gate_weight[t * k + j])));
      bool full = !no_res;
      if (full && seg_offsets != nullptr)
        full = uniform<LPR>(seg_offsets[s + 1]) - uniform<LPR>(seg_offsets[s]) != 1;
      float e[E];
      Piece<DT>::widen(load16(expert_out + (size_t)s * row_bytes + c * 16), e);
      if (full) {
        if (!have_x) {
          Piece<DT>::widen(load16(tokens + (size_t)t * row_bytes + c * 16), xv);
          have_x = true;
        }
        float cv[E];
        Piece<DT>::widen(load16(centroids + (size_t)s * row_bytes + c * 16), cv);
#pragma unroll
        for (int i = 0; i < E; ++i) e[i] += xv[i] - cv[i];
      }
#pragma unroll
      for (int i = 0; i < E; ++i) acc[i] = fmaf(w, e[i], acc[i]);
    }
    store16_stream(out + (size_t)t * row_bytes + c * 16, Piece<DT>::narrow(acc));
  }
}

template <typename DT, int LPR>
void launch_combine_lpr(const void* tokens, const void* centroids, const void* expert_out, const int32_t* seg_of,
                        const int32_t* seg_offsets, const float* gate_weight, void* out, int64_t T, int k,
                        uint32_t cpr, uint32_t flags, hipStream_t stream) {
  constexpr int G = 64 / LPR;
  const uint64_t waves = ((uint64_t)T + G - 1) / G;
  uint64_t blocks = (waves + 3) / 4;
  StretchPlan plan{};
  if (LPR == 64) plan = plan_combine(T, k, cpr, std::is_same<DT, BF16>::value);
  if (plan.workgroups() > blocks) blocks = plan.workgroups();
  hipLaunchKernelGGL((restore_combine_kernel<DT, LPR>), grid_of_blocks(blocks), dim3(256), 0, stream, (const char*)tokens,
                     (const char*)centroids, (const char*)expert_out, seg_of, seg_offsets, gate_weight, (char*)out,
                     (uint32_t)T, (uint32_t)k, cpr, flags, plan);
}

template <typename DT>
void launch_combine_typed(const void* tokens, const void* centroids, const void* expert_out, const int32_t* seg_of,
                          const int32_t* seg_offsets, const float* gate_weight, void* out, int64_t T, int k,
                          uint32_t cpr, uint32_t flags, hipStream_t stream) {
  if (cpr > 16)
    launch_combine_lpr<DT, 64>(tokens, centroids, expert_out, seg_of, seg_offsets, gate_weight, out, T, k, cpr, flags, stream);
  else if (cpr > 4)
    launch_combine_lpr<DT, 16>(tokens, centroids, expert_out, seg_of, seg_offsets, gate_weight, out, T, k, cpr, flags, stream);
  else
    launch_combine_lpr<DT, 4>(tokens, centroids, expert_out, seg_of, seg_offsets, gate_weight, out, T, k, cpr, flags, stream);
}

template <typename DT, int LPR>
void launch_lpr(const void* tokens, const void* centroids, const void* expert_out, const int32_t* seg_of,
                const int32_t* seg_offsets, const int32_t* perm, const int32_t* num_segments, void* out, int64_t N,
                int k, uint32_t cpr, uint32_t flags, hipStream_t stream) {
  constexpr int G = 64 / LPR;
  const uint64_t groups = ((uint64_t)N + kRows - 1) / kRows;
  const uint64_t waves = (groups + G - 1) / G;
  uint64_t blocks = (waves + 3) / 4;
  StretchPlan plan{};
  if (LPR == 64 && num_segments != nullptr) plan = plan_restore(N, k, cpr);
  if (plan.workgroups() > blocks) blocks = plan.workgroups();
  hipLaunchKernelGGL((restore_kernel<DT, LPR>), grid_of_blocks(blocks), dim3(256), 0, stream, (const char*)tokens,
                     (const char*)centroids, (const char*)expert_out, seg_of, seg_offsets, perm, num_segments,
                     (char*)out, (uint32_t)N, (uint32_t)k, cpr, flags, plan);
}

template <typename DT>
void launch_typed(const void* tokens, const void* centroids, const void* expert_out, const int32_t* seg_of,
                  const int32_t* seg_offsets, const int32_t* perm, const int32_t* num_segments, void* out, int64_t N,
                  int k, uint32_t cpr, uint32_t flags, hipStream_t stream) {
  if (cpr > 16)
    launch_lpr<DT, 64>(tokens, centroids, expert_out, seg_of, seg_offsets, perm, num_segments, out, N, k, cpr, flags, stream);
  else if (cpr > 4)
    launch_lpr<DT, 16>(tokens, centroids, expert_out, seg_of, seg_offsets, perm, num_segments, out, N, k, cpr, flags, stream);
  else
    launch_lpr<DT, 4>(tokens, centroids, expert_out, seg_of, seg_offsets, perm, num_segments, out, N, k, cpr, flags, stream);
}

}  // namespace

hipError_t launch_restore(const void* tokens, const void* centroids, const void* expert_out,
                          const int32_t* seg_of, const int32_t* seg_offsets, const int32_t* perm,
                          const int32_t* num_segments, void* out, int64_t N, int k, int d, bool bf16, uint32_t flags,
                          hipStream_t stream) {
  const uint32_t cpr = (uint32_t)((size_t)d * (bf16 ? 2 : 4) / 16);
  if (bf16)
    launch_typed<BF16>(tokens, centroids, expert_out, seg_of, seg_offsets, perm, num_segments, out, N, k, cpr, flags, stream);
  else
    launch_typed<F32>(tokens, centroids, expert_out, seg_of, seg_offsets, perm, num_segments, out, N, k, cpr, flags, stream);
  return hipGetLastError();
}

hipError_t launch_restore_combine(const void* tokens, const void* centroids, const void* expert_out,
                                  const int32_t* seg_of, const int32_t* seg_offsets, const float* gate_weight,
                                  void* out, int64_t T, int k, int d, bool bf16, uint32_t flags, hipStream_t stream) {
  const uint32_t cpr = (uint32_t)((size_t)d * (bf16 ? 2 : 4) / 16);
  if (bf16)
    launch_combine_typed<BF16>(tokens, centroids, expert_out, seg_of, seg_offsets, gate_weight, out, T, k, cpr, flags, stream);
  else
    launch_combine_typed<F32>(tokens, centroids, expert_out, seg_of, seg_offsets, gate_weight, out, T, k, cpr, flags, stream);
  return hipGetLastError();
}

}  // namespace lshmoe
