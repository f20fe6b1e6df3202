// Shared device helpers for the gfx950 kernels: storage-type traits and
// 16-byte vector access.  Wavefront size is 64 throughout.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace lshmoe {

constexpr int kWave = 64;

struct F32 {};   // IEEE binary32 storage
struct BF16 {};  // bfloat16 storage (upper half of binary32)

// Two binary32 -> two bfloat16, round to nearest even; NaN stays NaN.  One instruction (v_cvt_pk_bf16_f32): rounding with
// integer operations took six per element, in kernels that move rows a third of their vector work.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t f32_to_bf16_pair(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// v / n for a member count n (2^30 at most) with y = 1 / n (computed once per row), element by element: one Newton step on
// v * y, in four operations instead of the general division's eleven.  It is correctly rounded by Markstein's theorem (y is
// the correctly rounded reciprocal) unless the quotient is subnormal; there it is off by 2^-149 in up to one case of
// seventy, which rows of binary32 show and go through the general division for (with it for all of them the cluster sums
// of 10007 x 1000 took 22.5 us, so 21.5).  r is zero where v * y is exact and NaN where it is infinite: the product
// stands then.
template <typename DT, int E> __device__ __forceinline__ void div_count(float (&v)[E], float n, float y) {
  if (std::is_same<DT, F32>::value) {
    float least = fabsf(v[0]);
#pragma unroll
    for (int i = 1; i < E; ++i) least = fminf(least, fabsf(v[i]));
    if (least < 0x1p-96f) {                    // 2^-126 * 2^30
#pragma unroll
      for (int i = 0; i < E; ++i) v[i] = v[i] / n;
      return;
    }
  }
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const float q = v[i] * y;
    const float r = fmaf(-q, n, v[i]);
    v[i] = fabsf(r) > 0.0f ? fmaf(r, y, q) : q;
  }
}

// One wave per row (or cluster), or several waves to a few tokens, can mean more than 2^32 threads, which a
// one-dimensional launch cannot express (a dispatch counts work-items per dimension in 32 bits): grids beyond 2^22
// workgroups (of at most 512 threads) are folded into rows of kFoldedRow.  Surplus workgroups of the last row leave
// through the kernels' bounds checks.  The width is a constant: a kernel that asks for the grid's width waits for one more
// load before it can start (hash of 16384 rows of 768 bf16: 8.6 against 8.0 us).
constexpr uint32_t kFoldedRow = 1u << 16;
inline dim3 grid_of_blocks(uint64_t blocks) {
  if (blocks <= 1ull << 22) return dim3((uint32_t)(blocks == 0 ? 1 : blocks));
  return dim3(kFoldedRow, (uint32_t)((blocks + kFoldedRow - 1) / kFoldedRow));
}
__device__ __forceinline__ uint64_t linear_block() { return (uint64_t)blockIdx.y * kFoldedRow + blockIdx.x; }

// Rows are moved as raw 16-byte pieces (uint4) and only widened to binary32
// where arithmetic happens, so that loads in flight cost 4 registers each.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint4 load16(const char* p) { return *reinterpret_cast<const uint4*>(p); }
__device__ __forceinline__ void store16(char* p, uint4 v) { *reinterpret_cast<uint4*>(p) = v; }
// Streaming store: the line is not kept in the caches (outputs that nobody in this kernel reads again).
__device__ __forceinline__ void store16_stream(char* p, uint4 v) {
  const u32x4 w = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(p));
}

// Streaming load: rows that are read once should not push out rows that others will read again.
__device__ __forceinline__ uint4 load16_stream(const char* p) {
  const u32x4 w = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  return make_uint4(w.x, w.y, w.z, w.w);
}

template <typename DT> struct Piece;   // arithmetic on one 16-byte piece

template <> struct Piece<F32> {
  static constexpr int kElems = 4;
  static __device__ __forceinline__ void widen(uint4 q, float (&v)[4]) {
    v[0] = __uint_as_float(q.x); v[1] = __uint_as_float(q.y); v[2] = __uint_as_float(q.z); v[3] = __uint_as_float(q.w);
  }
  static __device__ __forceinline__ uint4 narrow(const float (&v)[4]) {
    return make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3]));
  }
};

template <> struct Piece<BF16> {
  static constexpr int kElems = 8;
  static __device__ __forceinline__ void widen(uint4 q, float (&v)[8]) {
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __uint_as_float(w[i] << 16);
      v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
  static __device__ __forceinline__ uint4 narrow(const float (&v)[8]) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = f32_to_bf16_pair(v[2 * i], v[2 * i + 1]);
    return make_uint4(w[0], w[1], w[2], w[3]);
  }
};

template <typename DT> struct ItemSize;
template <> struct ItemSize<F32> { static constexpr int value = 4; };
template <> struct ItemSize<BF16> { static constexpr int value = 2; };

}  // namespace lshmoe
