// Records the launches that the C ABI makes at the ends of its documented ranges.  The program defines the runtime's
// launch calls itself, so no GPU is needed and nothing is launched; pointers are never dereferenced.
//
// A dispatch counts the work-items of a dimension in 32 bits: workgroups x workgroup size must stay below 2^32 in each,
// or only a part of the grid runs without an error.
#include <hip/hip_runtime.h>
#include <stdio.h>

#include "../../include/lshmoe.h"

static int failures = 0, launches = 0;
static long long now_T = 0;
static int now_rows = 0, now_gate = 0, now_d = 0;
static const char* now_call = "";
static dim3 push_grid, push_block;
static size_t push_lds;
static hipStream_t push_stream;

extern "C" {
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  push_grid = grid; push_block = block; push_lds = lds; push_stream = stream;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
  *grid = push_grid; *block = push_block; *lds = push_lds; *stream = push_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3 grid, dim3 block, void**, size_t lds, hipStream_t) {
  ++launches;
  const unsigned long long limit = 1ull << 32;
  if ((unsigned long long)grid.x * block.x >= limit || (unsigned long long)grid.y * block.y >= limit || grid.z != 1 ||
      grid.y > 65535u || grid.x == 0 || grid.y == 0 || lds > 160 * 1024) {
    if (++failures <= 20)
      printf("FAIL %s T=%lld d=%d rows=%d gate=%d: grid %u x %u of %u threads, %zu bytes of LDS\n", now_call, now_T, now_d,
             now_rows, now_gate, grid.x, grid.y, block.x, lds);
  }
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
}

static void expect_ok(int status) {
  if (status != LSHMOE_OK && ++failures <= 20) printf("FAIL %s T=%lld d=%d rows=%d: %s\n", now_call, now_T, now_d, now_rows, lshmoe_last_error());
}

int main() {
  void* p = (void*)0x1000;
  int32_t* pi = (int32_t*)p;
  uint64_t* pu = (uint64_t*)p;
  float* pf = (float*)p;
  const long long top = (1ll << 30) - 1;
  const long long Ts[] = {1, 33, 8191, 8192, 8193, 16384, 16385, 24575, 24576, 32768, 32769, 65535, 65536, 1ll << 27,
                          (1ll << 28) - 31, 1ll << 29, (1ll << 29) + 1, top - 64, top};
  const int hashes[][2] = {{1, 2}, {31, 2}, {2, 8}, {2, 16}, {1, 20}, {2, 32}, {2, 24}, {3, 32}, {2, 64}, {5, 32}, {10, 16}, {4, 64}, {1, 256}, {7, 100}};
  for (int dt = 0; dt < 2; ++dt) {
    const lshmoe_dtype dtype = dt ? LSHMOE_BF16 : LSHMOE_F32;
    for (long long T : Ts) {
      now_T = T;
      for (const auto& h : hashes) {
        const int L = h[0], r = h[1];
        now_rows = L * r;
        now_gate = 0;
        for (int pieces : {1, 8, 13, 32}) {
          now_d = pieces * (dt ? 8 : 4);
          now_call = "hash";
          expect_ok(lshmoe_hash(p, p, T, now_d, L, r, dtype, pu, nullptr));
        }
        if (r % 8 != 0) continue;
        now_d = 32 * (dt ? 8 : 4);
        for (int E : {1, 16, 64, 128}) {
          now_gate = E;
          now_call = "hash + gate";
          expect_ok(lshmoe_hash_gate(p, p, p, T, now_d, L, r, E, dtype, pu, pf, nullptr));
        }
      }
      now_gate = 0;
      now_d = dt ? 8 : 4;
      for (int B : {1, 63}) {
        now_rows = B;
        now_call = "hash sphere";
        expect_ok(lshmoe_hash_sphere(p, p, pf, T, now_d, B, dtype, pu, nullptr));
      }
      for (int k : {1, 2, 8}) {
        if (T * k > top) continue;
        for (int pieces : {1, 3, 9, 70, 64, 128, 192}) {   // the last three may be dealt by columns
          if ((unsigned long long)T * k * pieces > 0xffffff00ull) continue;
          now_d = pieces * (dt ? 8 : 4);
          now_rows = k;
          now_call = "compress";
          expect_ok(lshmoe_compress(p, pi, pu, T, now_d, k, 8, 3, 16, dtype, p, pi, pi, pi, pi, pi, pi, p, ~(size_t)0, nullptr));
          now_call = "decompress";
          expect_ok(lshmoe_decompress(p, p, p, pi, pi, nullptr, nullptr, T, now_d, k, dtype, 0, p, nullptr));
          expect_ok(lshmoe_decompress(p, p, p, pi, pi, pi, pi, T, now_d, k, dtype, 0, p, nullptr));
          now_call = "decompress combine";
          expect_ok(lshmoe_decompress_combine(p, p, p, pi, pi, pf, T, now_d, k, dtype, 0, p, nullptr));
          now_call = "backward";
          expect_ok(lshmoe_decompress_combine_backward(p, p, p, pi, pi, pf, p, T, now_d, k, dtype, 0, pf, p, nullptr));
          expect_ok(lshmoe_decompress_backward(p, pi, pi, pi, pi, T, now_d, k, dtype, p, p, ~(size_t)0, nullptr));
          expect_ok(lshmoe_compress_backward(p, p, p, pi, pi, T, now_d, k, dtype, 0, p, nullptr));
        }
      }
    }
  }
  printf("%d launches, %d failures\n", launches, failures);
  return failures || launches < 1000 ? 1 : 0;
}
