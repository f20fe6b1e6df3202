// Looks at the arguments of the launches that the C ABI makes.  The program defines the runtime's registration and launch
// calls itself, so no GPU is needed and nothing is launched; pointers are never dereferenced.
#include <hip/hip_runtime.h>
#include <stdio.h>
#include <string.h>

#include <map>
#include <string>

#include "../../include/lshmoe.h"

static int failures = 0, checks = 0;

static std::map<const void*, std::string>& kernel_names() {
  static std::map<const void*, std::string> names;   // filled before main, while the objects register their kernels
  return names;
}

// What the launch of the kernel with this in its name had as argument number `index`, of the last call.
static const char* wanted = "";
static int wanted_index = 0, seen = 0;
static uint32_t seen_value = 0;

static dim3 push_grid, push_block;
static size_t push_lds;
static hipStream_t push_stream;

extern "C" {
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned int, uint3*, uint3*, dim3*, dim3*, int*) {
  kernel_names()[host] = name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  push_grid = grid; push_block = block; push_lds = lds; push_stream = stream;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
  *grid = push_grid; *block = push_block; *lds = push_lds; *stream = push_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* host, dim3, dim3, void** args, size_t, hipStream_t) {
  if (kernel_names()[host].find(wanted) == std::string::npos) return hipSuccess;
  ++seen;
  memcpy(&seen_value, args[wanted_index], sizeof seen_value);
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
}

static void expect(const char* what, long long T, int d, int k, int status, uint32_t value) {
  ++checks;
  if (status == LSHMOE_OK && seen == 1 && seen_value == value) return;
  if (++failures <= 20)
    printf("FAIL %s T=%lld d=%d k=%d: status %d, %d launches, argument %u instead of %u\n", what, T, d, k, status, seen, seen_value, value);
}

int main() {
  void* p = (void*)0x1000;
  int32_t* pi = (int32_t*)p;
  uint64_t* pu = (uint64_t*)p;
  // The highest entry of seg_offsets that the centroid kernel asks for before it knows the number of clusters S: the
  // compress call's array has N + 1 of them, the one that comes back for the segment sums may have S + 1 (0: wait for S).
  wanted = "centroid_kernel";
  wanted_index = 8;
  for (int dt = 0; dt < 2; ++dt) {
    const lshmoe_dtype dtype = dt ? LSHMOE_BF16 : LSHMOE_F32;
    for (long long T : {1ll, 5ll, 1000ll, 65536ll}) {
      for (int k : {1, 2}) {
        for (int pieces : {1, 9, 17, 128, 600}) {
          const int d = pieces * (dt ? 8 : 4);
          seen = 0;
          expect("compress", T, d, k, lshmoe_compress(p, pi, pu, T, d, k, 8, 3, 16, dtype, p, pi, pi, pi, pi, pi, pi, p, ~(size_t)0, nullptr),
                 (uint32_t)(T * k));
          seen = 0;
          expect("segment sums", T, d, k, lshmoe_decompress_backward(p, pi, pi, pi, pi, T, d, k, dtype, p, p, ~(size_t)0, nullptr), 0);
        }
      }
    }
  }
  printf("%d checks, %d failures\n", checks, failures);
  return failures || checks < 80 ? 1 : 0;
}
