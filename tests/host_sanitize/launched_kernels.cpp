// Looks at the kernels that the C ABI launches.  The program defines the runtime's registration and launch
// calls itself, so no GPU is needed and nothing is launched; pointers are never dereferenced.
#include <hip/hip_runtime.h>
#include <stdio.h>

#include <map>
#include <string>

#include "../../include/lshmoe.h"

static int failures = 0, checks = 0;

static std::map<const void*, std::string>& kernel_names() {
  static std::map<const void*, std::string> names;   // filled before main, while the objects register their kernels
  return names;
}

// The kernel with this in its name that the last call launched.
static const char* wanted = "";
static int seen = 0;
static std::string seen_name;

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
hipError_t hipLaunchKernel(const void* host, dim3, dim3, void**, size_t, hipStream_t) {
  if (kernel_names()[host].find(wanted) == std::string::npos) return hipSuccess;
  ++seen;
  seen_name = kernel_names()[host];
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
}

// Exactly one launch of the wanted kernel, with this in its name.
static void expect(const char* what, long long T, int d, int k, int status, const char* part) {
  ++checks;
  if (status == LSHMOE_OK && seen == 1 && seen_name.find(part) != std::string::npos) return;
  if (++failures <= 20) printf("FAIL %s T=%lld d=%d k=%d: status %d, %d launches, %s\n", what, T, d, k, status, seen, seen_name.c_str());
}

int main() {
  void* p = (void*)0x1000;
  int32_t* pi = (int32_t*)p;
  uint64_t* pu = (uint64_t*)p;
  // Whole-wave rows (more than 256 bytes): the compress call's seg_offsets has N + 1 entries, and the instance that asks for
  // them before it knows the number of clusters S is for that call alone; what comes back for the segment sums may end at S.
  wanted = "centroid_kernel";
  for (int dt = 0; dt < 2; ++dt) {
    const lshmoe_dtype dtype = dt ? LSHMOE_BF16 : LSHMOE_F32;
    for (long long T : {1ll, 5ll, 1000ll, 65536ll}) {
      for (int k : {1, 2}) {
        for (int pieces : {17, 128, 600}) {
          const int d = pieces * (dt ? 8 : 4);
          seen = 0;
          expect("compress", T, d, k, lshmoe_compress(p, pi, pu, T, d, k, 8, 3, 16, dtype, p, pi, pi, pi, pi, pi, pi, p, ~(size_t)0, nullptr),
                 "Li64ELb1E");
          seen = 0;
          expect("segment sums", T, d, k, lshmoe_decompress_backward(p, pi, pi, pi, pi, T, d, k, dtype, p, p, ~(size_t)0, nullptr),
                 "Li64ELb0E");
        }
      }
    }
  }
  printf("%d checks, %d failures\n", checks, failures);
  return failures || checks < 90 ? 1 : 0;
}
