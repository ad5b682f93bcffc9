// Every form of load_to_lds in use, a few of them in a row between accesses of LDS by the compiler's
// own hand, for a look at the code that comes out (compiled, not run).
#include "../../paper_2503_04424_amd/csrc/kernels_update.h"

template <int SIZE, int SCOPE>
__global__ void forms(const char* from, float* to, int rows) {
  __shared__ float lds[4096];
  const unsigned at = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(mdet::upd_lds_ptr)lds);
  for (int r = 0; r < rows; ++r) {
    mdet::load_to_lds<SIZE, SCOPE>(from, (unsigned)(SIZE * threadIdx.x), at + 1024u * (unsigned)r);
    mdet::load_to_lds<SIZE, SCOPE>(from + 1024, (unsigned)(SIZE * threadIdx.x), at + 2048u);
    atomicAdd(&lds[threadIdx.x + r], 1.0f);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  to[threadIdx.x] = lds[threadIdx.x];
}
template __global__ void forms<16, 0>(const char*, float*, int);
template __global__ void forms<16, mdet::DEVICE_SCOPE>(const char*, float*, int);
template __global__ void forms<4, 0>(const char*, float*, int);
template __global__ void forms<4, mdet::DEVICE_SCOPE>(const char*, float*, int);
