// A kernel that reports to the host: what a stream's states or fields hold, and
// that everything before it on the stream is done.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "tc_launch.h"

namespace tc {

// The words must be in host memory before the flag is.  Plain stores stay in the
// XCD's L2, and a write-back of it by a release of the flag alone does not do:
// with no store of its own outstanding, the compiler leaves out the wait between
// the write-back and the flag's store, and a host that sees the flag first reads
// states of the round before.  So the words are stored through to the system,
// and each wave waits for its own.
__global__ void __launch_bounds__(1024) k_publish(const uint64_t* src, uint64_t* dst, int words, uint64_t* flag,
                                                  uint64_t seq) {
  for (int i = threadIdx.x; i < words; i += blockDim.x)
    __hip_atomic_store(dst + i, src[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(flag, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

hipError_t launch_publish(const void* src, void* dst, int words, uint64_t* flag, uint64_t seq, hipStream_t stream) {
  // (the launch's own status: the last error may be another call's)
  void* args[] = {&src, &dst, &words, &flag, &seq};
  return hipLaunchKernel(reinterpret_cast<const void*>(k_publish), dim3(1), dim3(words > 64 ? 1024 : 64), args, 0,
                         stream);
}

}  // namespace tc
