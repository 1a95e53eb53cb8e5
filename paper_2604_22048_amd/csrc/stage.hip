// Copy of host inputs (batch plans, shear points) from the handle's pinned,
// device-mapped staging buffer into device workspace.  A kernel rather than
// an asynchronous memory copy, so that a call captured into a graph records
// kernel nodes only.  Source and destination are 16-byte aligned; the byte
// count is a multiple of 4 (the pieces are int32, int64 and double arrays).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "stage.h"

namespace bsi {

namespace {

// The pieces are short: one launch for all of a call's rather than one each.
__global__ void __launch_bounds__(256) stage_copy_kernel(StagePieces p) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int k = 0; k < p.n; ++k) {
    const uint4* __restrict__ src = static_cast<const uint4*>(p.src[k]);
    uint4* __restrict__ dst = static_cast<uint4*>(p.dst[k]);
    const int64_t n16 = (int64_t)(p.bytes[k] / 16);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) dst[i] = src[i];
    if (blockIdx.x == 0 && threadIdx.x < (p.bytes[k] % 16) / 4)
      reinterpret_cast<uint32_t*>(dst + n16)[threadIdx.x] =
          reinterpret_cast<const uint32_t*>(src + n16)[threadIdx.x];
  }
}

}  // namespace

hipError_t launch_stage_copy(const StagePieces& p, hipStream_t s) {
  size_t most = 0;
  for (int k = 0; k < p.n; ++k) {
    if ((p.bytes[k] & 3) || (reinterpret_cast<uintptr_t>(p.src[k]) & 15) ||
        (reinterpret_cast<uintptr_t>(p.dst[k]) & 15))
      return hipErrorInvalidValue;
    most = std::max(most, p.bytes[k]);
  }
  if (most == 0) return hipSuccess;
  const int64_t blocks = std::min<int64_t>(std::max<int64_t>(((int64_t)(most / 16) + 255) / 256, 1), 1024);
  hipLaunchKernelGGL(stage_copy_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p);
  return hipGetLastError();
}

}  // namespace bsi
