// Pieces of the staging copy (stage.hip): host data in mapped host memory (its
// device address) on its way to device workspace.
#pragma once

#include <hip/hip_runtime.h>

namespace bsi {

constexpr int kStagePieces = 4;

struct StagePieces {
  const void* src[kStagePieces];
  void* dst[kStagePieces];
  size_t bytes[kStagePieces];
  int n;
};

hipError_t launch_stage_copy(const StagePieces& p, hipStream_t s);

}  // namespace bsi
