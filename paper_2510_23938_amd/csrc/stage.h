// stage.h -- the stages in which the one-wave leaf kernels move chunk bytes
// through LDS.
#pragma once
#include <stdint.h>
#include <hip/hip_runtime.h>

namespace hv {

constexpr int kStageBytes = 128;  // bytes per chunk per stage

// Where a stage's bytes start in a chunk (from the first stage's), in 64 bits:
// a chunk may hold 2^37 bytes, 2^30 stages.
__host__ __device__ constexpr uint64_t stage_offset(uint32_t stage) { return (uint64_t)kStageBytes * stage; }

}  // namespace hv
