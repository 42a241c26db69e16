// Scratch of the sampler kernels (sampler.hip).
#pragma once

#include "common.h"

namespace mls {

// uint64 entries that resampling N particles needs
int64_t resample_scratch(int64_t N);

// The many-workgroup next step's scratch lies behind the solver's two work
// counters, in the allocation that the context makes at its creation: the
// step allocates nothing, also not on its first call (it may be captured).
constexpr size_t kStepScratchOff = 256, kStepScratchBytes = 32768;
struct StepScratch;
inline StepScratch* step_scratch(mls2mc_ctx* ctx)
{
    return reinterpret_cast<StepScratch*>(reinterpret_cast<char*>(ctx->d_queue) + kStepScratchOff);
}

}  // namespace mls
