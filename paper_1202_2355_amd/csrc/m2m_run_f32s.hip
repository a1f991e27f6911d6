// Run kernels of fits whose priors are smoothed, float particle state.
#include "m2m_run.h"

namespace m2m {

hipError_t launch_run_smooth_f32(int block, int kin, const FitDev& fd, const RunArgs& ra, int blocks,
                                size_t lds, const RunCall& call, hipStream_t s, hipEvent_t done) {
    if (block == 512) return launch_run_t<float, 512, true>(kin, fd, ra, blocks, lds, call, s, done);
    if (block == 1024) return launch_run_t<float, 1024, true>(kin, fd, ra, blocks, lds, call, s, done);
    return hipErrorInvalidValue;
}

}  // namespace m2m
