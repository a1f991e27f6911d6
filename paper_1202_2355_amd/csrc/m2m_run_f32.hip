// Run kernels (several steps per launch) with float particle state.
#include "m2m_run.h"

namespace m2m {

hipError_t launch_run_f32(int block, int kin, const FitDev& fd, const RunArgs& ra, int blocks,
                          size_t lds, const RunCall& call, hipStream_t s, hipEvent_t done) {
    if (block == 512) return launch_run_t<float, 512, false>(kin, fd, ra, blocks, lds, call, s, done);
    if (block == 1024) return launch_run_t<float, 1024, false>(kin, fd, ra, blocks, lds, call, s, done);
    return hipErrorInvalidValue;
}

hipError_t launch_runs_f32(int block, int kin, const FitDev* fits, const RunArgs* ras,
                           const RunTile* tiles, int blocks, size_t lds, int n_steps, uint32_t tag0,
                           hipStream_t s, hipEvent_t done) {
    if (block == 512) return launch_runs_t<float, 512>(kin, fits, ras, tiles, blocks, lds, n_steps, tag0, s, done);
    if (block == 1024) return launch_runs_t<float, 1024>(kin, fits, ras, tiles, blocks, lds, n_steps, tag0, s, done);
    return hipErrorInvalidValue;
}

}  // namespace m2m
