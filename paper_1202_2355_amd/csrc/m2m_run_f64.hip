// Run kernels (several steps per launch) with double particle state.
#include "m2m_run.h"

namespace m2m {

hipError_t launch_run_f64(int block, int kin, const FitDev& fd, const RunArgs& ra, int blocks,
                         size_t lds, hipStream_t s) {
    if (block == 512) return launch_run_kin<double, 512>(kin, fd, ra, blocks, lds, s);
    return hipErrorInvalidValue;
}

}  // namespace m2m
