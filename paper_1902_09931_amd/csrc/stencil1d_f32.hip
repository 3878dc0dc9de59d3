// float instances of the batched 1D stencil kernels.
#include "stencil1d_dev.h"

namespace mxs {

hipError_t launch_stencil1d_f32(const Stencil1DArgs &a, int threads, int grid, hipStream_t s) {
    return dispatch<float>(a, threads, grid, s);
}

}  // namespace mxs
