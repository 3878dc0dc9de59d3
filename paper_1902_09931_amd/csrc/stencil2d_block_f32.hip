// 2D stencils in block form, float storage.
#include "stencil2d_block_dev.h"

namespace mxs {

hipError_t launch_stencil2d_block_f32(int nwx, int nwy, const Stencil2DArgs &a, int threads, hipStream_t s) {
    return dispatch_block<float>(nwx, nwy, a, threads, s);
}

}  // namespace mxs
