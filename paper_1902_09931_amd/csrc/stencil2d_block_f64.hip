// 2D stencils in block form, double storage.
#include "stencil2d_block_dev.h"

namespace mxs {

hipError_t launch_stencil2d_block_f64(int nwx, int nwy, const Stencil2DArgs &a, int threads, hipStream_t s) {
    return dispatch_block<double>(nwx, nwy, a, threads, s);
}

}  // namespace mxs
