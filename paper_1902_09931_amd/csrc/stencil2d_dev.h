// Pieces shared by the 2D stencil kernels: the streaming form (stencil2d.hip)
// and the block form (stencil2d_block_dev.h).
#pragma once

#include "mxs_internal.h"

namespace mxs {
namespace {

// Strip and chunk of this workgroup.  order 0: the workgroups of one XCD
// take one contiguous range of tiles numbered strip by strip (a band of
// strips, chunks top to bottom); order 2: the same ranges numbered chunk by
// chunk (a band of chunks, strips left to right), so that horizontal
// neighbours, which share x halo columns, and vertical ones, which share
// rows, run on the same XCD at about the same time; order 1: workgroups in
// launch order, chunk by chunk.
__device__ __forceinline__ void tile_of(const Stencil2DArgs &a, int &strip, int &chunk) {
    if (a.order == 1) {
        chunk = blockIdx.x / a.nstrips;
        strip = blockIdx.x - chunk * a.nstrips;
        return;
    }
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    if (a.order == 0) {
        strip = tile / a.nchunks;
        chunk = tile - strip * a.nchunks;
    } else {
        chunk = tile / a.nstrips;
        strip = tile - chunk * a.nstrips;
    }
}

template <int NWX, int V> constexpr int halo_pad() {
    return NWX > 1 ? ((NWX - 1 + V - 1) / V) * V : 0;
}

template <typename A> __device__ __forceinline__ const A *coe_of(const Stencil2DArgs &a);
template <> __device__ __forceinline__ const double *coe_of<double>(const Stencil2DArgs &a) { return a.coe_d; }
template <> __device__ __forceinline__ const float *coe_of<float>(const Stencil2DArgs &a) { return a.coe_f; }

}  // namespace
}  // namespace mxs
