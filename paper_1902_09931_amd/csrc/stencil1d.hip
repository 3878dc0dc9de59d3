// Batched 1D stencils: choice of the kernels by storage type (stencil1d_dev.h
// holds them).
#include "mxs_internal.h"

namespace mxs {

size_t stencil1d_lds_bytes(int dtype, int taps, int threads, int max_sig, int vecs) {
    const int V = dtype == F64 ? St<double>::V : dtype == F32 ? St<float>::V : St<bf16>::V;
    const int acc = dtype == F64 ? 8 : 4;
    const int pad = taps > 1 ? ((taps - 1 + V - 1) / V) * V : 0;
    const size_t vals = (static_cast<size_t>(2 * pad + threads * V * vecs) * acc + 15) & ~static_cast<size_t>(15);
    return vals + static_cast<size_t>(max_sig) * sizeof(long long);
}

hipError_t launch_stencil1d(int dtype, const Stencil1DArgs &a, int threads, int grid, hipStream_t s) {
    switch (dtype) {
    case F64: return launch_stencil1d_f64(a, threads, grid, s);
    case F32: return launch_stencil1d_f32(a, threads, grid, s);
    case BF16: return launch_stencil1d_bf16(a, threads, grid, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace mxs
