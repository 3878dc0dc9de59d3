// WENO advection variant of the periodic xy stencil (Sec. 4.3): launch
// arguments shared by the kernel (weno.hip) and its plan (api.cpp).
#pragma once

#include "mxs_internal.h"

namespace mxs {

struct WenoArgs {
    const void *phi, *u, *v;   // device, FP64, ny rows of pitch ld
    void *out;                 // device, FP64
    long long ld;
    int nx, ny;
    double rdx, rdy;           // 1 / dx, 1 / dy
    double floor_x, floor_y;   // the weights' floor 1e-99 times dx^2 and dy^2
    int rows;                  // output rows per workgroup (1, 4 or 8)
    int nchunks, nstrips;
    int order;                 // tile order, as for the 2D stencils
    int nt_store;              // non-temporal output stores
};

size_t weno_lds_bytes(int rows, int threads);
bool weno_rows_ok(int rows);
hipError_t launch_weno_adv(const WenoArgs &a, int threads, hipStream_t s);

}  // namespace mxs
