// Column solves in one launch: every workgroup solves a strip of columns held
// in its registers (strips_dev.h), so the columns are read once and no carry
// between segments goes through memory.  The three phases (cols_dev.h) read
// the right-hand side twice and need two more launches, but move 2 KiB of a
// row at a time; a strip moves pieces of 32 to 128 bytes of every row, which
// memory serves at 2.5 to 4.8 TB/s (a copy with the same pieces and no
// arithmetic measured the same to within 10%, so the piece size is what
// bounds it).  strip_shape_for picks the piece: wide strips where there are
// enough columns to fill the CUs with them, narrow ones otherwise.
#include "strips_dev.h"

namespace mxs {

namespace {

template <typename TR, typename TX, int BW, int EPI, int NT, int CW, int LMAX>
__global__ void __launch_bounds__(NT) strips_kernel(const StripInst *__restrict__ inst, const int *__restrict__ map,
                                                    int count) {
    __shared__ double2 xch[2 * (NT / 64) * CW];
    const int b = xcd_tile(blockIdx.x, count);   // neighbouring strips, which share cache lines, on one XCD
    const StripInst &I = inst[map ? map[b] : 0];
    strip_block<TR, TX, BW, EPI, NT, CW, LMAX>(I, b - I.blk0, xch);
}

template <typename TR, typename TX, int BW, int EPI>
hipError_t strips_shape(int shape, const StripInst *inst, const int *map, int blocks, hipStream_t s) {
    switch (shape) {
    case 0: hipLaunchKernelGGL((strips_kernel<TR, TX, BW, EPI, 256, 4, 8>), dim3(blocks), dim3(256), 0, s, inst, map, blocks); break;
    case 1: hipLaunchKernelGGL((strips_kernel<TR, TX, BW, EPI, 512, 4, 8>), dim3(blocks), dim3(512), 0, s, inst, map, blocks); break;
    case 2: hipLaunchKernelGGL((strips_kernel<TR, TX, BW, EPI, 512, 16, 32>), dim3(blocks), dim3(512), 0, s, inst, map, blocks); break;
    case 3: hipLaunchKernelGGL((strips_kernel<TR, TX, BW, EPI, 1024, 16, 32>), dim3(blocks), dim3(1024), 0, s, inst, map, blocks); break;
    case 4: hipLaunchKernelGGL((strips_kernel<TR, TX, BW, EPI, 512, 8, 32>), dim3(blocks), dim3(512), 0, s, inst, map, blocks); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename TR, typename TX>
hipError_t strips_bw(int bw, int shape, const StripInst *inst, const int *map, int blocks, hipStream_t s) {
    return bw == 1 ? strips_shape<TR, TX, 1, 0>(shape, inst, map, blocks, s)
                   : strips_shape<TR, TX, 2, 0>(shape, inst, map, blocks, s);
}

}  // namespace

// Measured on FP64 grids, Cahn-Hilliard update, three phases against strips:
// 512^2 14.8 / 6.5 us (shape 0), 1024^2 19.0 / 12.4 (1; shape 2: 17), 2500 x
// 700 27.4 / 17.5 (2; shape 1: 20.5), 8000 x 1000 63.8 / 57.9 (2; shape 1:
// 90), 3000 x 2000 68.8 / 53.7 (3; shape 4: 57), 1536^2 38.9 / 33.5 (4;
// shape 3: 40), 2048^2 43.8 / 47.8 (4), 2051 x 3000 75 / 90 (1024 threads of
// 32 rows, 8 columns).  The plain solve, which has half the words to move,
// gains more (2048^2 27.6 / 19.2).
int strip_shape_for(int ny_max, long long sum_nx, int epilogue) {
    if (ny_max <= 1024) return sum_nx >= 2048 ? 2 : ny_max <= 512 ? 0 : 1;
    if (ny_max > 2048) return -1;
    if (sum_nx >= 2800) return 3;
    return epilogue == 0 || sum_nx * ny_max <= 3000000 ? 4 : -1;
}

StripShape strip_shape(int shape) {
    constexpr StripShape k[] = {{256, 4, 8}, {512, 4, 8}, {512, 16, 32}, {1024, 16, 32}, {512, 8, 32}};
    return k[shape];
}

size_t strip_tab_size(int shape) {
    const StripShape k = strip_shape(shape);
    return strip_tab_doubles(64 / k.columns, k.threads / 64);
}

void fill_strip(const CyclicFactor &f, int bw, int nx, int ny, int shape, StripInst *si, double *tab) {
    const StripShape k = strip_shape(shape);
    const int segs = k.threads / k.columns;
    si->nx = nx;
    si->ny = ny;
    si->L = (ny + segs - 1) / segs;
    si->nseg = (ny + si->L - 1) / si->L;
    si->p1 = f.p1;
    si->p2 = bw == 2 ? f.p2 : 0.0;
    si->invK = f.invK;
    fill_strip_tab(f, bw, ny, si->L, 64 / k.columns, k.threads / 64, tab);
}

hipError_t launch_strips(int rhs_dtype, int x_dtype, int bw, int epilogue, int shape, const StripInst *inst,
                         const int *map, int blocks, hipStream_t s) {
    if (bw != 1 && bw != 2) return hipErrorInvalidValue;
    if (epilogue == 0) {
        if (rhs_dtype == F64 && x_dtype == F64) return strips_bw<double, double>(bw, shape, inst, map, blocks, s);
        if (rhs_dtype == F32 && x_dtype == F32) return strips_bw<float, float>(bw, shape, inst, map, blocks, s);
        if (rhs_dtype == BF16 && x_dtype == BF16) return strips_bw<bf16, bf16>(bw, shape, inst, map, blocks, s);
    } else if (bw == 2) {
        if (rhs_dtype == F64 && x_dtype == F64) return strips_shape<double, double, 2, 1>(shape, inst, map, blocks, s);
        if (rhs_dtype == F32 && x_dtype == F32) return strips_shape<float, float, 2, 1>(shape, inst, map, blocks, s);
        if (rhs_dtype == F32 && x_dtype == BF16) return strips_shape<float, bf16, 2, 1>(shape, inst, map, blocks, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace mxs
