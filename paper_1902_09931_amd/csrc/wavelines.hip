// Cyclic banded line solves with the whole line in the registers of one
// wavefront (lines of at most kWaveLineMax elements).  Same factorisation as
// the other line kernels: the forward recurrence y_i = r_i + p1 y_{i-1} +
// p2 y_{i-2} and the backward one u_i = y_i + p1 u_{i+1} + p2 u_{i+2}, both
// cyclic, then x = u / K (the periodic line inversions of the ADI scheme,
// Sec. 5.1).
//
// Layout: the line is cut into blocks of 64 E elements; in every block lane l
// holds the E consecutive elements 64 E c + E l + j, j = 0..E-1 (E = 4, 8 or
// 16 by line length).  Loads and stores stay coalesced: a block is read with
// one element per lane per instruction and transposed through a small LDS
// buffer of the wavefront.  With the state s_i = (y_i, y_{i-1}) the
// recurrence is s_i = M s_{i-1} + (r_i, 0), M = [[p1, p2], [1, 0]].
//
// Each direction takes two passes over the registers:
//   A. from a zero state at the line start: every lane runs the recurrence
//      over its E elements; a scan of the lane totals within each row of 16
//      lanes (DPP row shifts, multipliers M^E .. M^8E) and a chain over the
//      four row totals (readlane, multiplier M^16E) from the state entering
//      the block give every lane the state entering it, and the state after
//      the line's last element, F;
//   B. the cyclic closure x0 = (I - M^n)^{-1} F is the true state entering
//      the line; a lane's true incoming state is its zero-start state plus
//      M^(index of its first element) x0, and the lane reruns its recurrence
//      from it, which gives the true values directly.
// The backward recurrence is the same with the order of blocks, rows, lanes
// and elements reversed (closure z0 from the state after element 0), and its
// values leave scaled by 1/K.  Elements past the line's end are zero inputs;
// from a zero state they keep the state zero, so the top of a partial block
// needs no special case in the backward zero-start pass.  All powers of M
// come from a table computed on the host: M^k (k <= 256) and M^(256 c).
#include "wave_dev.h"

namespace mxs {

namespace {

// Ragged lines of every class in one launch, one wavefront each: positions
// first .. first + count - 1 of the sorted order, the class read from the
// line's length.  NBMAX (4 or 16): the largest class that the kernel holds
// registers for.  A batch that leaves the chip mostly idle takes the time of
// one launch and of one line's chain of loads and scans, so no wavefront gets
// a second line: with up to 16 short lines one after the other in a wavefront,
// 300 tridiagonal FP64 lines of 64 .. 1500 elements took 24.3 us, 3000 of
// 64 .. 4096 40.5 us; now 4.9 and 21 us.
template <typename T, int BW, int NBMAX>
__global__ void __launch_bounds__(64) wave_units_kernel(const RaggedLines a, int first, int count) {
    __shared__ __align__(16) T stage[Stage<T, WaveShape<NBMAX>::E>::SIZE];
    const int k = blockIdx.x;
    if (k >= count) return;
    const int b = as_global(a.order)[first + k];
    const gptr<const long long> offs = as_global(a.offsets);
    const long long n = offs[b + 1] - offs[b];
    const RaggedSrc<T> src{a};
    if constexpr (NBMAX == 16) {
        if (n > 8 * kWaveBlock) return wave_line<T, BW, 16>(src, first + k, stage);
        if (n > 4 * kWaveBlock) return wave_line<T, BW, 8>(src, first + k, stage);
    }
    if (n > 2 * kWaveBlock) wave_line<T, BW, 4>(src, first + k, stage);
    else if (n > kWaveBlock) wave_line<T, BW, 2>(src, first + k, stage);
    else wave_line<T, BW, 1>(src, first + k, stage);
}

// One ragged line of class NB per wavefront (positions first .. first +
// count - 1 of the sorted order): one launch per class, each with the
// registers of its own class.
template <typename T, int BW, int NB>
__global__ void __launch_bounds__(64) wave_ragged_kernel(const RaggedLines a, int first, int count) {
    __shared__ __align__(16) T stage[Stage<T, WaveShape<NB>::E>::SIZE];
    const int k = blockIdx.x;
    if (k >= count) return;
    wave_line<T, BW, NB>(RaggedSrc<T>{a}, first + k, stage);
}

template <typename T, int BW, int NB>
__global__ void __launch_bounds__(64) wave_rows_kernel(const RowsInst *__restrict__ inst,
                                                       const int *__restrict__ map, int first,
                                                       int count) {
    __shared__ __align__(16) T stage[Stage<T, WaveShape<NB>::E>::SIZE];
    const int k = blockIdx.x;
    if (k >= count) return;
    wave_line<T, BW, NB>(RowsSrc<T>{inst, map}, first + k, stage);
}

// A launch holds fewer than 2^32 threads and is cut off without an error beyond,
// so more lines than this go out in several.
constexpr int kLinesPerLaunch = 1 << 25;
template <class Launch> hipError_t in_pieces(int first, int count, Launch launch) {
    hipError_t e = hipSuccess;
    for (long long k = 0; k < count && e == hipSuccess; k += kLinesPerLaunch)
        e = launch(static_cast<int>(first + k), static_cast<int>(count - k < kLinesPerLaunch ? count - k : kLinesPerLaunch));
    return e;
}

template <typename T>
hipError_t units_bw(int bw, int nb, const RaggedLines &a, int first, int count, hipStream_t s) {
    const dim3 grid(count), block(64);
    if (bw == 2 && nb <= 4)
        hipLaunchKernelGGL((wave_units_kernel<T, 2, 4>), grid, block, 0, s, a, first, count);
    else if (bw == 2)
        hipLaunchKernelGGL((wave_units_kernel<T, 2, 16>), grid, block, 0, s, a, first, count);
    else if (nb <= 4)
        hipLaunchKernelGGL((wave_units_kernel<T, 1, 4>), grid, block, 0, s, a, first, count);
    else
        hipLaunchKernelGGL((wave_units_kernel<T, 1, 16>), grid, block, 0, s, a, first, count);
    return hipGetLastError();
}

template <typename T, int BW>
hipError_t ragged_nb(int nb, const RaggedLines &a, int first, int count, hipStream_t s) {
    const dim3 grid(count), block(64);
    switch (nb) {
    case 1: hipLaunchKernelGGL((wave_ragged_kernel<T, BW, 1>), grid, block, 0, s, a, first, count); break;
    case 2: hipLaunchKernelGGL((wave_ragged_kernel<T, BW, 2>), grid, block, 0, s, a, first, count); break;
    case 4: hipLaunchKernelGGL((wave_ragged_kernel<T, BW, 4>), grid, block, 0, s, a, first, count); break;
    case 8: hipLaunchKernelGGL((wave_ragged_kernel<T, BW, 8>), grid, block, 0, s, a, first, count); break;
    case 16: hipLaunchKernelGGL((wave_ragged_kernel<T, BW, 16>), grid, block, 0, s, a, first, count); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename T, int BW>
hipError_t rows_nb(int nb, const RowsInst *inst, const int *map, int first, int count, hipStream_t s) {
    const dim3 grid(count), block(64);
    switch (nb) {
    case 1: hipLaunchKernelGGL((wave_rows_kernel<T, BW, 1>), grid, block, 0, s, inst, map, first, count); break;
    case 2: hipLaunchKernelGGL((wave_rows_kernel<T, BW, 2>), grid, block, 0, s, inst, map, first, count); break;
    case 4: hipLaunchKernelGGL((wave_rows_kernel<T, BW, 4>), grid, block, 0, s, inst, map, first, count); break;
    case 8: hipLaunchKernelGGL((wave_rows_kernel<T, BW, 8>), grid, block, 0, s, inst, map, first, count); break;
    case 16: hipLaunchKernelGGL((wave_rows_kernel<T, BW, 16>), grid, block, 0, s, inst, map, first, count); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename T>
hipError_t rows_bw(int bw, int nb, const RowsInst *inst, const int *map, int first, int count,
                   hipStream_t s) {
    return bw == 2 ? rows_nb<T, 2>(nb, inst, map, first, count, s)
                   : rows_nb<T, 1>(nb, inst, map, first, count, s);
}

}  // namespace

hipError_t launch_wave_units(int dtype, int bw, int nb, const RaggedLines &a, int first, int count,
                             hipStream_t s) {
    if (bw != 1 && bw != 2) return hipErrorInvalidValue;
    return in_pieces(first, count, [&](int k, int n) {
        switch (dtype) {
        case F64: return units_bw<double>(bw, nb, a, k, n, s);
        case F32: return units_bw<float>(bw, nb, a, k, n, s);
        case BF16: return units_bw<bf16>(bw, nb, a, k, n, s);
        default: return hipErrorInvalidValue;
        }
    });
}

hipError_t launch_wave_ragged(int dtype, int bw, int nb, const RaggedLines &a, int first, int count,
                              hipStream_t s) {
    if (bw != 1 && bw != 2) return hipErrorInvalidValue;
    return in_pieces(first, count, [&](int k, int n) {
        switch (dtype) {
        case F64: return bw == 2 ? ragged_nb<double, 2>(nb, a, k, n, s) : ragged_nb<double, 1>(nb, a, k, n, s);
        case F32: return bw == 2 ? ragged_nb<float, 2>(nb, a, k, n, s) : ragged_nb<float, 1>(nb, a, k, n, s);
        case BF16: return bw == 2 ? ragged_nb<bf16, 2>(nb, a, k, n, s) : ragged_nb<bf16, 1>(nb, a, k, n, s);
        default: return hipErrorInvalidValue;
        }
    });
}

hipError_t launch_wave_rows(int dtype, int bw, int nb, const RowsInst *inst, const int *map, int first,
                            int count, hipStream_t s) {
    return in_pieces(first, count, [&](int k, int n) {
        switch (dtype) {
        case F64: return rows_bw<double>(bw, nb, inst, map, k, n, s);
        case F32: return rows_bw<float>(bw, nb, inst, map, k, n, s);
        case BF16: return rows_bw<bf16>(bw, nb, inst, map, k, n, s);
        default: return hipErrorInvalidValue;
        }
    });
}

}  // namespace mxs
