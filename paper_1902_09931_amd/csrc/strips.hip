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

namespace {

// Most columns for which strips are used instead of the three phases, by the
// columns' mean rows.  Once the CUs are full a strip of 16 columns takes 10 ns
// (tridiagonal) or 16 (pentadiagonal) however few rows it has, and moves short
// pieces of many rows; the phases take about 6 (double), 3.5 (float) or 2.2 ps
// (bfloat16) per point, but 9 to 12 us for their three launches.  So strips are
// for few columns, and for many only with rows enough.  Phases / strips, us:
//   plain solves: pentadiagonal double  4096 columns x 32 rows 10.4 / 8.4,
//     16384 x 64 11.7 / 20.3, 16384 x 320 31.3 / 25.7, 131072 x 200 145 / 177,
//     131072 x 400 293 / 220, 10^6 x 8 101 / 981;  tridiagonal float 8192 x 64
//     9.6 / 7.6, 16384 x 64 9.4 / 12.8, 32768 x 400 41.8 / 33.2;  pentadiagonal
//     float 8192 x 256 11.9 / 12.4, 16384 x 256 15.7 / 22.4, 32768 x 512 47.7 /
//     46.8, 32768 x 1200 113 / 165;  pentadiagonal bfloat16 6000 x 64 11.7 / 11.2,
//     12000 x 256 16.6 / 18.8, 6000 x 1200 35.2 / 39.7
//   Cahn-Hilliard steps (8192 columns are one round of two workgroups per CU):
//     double 64 x 64 14.0 / 11.1, 1024 x 64 19.5 / 12.9;  float 4 grids of 2048
//     columns x 64 rows 20.5 / 21.9, x 100 24.1 / 22.9, 9 of 1024 x 100 21.2 /
//     24.6;  double 4 of 4096 x 65 31 / 41, x 256 64 / 60, 16 of 4096 x 256 238 /
//     252, x 400 376 / 353;  float 64 of 256 x 256 34 / 40, of 1024 x 512 235 /
//     246, of 1024 x 700 335 / 322;  bfloat16 64 of 1024 x 700 280 / 288
struct ColumnLimit {
    int rows;            // for columns of fewer rows than this
    long long columns;
};
constexpr long long kAny = 1LL << 40;

long long columns_max(int dtype, int bw, int epilogue, long long rows) {
    static constexpr ColumnLimit plain[3][2][5] = {
        {{{200, 10000}, {2049, kAny}}, {{150, 7000}, {320, 10000}, {2049, kAny}}},                  // double
        {{{150, 10000}, {400, 14000}, {2049, kAny}}, {{150, 5000}, {512, 9000}, {1025, kAny}, {2049, 9000}}},
        {{{320, 10000}, {800, 20000}, {2049, 10000}}, {{1025, 9000}, {2049, 5000}}},                // bfloat16
    };
    static constexpr ColumnLimit update[3][5] = {
        {{256, 8192}, {320, 20000}, {2049, kAny}},
        {{65, 5000}, {400, 8192}, {600, 20000}, {1025, kAny}, {2049, 8192}},
        {{600, 8192}, {1025, 20000}, {2049, 8192}},
    };
    const ColumnLimit *l = epilogue ? update[dtype] : plain[dtype][bw - 1];
    for (int k = 0; k < 5; ++k)
        if (rows < l[k].rows) return l[k].columns;
    return 0;
}

}  // namespace

// Shapes, measured on FP64 grids, Cahn-Hilliard update, three phases against
// strips: 512^2 14.8 / 6.5 us (shape 0), 1024^2 19.0 / 12.4 (1; shape 2: 17),
// 2500 x 700 27.4 / 17.5 (2; shape 1: 20.5), 8000 x 1000 63.8 / 57.9 (2; shape
// 1: 90), 3000 x 2000 68.8 / 53.7 (3; shape 4: 57), 1536^2 38.9 / 33.5 (4;
// shape 3: 40), 2048^2 43.8 / 47.8 (4), 2051 x 3000 75 / 90 (1024 threads of
// 32 rows, 8 columns).  The plain solve, which has half the words to move,
// gains more (2048^2 27.6 / 19.2).  From 64 segments on the phases give a
// column 16 threads instead of 4 in their middle one, and the update of few
// columns of 2017 .. 2048 rows goes to them (steps of 512 x 2048 double 31.1 /
// 33.9 us, of 1024 x 2048 float 28.3 / 30.8, double 43.6 / 40.1).
int strip_shape_for(int ny_max, long long sum_nx, long long points, int x_dtype, int bw, int epilogue) {
    if (ny_max > 2048 || sum_nx > columns_max(x_dtype, bw, epilogue, points / sum_nx)) return -1;
    if (ny_max <= 1024) return sum_nx >= 2048 ? 2 : ny_max <= 512 ? 0 : 1;
    if (sum_nx >= 2800) return 3;
    if (epilogue && sum_nx * ny_max > 3000000) return -1;
    if (epilogue && cols_b_groups((ny_max + kSeg - 1) / kSeg) == 16 && (x_dtype != F64 || sum_nx < 768)) return -1;
    return 4;
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
