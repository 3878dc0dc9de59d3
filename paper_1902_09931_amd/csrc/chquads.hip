// The x sweep of the ADI Cahn-Hilliard step with its right-hand side formed
// inside the row solves (chrows.hip states the operator), for rows whose
// length is a multiple of 4: a workgroup takes 4 consecutive rows of one
// instance and every thread the 4 columns of one quad; rows of more than 2048
// elements (LPR = 256 below) 2 rows and two quads per thread.
//
// Right-hand side: a thread reads its quad of the 8 (or 6) input rows j0 - 2 ..
// j0 + 5 (the rows' windows along y), 16 or 32 bytes per row and time level,
// and walks them with one accumulator per output value.  Its x neighbours
// (two columns on each side) are the neighbouring lanes' values, moved by
// wavefront shifts; the two ends of a wavefront take theirs from 32 halo
// values that its lanes load beside the quads.  Nothing but the finished R
// goes through LDS: 16 bytes per point and direction instead of the 140
// bytes of reading every window from staged rows.
//
// Solve: R is stored to LDS in the line solver's order and every thread
// solves with 16 elements of one row (groups_dev.h: LPR = 16 .. 256 lanes
// per row, so a workgroup has 4 LPR threads, 2 LPR at 256, and long rows take
// more wavefronts, not more registers); the solution returns through the same LDS
// space and leaves as whole quads.
#include "ch_dev.h"
#include "groups_dev.h"

namespace mxs {

namespace {

// Address of a byte offset from a uniform base (one 32-bit register per lane).
template <typename T> __device__ __forceinline__ gptr<T> at_byte(gptr<T> base, unsigned o) {
    using C = std::conditional_t<std::is_const<T>::value, const char, char>;
    return (gptr<T>)((gptr<C>)base + o);
}

// 4 consecutive values from global memory (16-byte aligned; 8 for bfloat16)
__device__ __forceinline__ void load4(gptr<const double> p, double *x) {
    load_vec<double>(p, x);
    load_vec<double>(p + 2, x + 2);
}
__device__ __forceinline__ void load4(gptr<const float> p, float *x) { load_vec<float>(p, x); }
__device__ __forceinline__ void load4(gptr<const bf16> p, float *x) {
    const v2u_t v = *reinterpret_cast<gptr<const v2u_t>>(p);
    x[0] = __uint_as_float(v.x << 16);
    x[1] = __uint_as_float(v.x & 0xffff0000u);
    x[2] = __uint_as_float(v.y << 16);
    x[3] = __uint_as_float(v.y & 0xffff0000u);
}
__device__ __forceinline__ void store4(gptr<double> p, const double *x) {
    store_vec<double>(p, x);
    store_vec<double>(p + 2, x + 2);
}
__device__ __forceinline__ void store4(gptr<float> p, const float *x) { store_vec<float>(p, x); }

// 4 consecutive values from / to LDS (16-byte aligned)
__device__ __forceinline__ void lds4(const double *p, double *x) {
    const v2d_t a = *reinterpret_cast<const v2d_t *>(p), b = *reinterpret_cast<const v2d_t *>(p + 2);
    x[0] = a.x; x[1] = a.y; x[2] = b.x; x[3] = b.y;
}
__device__ __forceinline__ void lds4(const float *p, float *x) {
    const v4f_t a = *reinterpret_cast<const v4f_t *>(p);
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
}
__device__ __forceinline__ void lds4_set(double *p, const double *x) {
    *reinterpret_cast<v2d_t *>(p) = v2d_t{x[0], x[1]};
    *reinterpret_cast<v2d_t *>(p + 2) = v2d_t{x[2], x[3]};
}
__device__ __forceinline__ void lds4_set(float *p, const float *x) {
    *reinterpret_cast<v4f_t *>(p) = v4f_t{x[0], x[1], x[2], x[3]};
}

// The previous (0x138) or next (0x130) lane's v; the wavefront's end lane,
// which has no such neighbour, gets `end`.
template <int CTRL> __device__ __forceinline__ float lane_shift(float v, float end) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(end), __float_as_int(v), CTRL, 0xf, 0xf, false));
}
template <int CTRL> __device__ __forceinline__ double lane_shift(double v, double end) {
    const long long b = __double_as_longlong(v), o = __double_as_longlong(end);
    const int lo = __builtin_amdgcn_update_dpp(static_cast<int>(o), static_cast<int>(b), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(static_cast<int>(o >> 32), static_cast<int>(b >> 32), CTRL, 0xf, 0xf, false);
    return __longlong_as_double(static_cast<long long>((static_cast<unsigned long long>(static_cast<unsigned>(hi)) << 32) |
                                                       static_cast<unsigned>(lo)));
}
constexpr int kPrevLane = 0x138, kNextLane = 0x130;

// k mod n for -n <= k < 2 n (rows and columns reach at most 5 past either
// end, and both extents are at least 8)
__device__ __forceinline__ int wrap_near(int k, int n) { return k < 0 ? k + n : k >= n ? k - n : k; }

// Rows per workgroup: 4, or 2 where 4 rows of the longest class would leave
// room for one workgroup per CU only.
template <int LPR> constexpr int kQuadRows = LPR == 256 ? 2 : 4;

// LDS of a workgroup: its rows as LPR chunks of 16 values (each followed by
// 16 bytes of padding), then the rows' exchange space of the line solver.
template <typename TW, int LPR> struct QuadLds {
    static constexpr int CH = kGroupE + 16 / static_cast<int>(sizeof(TW));
    static constexpr int ROW = LPR * CH;
    static constexpr size_t xch = sizeof(TW) * kQuadRows<LPR> * ROW;
    static constexpr size_t bytes = xch + sizeof(double2) * kQuadRows<LPR> * kGroupXch<LPR>;
};

// Wavefronts per SIMD the registers are bounded to: double holds 4 (128
// registers, no spills), float 5 with 3 rows requested ahead (94 registers;
// 4096^2 131.5 -> 128.6 us a step, 64-grid ensemble 248 -> 245; at 6, or 5 in
// double, the kernel spills and loses 15 to 25%).
template <typename T> constexpr int kQuadWaves = sizeof(T) == 8 ? 4 : 5;

template <typename T, typename TW, int LPR>
__global__ void __launch_bounds__(kQuadRows<LPR> *LPR, kQuadWaves<T>) ch_quads_kernel(const RhsInst *__restrict__ rhs,
                                                                       const RowsInst *__restrict__ rows,
                                                                       const RowGroup *__restrict__ work, int count) {
    using A = typename St<T>::acc;
    using Lds = QuadLds<TW, LPR>;
    constexpr int WR = kQuadRows<LPR>, GIN = WR + 4, CH = Lds::CH, NT = WR * LPR;
    constexpr int QPT = 4 * LPR / NT;      // quads per thread, NT apart
    constexpr bool ONE = NT <= 64;         // one wavefront per workgroup
    // Input rows requested ahead of the one being used.
    constexpr int AHEAD = sizeof(A) == 8 ? 2 : 3;
    // In double the terms of a value are added as their rows arrive.  In
    // float every value is summed in the order of ch_rhs_rows_kernel (the 13
    // taps, then the 5, then the difference), so that both kernels round
    // alike and a grid's float states do not depend on its width mod 4.
    constexpr bool ORDERED = sizeof(A) == 4;

    extern __shared__ __align__(16) unsigned char smem_raw[];
    TW *tile = reinterpret_cast<TW *>(smem_raw);

    const RowGroup g = work[xcd_tile(blockIdx.x, count)];
    const RhsInst &I = rhs[g.inst];
    const RowsInst &RI = rows[g.inst];
    const int t = threadIdx.x, lane = t & 63;
    const int nx = I.nx, ny = I.ny, j0 = g.j0;
    const gptr<const T> cur = as_global(static_cast<const T *>(I.cur));
    const gptr<const T> prev = as_global(static_cast<const T *>(I.prev));
    const int nq = nx >> 2;                        // quads per row

    A wb[25], wl[9];
#pragma unroll
    for (int k = 0; k < 25; ++k) wb[k] = bih_tap(k / 5, k % 5) ? wb_of<A>(I, k) : A(0);
#pragma unroll
    for (int k = 0; k < 9; ++k) wl[k] = lap_tap(k / 3, k % 3) ? wl_of<A>(I, k) : A(0);
    const A cdiff = cd_of<A>(I);
    long long roff[GIN];                           // offsets of the input rows j0 - 2 .. j0 + WR + 1
#pragma unroll
    for (int u = 0; u < GIN; ++u) roff[u] = static_cast<long long>(wrap_near(j0 - 2 + u, ny)) * nx;

#pragma unroll
    for (int h = 0; h < QPT; ++h) {
        const int qd = t + h * NT;                 // the thread's quad
        const int q0 = __builtin_amdgcn_readfirstlane(qd - lane);   // the wavefront's first
        const bool valid = qd < nq;
        TW *mine = tile + (qd >> 2) * CH + 4 * (qd & 3);
        A acc[WR][4];
#pragma unroll
        for (int r = 0; r < WR; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[r][i] = A(0);

        if (q0 < nq) {
            const int lv = min(63, nq - 1 - q0);   // the wavefront's last lane with a quad
            // lanes past the row's end load its first quad: the first of them
            // is then the right neighbour of the row's last quad
            const unsigned ob = (valid ? 4u * static_cast<unsigned>(qd) : 0u) * sizeof(T);

            // halo: lanes 0 .. 4 GIN - 1 load column slot lane % 4 (two
            // before the wavefront's first column, two after its 64 quads or
            // the row's last) of input row lane / 4
            const int hu = min(lane >> 2, GIN - 1), hh = lane & 3;
            const int hc = wrap_near(hh < 2 ? 4 * q0 - 2 + hh : 4 * (q0 + lv) + 2 + hh, nx);
            const long long ho = static_cast<long long>(wrap_near(j0 - 2 + hu, ny)) * nx + hc;
            const A hcv = to_acc<T>(gld<T>(cur, ho)), hpv = to_acc<T>(gld<T>(prev, ho));

            A c[GIN][4], q[GIN][4];
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                load4(at_byte(cur + roff[u], ob), c[u]);
                load4(at_byte(prev + roff[u], ob), q[u]);
            }

            // the halo values to the wavefront's end lanes, through LDS space
            // that only this wavefront uses until the tile is complete: slots
            // [row][4] of Cbar, then of C^3 - C
            A *hal = reinterpret_cast<A *>(tile + (q0 >> 2) * CH);
            static_assert(2 * 32 * sizeof(A) <= 16 * CH * sizeof(TW), "halo values fit the wavefront's part of a row");
            if (lane < 4 * GIN) {
                hal[lane] = A(2) * hcv - hpv;
                hal[32 + lane] = hcv * hcv * hcv - hcv;
            }
            wave_sync();
            A fx[ORDERED ? GIN : 1][6], dv[ORDERED ? GIN : 1][4];
#pragma unroll
            for (int u = 0; u < GIN; ++u) {
                if (u + AHEAD < GIN) {
                    load4(at_byte(cur + roff[u + AHEAD], ob), c[u + AHEAD]);
                    load4(at_byte(prev + roff[u + AHEAD], ob), q[u + AHEAD]);
                }
                __builtin_amdgcn_sched_barrier(0);
                A x[8], f[6];   // Cbar at the quad and two columns on each side; C^3 - C with one
#pragma unroll
                for (int i = 0; i < 4; ++i) x[2 + i] = A(2) * c[u][i] - q[u][i];
                x[0] = x[1] = x[6] = x[7] = A(0);
                f[0] = f[5] = A(0);
#pragma unroll
                for (int i = 0; i < 4; ++i) f[1 + i] = A(0);
                if (u >= 1 && u < GIN - 1) {
                    A hb[4];   // the row's halo: two columns before lane 0, two after lane 63
                    lds4(hal + 4 * u, hb);
                    x[1] = lane_shift<kPrevLane>(x[5], hb[1]);
                    x[6] = lane_shift<kNextLane>(x[2], hb[2]);
                    if (u >= 2 && u < GIN - 2) {
                        x[0] = lane_shift<kPrevLane>(x[4], hb[0]);
                        x[7] = lane_shift<kNextLane>(x[3], hb[3]);
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) f[1 + i] = c[u][i] * c[u][i] * c[u][i] - c[u][i];
                    if (u >= 2 && u < GIN - 2) {
                        A hf[4];
                        lds4(hal + 32 + 4 * u, hf);
                        f[0] = lane_shift<kPrevLane>(f[4], hf[1]);
                        f[5] = lane_shift<kNextLane>(f[1], hf[2]);
                    }
                }
                if constexpr (ORDERED) {
#pragma unroll
                    for (int i = 0; i < 6; ++i) fx[u][i] = f[i];
#pragma unroll
                    for (int i = 0; i < 4; ++i) dv[u][i] = c[u][i] - q[u][i];
                }
#pragma unroll
                for (int r = 0; r < WR; ++r) {
                    const int s = u - r;   // window row of input row u for output row r
                    if (s < 0 || s > 4) continue;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int pp = 0; pp < 5; ++pp)
                            if (bih_tap(s, pp)) acc[r][i] = fma(wb[s * 5 + pp], x[i + pp], acc[r][i]);
                    if constexpr (ORDERED) {
                        if (s != 4) continue;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
#pragma unroll
                            for (int k = 0; k < 3; ++k)
#pragma unroll
                                for (int pp = 0; pp < 3; ++pp)
                                    if (lap_tap(k, pp))
                                        acc[r][i] = fma(wl[k * 3 + pp], fx[r + 1 + k][i + pp], acc[r][i]);
                            acc[r][i] = fma(cdiff, dv[r + 2][i], acc[r][i]);
                        }
                    } else {
                        if (s < 1 || s > 3) continue;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
#pragma unroll
                            for (int pp = 0; pp < 3; ++pp)
                                if (lap_tap(s - 1, pp)) acc[r][i] = fma(wl[(s - 1) * 3 + pp], f[i + pp], acc[r][i]);
                            if (s == 2) acc[r][i] = fma(cdiff, c[u][i] - q[u][i], acc[r][i]);
                        }
                    }
                }
            }
        }

        // R to LDS, zero past the row's end
        wave_sync();
        if (!valid) {
#pragma unroll
            for (int r = 0; r < WR; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[r][i] = A(0);
        }
#pragma unroll
        for (int r = 0; r < WR; ++r) {
            TW x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = static_cast<TW>(acc[r][i]);
            lds4_set(mine + r * Lds::ROW, x);
        }
    }
    if constexpr (ONE) wave_sync();
    else __syncthreads();

    // 16 elements of one row per thread
    const int r = t / LPR, li = t % LPR;
    TW *chunk = tile + r * Lds::ROW + li * CH;
    double v[kGroupE];
#pragma unroll
    for (int k = 0; k < kGroupE; k += 4) {
        TW x[4];
        lds4(chunk + k, x);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[k + i] = to_f64<TW>(x[i]);
    }
    double2 *xch = reinterpret_cast<double2 *>(smem_raw + Lds::xch) + r * kGroupXch<LPR>;
    group_solve<LPR>(v, nx, li, LineCoef{RI.p1, RI.p2, RI.pow}, xch);
    const double invK = RI.invK;
#pragma unroll
    for (int k = 0; k < kGroupE; k += 4) {
        TW x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = from_f64<TW>(v[k + i] * invK);
        lds4_set(chunk + k, x);
    }
    if constexpr (ONE) wave_sync();
    else __syncthreads();
    const gptr<TW> out = as_global(static_cast<TW *>(RI.out));
#pragma unroll
    for (int h = 0; h < QPT; ++h) {
        const int qd = t + h * NT;
        const TW *mine = tile + (qd >> 2) * CH + 4 * (qd & 3);
#pragma unroll
        for (int k = 0; k < WR; ++k) {
            TW x[4];
            lds4(mine + k * Lds::ROW, x);
            if (qd < nq && j0 + k < ny)
                store4(at_byte(out + (j0 + k) * RI.ld, 4u * static_cast<unsigned>(qd) * static_cast<unsigned>(sizeof(TW))), x);
        }
    }
}

template <typename T, typename TW, int LPR>
hipError_t quads_lpr(const RhsInst *rhs, const RowsInst *rows, const RowGroup *work, int count, hipStream_t s) {
    hipLaunchKernelGGL((ch_quads_kernel<T, TW, LPR>), dim3(count), dim3(kQuadRows<LPR> * LPR),
                       (QuadLds<TW, LPR>::bytes), s, rhs, rows, work, count);
    return hipGetLastError();
}

template <typename T, typename TW>
hipError_t quads_nb(int nb, const RhsInst *rhs, const RowsInst *rows, const RowGroup *work, int count,
                    hipStream_t s) {
    switch (nb) {
    case 1: return quads_lpr<T, TW, 16>(rhs, rows, work, count, s);
    case 2: return quads_lpr<T, TW, 32>(rhs, rows, work, count, s);
    case 4: return quads_lpr<T, TW, 64>(rhs, rows, work, count, s);
    case 8: return quads_lpr<T, TW, 128>(rhs, rows, work, count, s);
    case 16: return quads_lpr<T, TW, 256>(rhs, rows, work, count, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

int ch_quad_rows(int nb) { return nb == 16 ? 2 : 4; }

hipError_t launch_ch_quads(int state_dtype, int nb, const RhsInst *rhs, const RowsInst *rows, const RowGroup *work,
                           int count, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    switch (state_dtype) {
    case F64: return quads_nb<double, double>(nb, rhs, rows, work, count, s);
    case F32: return quads_nb<float, float>(nb, rhs, rows, work, count, s);
    case BF16: return quads_nb<bf16, float>(nb, rhs, rows, work, count, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace mxs
