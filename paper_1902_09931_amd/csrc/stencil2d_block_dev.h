// Device code and launches of the 2D stencils in block form: every input row
// of a workgroup's chunk requested at once.  One source per storage type
// instantiates it (stencil2d_block_*.hip).
#pragma once

#include "stencil2d_dev.h"

namespace mxs {
namespace {

// Value of the neighbouring lane across the whole wavefront: SHR gives lane
// i the value of lane i - 1, SHL the value of lane i + 1 (DPP wave shifts;
// the lane at the end of the wavefront receives 0).
template <int CTRL> __device__ __forceinline__ double wave_shift(double v) {
    const unsigned long long b = static_cast<unsigned long long>(__double_as_longlong(v));
    const unsigned lo = static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(b), CTRL, 0xf, 0xf, false));
    const unsigned hi = static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(b >> 32), CTRL, 0xf, 0xf, false));
    return __longlong_as_double(static_cast<long long>((static_cast<unsigned long long>(hi) << 32) | lo));
}
template <int CTRL> __device__ __forceinline__ float wave_shift(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
constexpr int kDppWaveShl1 = 0x130;
constexpr int kDppWaveShr1 = 0x138;

// Block form (windows of 3 or 5 rows, and of 9 along y alone): a workgroup requests all GIN input
// rows of its chunk at once, GIN - NWY + 1 output rows, stages them in LDS
// with their x halo (NWX > 1) and computes every output row of the chunk;
// there is no streaming loop, so every load of the workgroup is in flight
// together, as in a plain copy.  Neighbouring chunks both read the NWY - 1
// rows they share; with chunks of one strip dispatched close together the
// second read is served by L2.  Rows and columns outside a non-periodic grid
// are read from clamped addresses: they only meet outputs that are not
// written (or padded taps of weight zero).
//
// XS (x exchange by lanes, centred windows only: left = right = NWX / 2 <=
// V): the x neighbours of a thread's V values come from the neighbouring
// lanes by DPP wave shifts instead of an LDS row; the two lanes at the ends
// of a wavefront load their outside neighbours themselves.  No LDS, no
// barrier.
template <typename T, int NWX, int NWY, int GIN, bool CLEAN, bool XS>
__device__ __forceinline__ void block_body(const Stencil2DArgs &a, int strip, int chunk, unsigned char *smem) {
    using A = typename St<T>::acc;
    constexpr int V = St<T>::V;
    constexpr int PAD = halo_pad<NWX, V>();
    constexpr int XW = V + NWX - 1;
    constexpr int ROWS = GIN - NWY + 1;
    constexpr int HPT = (GIN * 2 * PAD + 63) / 64;
    A *lds = reinterpret_cast<A *>(smem);
    const gptr<const T> in = as_global(static_cast<const T *>(a.in));
    const gptr<T> out = as_global(static_cast<T *>(a.out));
    const A *__restrict__ w = static_cast<const A *>(a.wts);
    const A *coe = coe_of<A>(a);
    const int nt = blockDim.x;
    const int t = threadIdx.x;
    const int W = nt * V;
    const int rowlen = PAD + W + PAD;
    const long long lo = static_cast<long long>(strip) * W;   // first column stored (as in stencil2d_kernel)
    const long long i0 = CLEAN && lo + W > a.nx ? a.nx - W : lo;
    const int j0 = chunk * ROWS;
    const int H = min(ROWS, a.ny - j0);
    const long long ib = i0 + static_cast<long long>(t) * V;
    const bool periodic = a.periodic != 0;

    // grid row of input row u
    auto in_row = [&](int u) __attribute__((always_inline)) {
        long long r = static_cast<long long>(j0) - a.T + u;
        if (periodic) return wrap_fast(r, a.ny);
        return r < 0 ? 0LL : (r >= a.ny ? static_cast<long long>(a.ny) - 1 : r);
    };
    // Column c of a row, inside the grid.  In a strip wider than a periodic grid
    // the columns past the last window meet no output; they repeat one near
    // the end, as a column more than a period away takes a division (64^2 FP32,
    // 3 rows: 11.8 us with it, 9.3 without).
    const long long cmax = static_cast<long long>(a.nx) + NWX;
    auto wrap_col = [&](long long c) __attribute__((always_inline)) { return wrap_fast(CLEAN ? c : min(c, cmax), a.nx); };
    auto in_col = [&](long long c) __attribute__((always_inline)) {
        return periodic ? wrap_col(c) : (c < 0 ? 0 : (c >= a.nx ? a.nx - 1LL : c));
    };
    A xin[GIN][V];
    if constexpr (CLEAN) {
#pragma unroll
        for (int u = 0; u < GIN; ++u) load_vec<T>(in + in_row(u) * a.ld + ib, xin[u]);
    } else {
        auto elements = [&](auto col) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < GIN; ++u) {
                const gptr<const T> rowp = in + in_row(u) * a.ld;
#pragma unroll
                for (int v = 0; v < V; ++v) xin[u][v] = to_acc<T>(gld<T>(rowp, col(ib + v)));
            }
        };
        if (periodic) elements(wrap_col);
        else elements([&](long long c) { return c >= a.nx ? a.nx - 1LL : c; });
    }
    constexpr int HX = NWX / 2;   // lane exchange: neighbours on each side
    const int lane = t & 63;
    // lane exchange: lane 0 loads the HX values left of its vector, lane 63
    // the HX values right of it
    A ev[GIN][HX > 0 ? HX : 1];
    if constexpr (XS && HX > 0) {
        if (lane == 0 || lane == 63) {
#pragma unroll
            for (int u = 0; u < GIN; ++u) {
                const gptr<const T> rowp = in + in_row(u) * a.ld;
#pragma unroll
                for (int h = 0; h < HX; ++h)
                    ev[u][h] = to_acc<T>(gld<T>(rowp, in_col(lane == 0 ? ib - HX + h : ib + V + h)));
            }
        }
    }
    A hv[HPT > 0 ? HPT : 1];
    const int hcount = GIN * 2 * PAD;
#pragma unroll
    for (int q = 0; q < (XS ? 0 : HPT); ++q) {
        const int h = min(t + q * nt, hcount - 1);
        const int u = h / (2 * PAD);
        const int hh = h - u * 2 * PAD;
        const long long c = in_col(hh < PAD ? i0 - PAD + hh : i0 + W + (hh - PAD));
        hv[q] = to_acc<T>(gld<T>(in + in_row(u) * a.ld, c));
    }
    if (a.ncoe) {
        // Horner's rule, coefficient loop outside (one uniform load per
        // coefficient), the same operations per element as point_fun
        const A top = coe[a.ncoe - 1];
        A f[GIN][V], hf[HPT > 0 ? HPT : 1];
#pragma unroll
        for (int u = 0; u < GIN; ++u)
#pragma unroll
            for (int v = 0; v < V; ++v) f[u][v] = top;
        constexpr int HQ = XS ? 0 : HPT;
        constexpr int EQ = XS ? HX : 0;
        A ef[GIN][EQ > 0 ? EQ : 1];
#pragma unroll
        for (int q = 0; q < HQ; ++q) hf[q] = top;
#pragma unroll
        for (int u = 0; u < GIN; ++u)
#pragma unroll
            for (int h = 0; h < EQ; ++h) ef[u][h] = top;
        for (int m = a.ncoe - 2; m >= 0; --m) {
            const A cm = coe[m];
#pragma unroll
            for (int u = 0; u < GIN; ++u)
#pragma unroll
                for (int v = 0; v < V; ++v) f[u][v] = f[u][v] * xin[u][v] + cm;
#pragma unroll
            for (int q = 0; q < HQ; ++q) hf[q] = hf[q] * hv[q] + cm;
#pragma unroll
            for (int u = 0; u < GIN; ++u)
#pragma unroll
                for (int h = 0; h < EQ; ++h) ef[u][h] = ef[u][h] * ev[u][h] + cm;
        }
#pragma unroll
        for (int u = 0; u < GIN; ++u)
#pragma unroll
            for (int v = 0; v < V; ++v) xin[u][v] = f[u][v];
#pragma unroll
        for (int q = 0; q < HQ; ++q) hv[q] = hf[q];
#pragma unroll
        for (int u = 0; u < GIN; ++u)
#pragma unroll
            for (int h = 0; h < EQ; ++h) ev[u][h] = ef[u][h];
    }
    // lane exchange: the window of every input row, columns ib - HX ..
    // ib + V - 1 + HX
    A xw[XS ? GIN : 1][XS ? V + 2 * HX : 1];
    if constexpr (XS) {
#pragma unroll
        for (int u = 0; u < GIN; ++u) {
#pragma unroll
            for (int h = 0; h < HX; ++h) {
                const A l = wave_shift<kDppWaveShr1>(xin[u][V - HX + h]);
                const A r = wave_shift<kDppWaveShl1>(xin[u][h]);
                xw[u][h] = lane == 0 ? ev[u][h] : l;
                xw[u][HX + V + h] = lane == 63 ? ev[u][h] : r;
            }
#pragma unroll
            for (int v = 0; v < V; ++v) xw[u][HX + v] = xin[u][v];
        }
    }
    if constexpr (NWX > 1 && !XS) {
#pragma unroll
        for (int u = 0; u < GIN; ++u) {
            A *dst = lds + u * rowlen + PAD + t * V;
#pragma unroll
            for (int v = 0; v < V; ++v) dst[v] = xin[u][v];
        }
#pragma unroll
        for (int q = 0; q < HPT; ++q) {
            const int h = t + q * nt;
            if (h < hcount) {
                const int u = h / (2 * PAD);
                const int hh = h - u * 2 * PAD;
                lds[u * rowlen + (hh < PAD ? hh : W + hh)] = hv[q];
            }
        }
        __syncthreads();
    }
    const bool store_vec_ok = ib + V <= a.nx && ib >= lo &&
                              (periodic || (ib >= a.L && ib + V - 1 <= a.nx - 1 - a.R));
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
        A acc[V];
#pragma unroll
        for (int v = 0; v < V; ++v) acc[v] = A(0);
#pragma unroll
        for (int q = 0; q < NWY; ++q) {
            if constexpr (XS) {
#pragma unroll
                for (int p = 0; p < NWX; ++p) {
                    const A wt = w[q * NWX + p];
#pragma unroll
                    for (int v = 0; v < V; ++v) acc[v] = fma(wt, xw[k + q][v + p], acc[v]);
                }
            } else if constexpr (NWX > 1) {
                A x[XW];
                const A *lp = lds + (k + q) * rowlen + PAD + t * V - a.L;
#pragma unroll
                for (int m = 0; m < XW; ++m) x[m] = lp[m];
#pragma unroll
                for (int p = 0; p < NWX; ++p) {
                    const A wt = w[q * NWX + p];
#pragma unroll
                    for (int v = 0; v < V; ++v) acc[v] = fma(wt, x[v + p], acc[v]);
                }
            } else {
                const A wt = w[q];
#pragma unroll
                for (int v = 0; v < V; ++v) acc[v] = fma(wt, xin[k + q][v], acc[v]);
            }
        }
        const int j = j0 + k;
        if (k >= H || (!periodic && (j < a.T || j > a.ny - 1 - a.B))) continue;
        const gptr<T> rowp = out + static_cast<long long>(j) * a.ld;
        if (CLEAN && store_vec_ok) {
            if (a.nt_store) store_vec_nt<T>(rowp + ib, acc);
            else store_vec<T>(rowp + ib, acc);
        } else {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const long long c = ib + v;
                if (c >= lo && c < a.nx && (periodic || (c >= a.L && c <= a.nx - 1 - a.R)))
                    gst<T>(rowp, c, from_acc<T>(acc[v]));
            }
        }
    }
}

template <typename T, int NWX, int NWY, int GIN, bool XS>
__global__ void __launch_bounds__(256) stencil2d_block_kernel(const Stencil2DArgs a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    int strip, chunk;
    tile_of(a, strip, chunk);
    const long long W = static_cast<long long>(blockDim.x) * St<T>::V;
    // a row holds a whole strip: vector loads only
    if (W <= a.nx)
        block_body<T, NWX, NWY, GIN, true, XS>(a, strip, chunk, smem_raw);
    else
        block_body<T, NWX, NWY, GIN, false, XS>(a, strip, chunk, smem_raw);
}

template <typename T, int NWX, int NWY, int GIN>
hipError_t launch_block(const Stencil2DArgs &a, int threads, hipStream_t s) {
    using A = typename St<T>::acc;
    constexpr int V = St<T>::V;
    const int grid = a.nstrips * a.nchunks;
    if constexpr (NWX > 1 && NWX / 2 <= V) {
        if (a.xshuffle) {
            if (a.L != NWX / 2 || a.R != NWX / 2) return hipErrorInvalidValue;
            hipLaunchKernelGGL((stencil2d_block_kernel<T, NWX, NWY, GIN, true>), dim3(grid), dim3(threads), 0, s, a);
            return hipGetLastError();
        }
    }
    if (a.xshuffle) return hipErrorInvalidValue;
    if constexpr (NWY == 1) return hipErrorInvalidValue;
    else {
    const size_t lds = NWX > 1 ? static_cast<size_t>(GIN) * (2 * halo_pad<NWX, V>() + threads * V) * sizeof(A) : 0;
    hipLaunchKernelGGL((stencil2d_block_kernel<T, NWX, NWY, GIN, false>), dim3(grid), dim3(threads), lds, s, a);
    return hipGetLastError();
    }
}

template <typename T>
hipError_t dispatch_block(int nwx, int nwy, const Stencil2DArgs &a, int threads, hipStream_t s) {
#define MXS_BCASE(X, Y, G) \
    if (nwx == X && nwy == Y && a.block_rows == G) return launch_block<T, X, Y, G>(a, threads, s);
    MXS_BCASE(1, 3, 8) MXS_BCASE(1, 3, 12) MXS_BCASE(1, 3, 16)
    MXS_BCASE(1, 5, 8) MXS_BCASE(1, 5, 12) MXS_BCASE(1, 5, 16)
    MXS_BCASE(3, 3, 8) MXS_BCASE(3, 3, 12) MXS_BCASE(3, 3, 16)
    MXS_BCASE(3, 5, 8) MXS_BCASE(3, 5, 12) MXS_BCASE(3, 5, 16)
    MXS_BCASE(5, 3, 8) MXS_BCASE(5, 3, 12) MXS_BCASE(5, 3, 16)
    MXS_BCASE(5, 5, 8) MXS_BCASE(5, 5, 12) MXS_BCASE(5, 5, 16)
    // 9 taps along y: 8 output rows from 16 input rows.  In bfloat16 the 8
    // values per thread of every row would need 256 registers.
    if constexpr (sizeof(T) > 2) {
        MXS_BCASE(1, 9, 16)
    }
    // along x: no shared rows, so only the number of rows in flight differs
    if (a.xshuffle) {
        MXS_BCASE(3, 1, 4) MXS_BCASE(3, 1, 8)
        MXS_BCASE(5, 1, 4) MXS_BCASE(5, 1, 8)
        MXS_BCASE(9, 1, 4) MXS_BCASE(9, 1, 8)
    }
#undef MXS_BCASE
    return hipErrorInvalidValue;
}

}  // namespace
}  // namespace mxs
