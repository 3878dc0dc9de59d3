// Batched 1D stencils over uneven signals stored back to back (the batched
// 1D form of the abstract).
//
// The concatenated array is cut into equal tiles of W = threads * V * U
// elements (U = kS1dVecs vectors per thread),
// regardless of where signals begin and end, so every workgroup moves the
// same number of bytes whatever the length mix.  One workgroup per tile (the
// launch is a single sweep over the array, like a copy): it stages the
// values (plus an x halo of PAD elements each side) and the slice of signal
// offsets that meets the tile in LDS, requesting all three at once.  Each
// vector of outputs finds its signal by binary search in that slice.
// Outputs whose window stays inside their signal read LDS directly (a
// vector whose elements all do takes a straight-line path); the few near a
// signal end wrap within the signal (periodic) and read the wrapped value
// from LDS when it is staged, else from global memory.
//
// One source per storage type instantiates this (stencil1d_*.hip) for every
// number of taps, so that a window is never padded with taps of weight zero:
// past a signal's end they would read the next signal's values, and zero times
// an infinity or a NaN is a NaN.
#pragma once

#include "mxs_internal.h"

namespace mxs {

namespace {

template <typename A> __device__ __forceinline__ const A *coe_of(const Stencil1DArgs &a);
template <> __device__ __forceinline__ const double *coe_of<double>(const Stencil1DArgs &a) { return a.coe_d; }
template <> __device__ __forceinline__ const float *coe_of<float>(const Stencil1DArgs &a) { return a.coe_f; }

// Output vector stores: non-temporal for 8- and 2-byte elements, plain for
// FP32, whichever measured faster over the 65,536-signal batch (FP64 419
// against 433 us; FP32 250 against 254 us).
template <typename T> __device__ __forceinline__ void put_vec(T *p, const typename St<T>::acc *x) {
    if constexpr (sizeof(T) == 4) store_vec<T>(p, x);
    else store_vec_nt<T>(p, x);
}

template <int TAPS, int V> constexpr int halo_pad() {
    return TAPS > 1 ? ((TAPS - 1 + V - 1) / V) * V : 0;
}

// TAPS: the window's taps; U: vectors per thread; PER: whether signals wrap.
// Two kernels rather than a test in one: without the wrapped reads a thread
// holds 94 registers instead of 146 (17 taps in double), and 65,536 signals of
// 64 .. 4096 take 517 us instead of 555.
// (bfloat16 with the longest wrapped windows needs one register more than 4
// wavefronts per SIMD can have, unless it is told to: 436 us instead of 403.)
template <typename T, int TAPS, int U, bool PER>
__global__ void __launch_bounds__(256, sizeof(T) == 2 && PER && TAPS > 15 ? 4 : 1) stencil1d_kernel(const Stencil1DArgs a) {
    using A = typename St<T>::acc;
    constexpr int V = St<T>::V;
    constexpr int PAD = halo_pad<TAPS, V>();

    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int nt = blockDim.x;
    const int t = threadIdx.x;
    const int W = nt * V * U;
    A *lds = reinterpret_cast<A *>(smem_raw);
    long long *soff = reinterpret_cast<long long *>(smem_raw + ((static_cast<size_t>(2 * PAD + W) * sizeof(A) + 15) & ~static_cast<size_t>(15)));

    const T *__restrict__ in = static_cast<const T *>(a.in);
    T *__restrict__ out = static_cast<T *>(a.out);
    const A *__restrict__ w = static_cast<const A *>(a.wts);
    const A *coe = coe_of<A>(a);

    // one tile per workgroup: the values (U vectors per thread, each vector
    // of the workgroup adjacent to the next thread's), their halo and the
    // offsets of the signals meeting the tile are all requested before any
    // is used
    const int tile = blockIdx.x;
    const long long e0 = static_cast<long long>(tile) * W;
    const int b0 = a.tile_first[tile];
    const int cnt = a.tile_first[tile + 1] - b0 + 2;   // offsets b0 .. b_last+1
    A xv[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const long long eb = e0 + static_cast<long long>(u * nt + t) * V;
        if (eb + V <= a.total) {
            load_vec<T>(in + eb, xv[u]);
        } else {
#pragma unroll
            for (int v = 0; v < V; ++v) xv[u][v] = eb + v < a.total ? to_acc<T>(in[eb + v]) : A(0);
        }
    }
    A hv = A(0);
    if (t < 2 * PAD) {
        const long long c = t < PAD ? e0 - PAD + t : e0 + W + (t - PAD);
        if (c >= 0 && c < a.total) hv = to_acc<T>(in[c]);
    }
    for (int k = t; k < cnt; k += nt) soff[k] = a.offsets[b0 + k];
    if (a.ncoe) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int v = 0; v < V; ++v) xv[u][v] = point_fun<A>(xv[u][v], coe, a.ncoe);
        hv = point_fun<A>(hv, coe, a.ncoe);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int v = 0; v < V; ++v) lds[PAD + (u * nt + t) * V + v] = xv[u][v];
    if (t < 2 * PAD) lds[t < PAD ? t : W + t] = hv;
    __syncthreads();

#pragma unroll
    for (int u = 0; u < U; ++u) {
        const long long eb = e0 + static_cast<long long>(u * nt + t) * V;
        A res[V];
        bool wr[V];
        // the signal holding the vector's first element (binary search in
        // the tile's offsets); later elements of the vector step to the next
        // signal when they cross its start
        int lo = 0;
        {
            int hi = cnt - 2;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (soff[mid] <= eb) lo = mid; else hi = mid - 1;
            }
        }
        long long sb = soff[lo], se = soff[lo + 1];
        // the common case: the whole vector lies in one signal with every
        // window inside it (no wrap, every output written): straight-line
        // FMAs over the staged values
        if (eb >= sb + a.L && eb + V - 1 + a.R <= se - 1) {
            const A *lp = lds + PAD + (eb - e0) - a.L;
            A x[V + TAPS - 1];
#pragma unroll
            for (int k = 0; k < V + TAPS - 1; ++k) x[k] = lp[k];
#pragma unroll
            for (int v = 0; v < V; ++v) {
                A acc = A(0);
#pragma unroll
                for (int p = 0; p < TAPS; ++p) acc = fma(w[p], x[v + p], acc);
                res[v] = acc;
            }
            put_vec<T>(out + eb, res);
            continue;
        }
        // a vector that meets one signal end at most: its elements are in the
        // signal [sb, se) or in the next one, so two windows cover them, each
        // with the taps past its own signal's ends read from where they wrap
        // to; every such read is requested before any is used.  Without a wrap
        // the outputs nearest a signal's end are left out, and for long windows
        // the element path below, which skips them, is the faster one, but for
        // bfloat16 with its 8 elements per vector (500,000 signals of 20 .. 40,
        // 17 taps: double 108 us here, 90 there, float 57 and 53, bfloat16 55 and
        // 75; 7 taps in double 72 and 77).
        if ((PER || TAPS < 10 || sizeof(T) == 2) && eb + V <= a.total && (se >= eb + V || soff[lo + 2] >= eb + V)) {
            const bool cross = se < eb + V;
            const long long sb2 = cross ? se : sb, se2 = cross ? soff[lo + 2] : se;
            const A *lp = lds + PAD + (eb - e0) - a.L;
            A x[V + TAPS - 1], y[V + TAPS - 1];
#pragma unroll
            for (int k = 0; k < V + TAPS - 1; ++k) {
                x[k] = y[k] = lp[k];
                const long long idx = eb - a.L + k;
                if constexpr (PER) {
                    const long long ix = idx < sb ? idx + (se - sb) : idx >= se ? idx - (se - sb) : idx;
                    const long long iy = idx < sb2 ? idx + (se2 - sb2) : idx >= se2 ? idx - (se2 - sb2) : idx;
                    if (ix != idx) x[k] = to_acc<T>(in[ix]);
                    if (iy != idx) y[k] = to_acc<T>(in[iy]);
                }
            }
            if (PER && a.ncoe) {
#pragma unroll
                for (int k = 0; k < V + TAPS - 1; ++k) {
                    const long long idx = eb - a.L + k;
                    if (idx < sb || idx >= se) x[k] = point_fun<A>(x[k], coe, a.ncoe);
                    if (idx < sb2 || idx >= se2) y[k] = point_fun<A>(y[k], coe, a.ncoe);
                }
            }
            bool all = true;
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const bool second = eb + v >= se;
                A acc = A(0);
#pragma unroll
                for (int p = 0; p < TAPS; ++p) acc = fma(w[p], second ? y[v + p] : x[v + p], acc);
                res[v] = acc;
                const long long i = eb + v - (second ? sb2 : sb), n = second ? se2 - sb2 : se - sb;
                wr[v] = PER || (i >= a.L && i <= n - 1 - a.R);
                all = all && wr[v];
            }
            if (all) {
                put_vec<T>(out + eb, res);
            } else {
#pragma unroll
                for (int v = 0; v < V; ++v)
                    if (wr[v]) out[eb + v] = from_acc<T>(res[v]);
            }
            continue;
        }
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const long long e = eb + v;
            res[v] = A(0);
            wr[v] = false;
            if (e >= a.total) continue;
            while (e >= se) {
                ++lo;
                sb = se;
                se = soff[lo + 1];
            }
            const long long n = se - sb;
            const long long i = e - sb;
            if (!PER && (i < a.L || i > n - 1 - a.R)) continue;
            wr[v] = true;
            A acc = A(0);
            if (i >= a.L && i + a.R <= n - 1) {
                const A *lp = lds + PAD + (e - e0) - a.L;
#pragma unroll
                for (int p = 0; p < TAPS; ++p) acc = fma(w[p], lp[p], acc);
            } else {
                for (int p = 0; p < TAPS; ++p) {
                    long long ii = i + p - a.L;
                    if (ii < 0) ii += n;
                    else if (ii >= n) ii -= n;
                    const long long idx = sb + ii;
                    A val;
                    if (idx >= e0 - PAD && idx < e0 + W + PAD) {
                        val = lds[PAD + (idx - e0)];
                    } else {
                        val = to_acc<T>(in[idx]);
                        if (a.ncoe) val = point_fun<A>(val, coe, a.ncoe);
                    }
                    acc = fma(w[p], val, acc);
                }
            }
            res[v] = acc;
        }
        bool all = eb + V <= a.total;
#pragma unroll
        for (int v = 0; v < V; ++v) all = all && wr[v];
        if (all) {
            put_vec<T>(out + eb, res);
        } else {
#pragma unroll
            for (int v = 0; v < V; ++v)
                if (wr[v]) out[eb + v] = from_acc<T>(res[v]);
        }
    }
}

template <typename T, int TAPS>
hipError_t launch_one(const Stencil1DArgs &a, int threads, int grid, hipStream_t s) {
    size_t lds = stencil1d_lds_bytes(std::is_same<T, double>::value ? F64
                                           : std::is_same<T, float>::value ? F32 : BF16,
                                           TAPS, threads, a.max_sig_per_tile, a.vecs);
    if (a.vecs != kS1dVecs && a.vecs != 1) return hipErrorInvalidValue;
    // Two taps in double are so little work that 8 workgroups per CU get into
    // each other's way in memory: 65,536 signals of 64 .. 4096 take 374 us with
    // 8 or 9, 355 with 6, and 4 cost short signals (500,000 of 20 .. 40: 52, 54,
    // 60 us).
    if (sizeof(T) == 8 && TAPS == 2 && a.vecs == kS1dVecs) lds = lds > 26 * 1024 ? lds : 26 * 1024;
    const dim3 g(grid), b(threads);
    if (a.vecs == kS1dVecs && a.periodic)
        hipLaunchKernelGGL((stencil1d_kernel<T, TAPS, kS1dVecs, true>), g, b, lds, s, a);
    else if (a.vecs == kS1dVecs)
        hipLaunchKernelGGL((stencil1d_kernel<T, TAPS, kS1dVecs, false>), g, b, lds, s, a);
    else if (a.periodic)
        hipLaunchKernelGGL((stencil1d_kernel<T, TAPS, 1, true>), g, b, lds, s, a);
    else
        hipLaunchKernelGGL((stencil1d_kernel<T, TAPS, 1, false>), g, b, lds, s, a);
    return hipGetLastError();
}

template <typename T, int TAPS = kMaxTaps1D>
hipError_t dispatch(const Stencil1DArgs &a, int threads, int grid, hipStream_t s) {
    if (a.L + a.R + 1 == TAPS) return launch_one<T, TAPS>(a, threads, grid, s);
    if constexpr (TAPS > 1) return dispatch<T, TAPS - 1>(a, threads, grid, s);
    else return hipErrorInvalidValue;
}

}  // namespace
}  // namespace mxs
