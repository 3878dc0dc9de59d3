// 2D stencils in the x, y and xy directions, periodic or non-periodic, with
// fixed weights or a point function (Sec. 3, Sec. 4.1, Sec. 4.2).
//
// One kernel template covers every direction.  A workgroup owns a strip of
// W = threads * V columns and a chunk of `rows` output rows.  It streams the
// input rows of its chunk top to bottom; each thread keeps, per pending
// output row, an accumulator vector of V outputs in registers (NWY rows,
// shifted by one row as each output row completes).  When an input row arrives, its window along x (V + NWX - 1 values,
// read from an LDS copy of the row with its x halo, or straight from
// registers when NWX == 1) is multiplied into every pending output row it
// touches; the output row whose window is complete is written out.  Each
// input element is therefore read from HBM once per chunk (plus the NWY - 1
// halo rows shared with the chunk above), and each output element written
// once, with 8- or 16-byte vector accesses.
//
// The window is padded to the compiled widths NWX x NWY in {1,3,5,9,17};
// padded taps carry weight zero.  Weights live in device memory in the
// accumulation type and are read with uniform (scalar) loads.
#include "stencil2d_dev.h"

#include <type_traits>

namespace mxs {

namespace {

// Input rows loaded per round (into LDS when NWX > 1).
template <int NWY> constexpr int stage_rows() {
    return 4;
}

// Load element c of an input row, wrapping (periodic) or as zero when outside
// [0, nx) (non-periodic: such values never reach a written output).
template <typename T>
__device__ __forceinline__ typename St<T>::acc load_elem(const T *rowp, long long c, int nx,
                                                         bool periodic) {
    using A = typename St<T>::acc;
    if (c < 0 || c >= nx) {
        if (!periodic) return A(0);
        c = wrap_ll(c, nx);
    }
    return to_acc<T>(rowp[c]);
}

template <typename T, int NWX, int NWY>
__global__ void __launch_bounds__(256) stencil2d_kernel(const Stencil2DArgs a) {
    using A = typename St<T>::acc;
    constexpr int V = St<T>::V;
    constexpr int PAD = halo_pad<NWX, V>();
    constexpr int G = stage_rows<NWY>();
    constexpr int XW = V + NWX - 1;

    extern __shared__ __align__(16) unsigned char smem_raw[];
    A *lds = reinterpret_cast<A *>(smem_raw);

    const T *__restrict__ in = static_cast<const T *>(a.in);
    T *__restrict__ out = static_cast<T *>(a.out);
    const A *__restrict__ w = static_cast<const A *>(a.wts);
    const A *coe = coe_of<A>(a);

    const int nt = blockDim.x;
    const int t = threadIdx.x;
    const int W = nt * V;
    const int rowlen = PAD + W + PAD;
    int strip, chunk;
    tile_of(a, strip, chunk);
    // The last strip of a row starts early enough to lie inside the grid and
    // stores only the columns from lo on, the ones the strip before it leaves:
    // a strip that hangs over the grid's edge would go element by element.
    const long long lo = static_cast<long long>(strip) * W;
    const long long i0 = a.nx >= W && lo + W > a.nx ? a.nx - W : lo;
    const int j0 = chunk * a.rows;
    const int H = min(a.rows, a.ny - j0);
    const int niter = H + NWY - 1;
    const long long ib = i0 + static_cast<long long>(t) * V;
    const bool periodic = a.periodic != 0;
    // Odd chunks walk their rows bottom to top (the window flipped
    // vertically), so the halo rows two neighbouring chunks share are read
    // by both at about the same time and the second read hits in L2.
    const bool up = (chunk & 1) != 0;
    // first input row, and the step between input rows
    const long long rfirst = up ? static_cast<long long>(j0) + H - 1 + a.B : static_cast<long long>(j0) - a.T;
    const int rstep = up ? -1 : 1;
    // upward chunks use the vertically flipped weights (uploaded by the plan)
    const A *__restrict__ wv = up ? static_cast<const A *>(a.wts_up) : w;
    const bool full_vec = ib + V <= a.nx;
    const bool store_vec_ok = full_vec && ib >= lo && (periodic || (ib >= a.L && ib + V - 1 <= a.nx - 1 - a.R));
    // A vector that is not stored whole is stored element by element, those from
    // v0 up to v1.  In bfloat16 windows of several columns and 3 rows need 156
    // registers so, and 169 with a test of every column, one more than 3
    // wavefronts per SIMD can have (4096^2, 5 x 3: 35.5 us with 3 of them, 40.8
    // with 2); other kernels do with fewer registers with the test.
    constexpr bool BY_INDEX = sizeof(T) == 2 && NWX > 1 && NWY == 3;
    int v0 = 0, v1 = 0;
    if constexpr (BY_INDEX) {
        v0 = static_cast<int>(max((periodic ? lo : max(lo, static_cast<long long>(a.L))) - ib, 0LL));
        v1 = static_cast<int>(min(a.nx - (periodic ? 0 : a.R) - ib, static_cast<long long>(V)));
    }

    A acc[NWY][V];
#pragma unroll
    for (int q = 0; q < NWY; ++q)
#pragma unroll
        for (int v = 0; v < V; ++v) acc[q][v] = A(0);

    // Halo values per stage: G rows x 2*PAD columns, at most HPT per thread.
    constexpr int HPT = (G * 2 * PAD + 63) / 64;
    const int hcount = G * 2 * PAD;

    // A stage is "clean" when all its G rows exist (periodic, or inside the
    // grid) and the strip lies inside the grid: its
    // loads are then issued as straight-line code with no alternative path
    // writing the same registers, so none of them waits for the others (or
    // for earlier stores); halo values outside a non-periodic grid are loaded
    // from a clamped address and zeroed when staged.
    const bool strip_clean = i0 + W <= a.nx;
    auto clean_stage = [&](int s0) __attribute__((always_inline)) {
        if (!strip_clean || s0 + G > niter) return false;
        if (periodic) return true;
        const long long ra = rfirst + static_cast<long long>(rstep) * s0;
        const long long rb = rfirst + static_cast<long long>(rstep) * (s0 + G - 1);
        return (ra < rb ? ra : rb) >= 0 && (ra > rb ? ra : rb) < a.ny;
    };
    // halo slot h of a stage: its row within the stage and its column
    auto halo_slot = [&](int h, int &u, long long &c) __attribute__((always_inline)) {
        u = h / (2 * PAD);
        const int hh = h - u * 2 * PAD;
        c = hh < PAD ? i0 - PAD + hh : i0 + W + (hh - PAD);
    };

    // Loads of a clean stage s0 (main vectors and halo values) into registers.
    auto load_clean = [&](int s0, A (&xin)[G][V], A (&hv)[HPT > 0 ? HPT : 1]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < G; ++u) {
            long long r = rfirst + static_cast<long long>(rstep) * (s0 + u);
            if (periodic) r = wrap_fast(r, a.ny);
            load_vec<T>(in + r * a.ld + ib, xin[u]);
        }
        if constexpr (NWX > 1) {
#pragma unroll
            for (int q = 0; q < HPT; ++q) {
                const int h = min(t + q * nt, hcount - 1);
                int u;
                long long c;
                halo_slot(h, u, c);
                c = periodic ? wrap_fast(c, a.nx) : (c < 0 ? 0 : (c >= a.nx ? a.nx - 1 : c));
                long long r = rfirst + static_cast<long long>(rstep) * (s0 + u);
                if (periodic) r = wrap_fast(r, a.ny);
                hv[q] = to_acc<T>(in[r * a.ld + c]);
            }
        }
    };
    // Loads of any stage s0.
    auto load_stage = [&](int s0, A (&xin)[G][V], A (&hv)[HPT > 0 ? HPT : 1]) __attribute__((always_inline)) {
        if (clean_stage(s0)) {
            load_clean(s0, xin, hv);
            return;
        }
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const int s = s0 + u;
            long long r = rfirst + static_cast<long long>(rstep) * s;
            bool rv = s < niter;
            if (periodic) r = wrap_fast(r, a.ny);
            else rv = rv && r >= 0 && r < a.ny;
            if (rv) {
                const T *rowp = in + r * a.ld;
                if (full_vec) {
                    load_vec<T>(rowp + ib, xin[u]);
                } else {
#pragma unroll
                    for (int v = 0; v < V; ++v) xin[u][v] = load_elem<T>(rowp, ib + v, a.nx, periodic);
                }
            } else {
#pragma unroll
                for (int v = 0; v < V; ++v) xin[u][v] = A(0);
            }
        }
        if constexpr (NWX > 1) {
#pragma unroll
            for (int q = 0; q < HPT; ++q) {
                const int h = t + q * nt;
                A val = A(0);
                if (h < hcount) {
                    const int u = h / (2 * PAD);
                    const int hh = h - u * 2 * PAD;
                    const long long c = hh < PAD ? i0 - PAD + hh : i0 + W + (hh - PAD);
                    const int s = s0 + u;
                    long long r = rfirst + static_cast<long long>(rstep) * s;
                    bool rv = s < niter;
                    if (periodic) r = wrap_fast(r, a.ny);
                    else rv = rv && r >= 0 && r < a.ny;
                    if (rv) val = load_elem<T>(in + r * a.ld, c, a.nx, periodic);
                }
                hv[q] = val;
            }
        }
    };

    // acc[k] holds output row s - (NWY-1) + k; input row s meets it with
    // window row NWY-1-k.  After the row, acc[0] is complete: it is written
    // and the window shifts by one row.
    // clean: the output row exists and the whole strip is stored with vectors
    auto consume = [&](const A *x, int s, bool clean) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < NWY; ++k) {
#pragma unroll
            for (int p = 0; p < NWX; ++p) {
                const A wt = wv[(NWY - 1 - k) * NWX + p];
#pragma unroll
                for (int v = 0; v < V; ++v) acc[k][v] = fma(wt, x[v + p], acc[k][v]);
            }
        }
        const int jj = s - (NWY - 1);
        if (clean) {
            T *rowp = out + static_cast<long long>(up ? j0 + H - 1 - jj : j0 + jj) * a.ld;
            if (a.nt_store) store_vec_nt<T>(rowp + ib, acc[0]);
            else store_vec<T>(rowp + ib, acc[0]);
        } else if (jj >= 0 && jj < H) {
            const int j = up ? j0 + H - 1 - jj : j0 + jj;
            if (periodic || (j >= a.T && j <= a.ny - 1 - a.B)) {
                T *rowp = out + static_cast<long long>(j) * a.ld;
                if (store_vec_ok) {
                    if (a.nt_store) store_vec_nt<T>(rowp + ib, acc[0]);
                    else store_vec<T>(rowp + ib, acc[0]);
                } else {
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        const long long c = ib + v;
                        if constexpr (BY_INDEX) {
                            if (v >= v0 && v < v1) rowp[c] = from_acc<T>(acc[0][v]);
                        } else if (c >= lo && c < a.nx && (periodic || (c >= a.L && c <= a.nx - 1 - a.R))) {
                            rowp[c] = from_acc<T>(acc[0][v]);
                        }
                    }
                }
            }
        }
#pragma unroll
        for (int k = 0; k + 1 < NWY; ++k)
#pragma unroll
            for (int v = 0; v < V; ++v) acc[k][v] = acc[k + 1][v];
#pragma unroll
        for (int v = 0; v < V; ++v) acc[NWY - 1][v] = A(0);
    };

    // A stage is consumed "clean" when its G rows all produce output rows that
    // exist, the strip is stored with whole vectors, and the next stage's
    // loads are clean too: its loads and stores are then straight-line code
    // with fixed counts, so waiting for the next stage's loads never waits
    // for this stage's stores.
    const bool strip_store_clean =
        strip_clean && i0 == lo && (periodic || (i0 >= a.L && i0 + W - 1 <= static_cast<long long>(a.nx) - 1 - a.R));
    auto clean_iter = [&](int s0) __attribute__((always_inline)) {
        if (!strip_store_clean || s0 < NWY - 1 || s0 + G - NWY >= H || !clean_stage(s0 + G)) return false;
        if (periodic) return true;
        const int ja = up ? j0 + H - 1 - (s0 - (NWY - 1)) : j0 + (s0 - (NWY - 1));
        const int jb = up ? j0 + H - 1 - (s0 + G - NWY) : j0 + (s0 + G - NWY);
        return (ja < jb ? ja : jb) >= a.T && (ja > jb ? ja : jb) <= a.ny - 1 - a.B;
    };

    A cur[G][V], nxt[G][V];
    A hcur[HPT > 0 ? HPT : 1], hnxt[HPT > 0 ? HPT : 1];
    load_stage(0, cur, hcur);

    auto iteration = [&](int s0, bool clean) __attribute__((always_inline)) {
        // the point function is applied once per loaded element: Horner's
        // rule with the coefficient loop outside and the stage's elements
        // inside (the same operations, in the same order, per element)
        if (a.ncoe) {
            constexpr int HQ = NWX > 1 ? HPT : 0;
            A f[G][V], hf[HQ > 0 ? HQ : 1];
            const A top = coe[a.ncoe - 1];
#pragma unroll
            for (int u = 0; u < G; ++u)
#pragma unroll
                for (int v = 0; v < V; ++v) f[u][v] = top;
#pragma unroll
            for (int q = 0; q < HQ; ++q) hf[q] = top;
            for (int m = a.ncoe - 2; m >= 0; --m) {
                const A cm = coe[m];
#pragma unroll
                for (int u = 0; u < G; ++u)
#pragma unroll
                    for (int v = 0; v < V; ++v) f[u][v] = f[u][v] * cur[u][v] + cm;
#pragma unroll
                for (int q = 0; q < HQ; ++q) hf[q] = hf[q] * hcur[q] + cm;
            }
#pragma unroll
            for (int u = 0; u < G; ++u)
#pragma unroll
                for (int v = 0; v < V; ++v) cur[u][v] = f[u][v];
#pragma unroll
            for (int q = 0; q < HQ; ++q) hcur[q] = hf[q];
        }
        if constexpr (NWX > 1) {
            __syncthreads();   // the previous stage's LDS reads are done
#pragma unroll
            for (int u = 0; u < G; ++u) {
                A *dst = lds + u * rowlen + PAD + t * V;
#pragma unroll
                for (int v = 0; v < V; ++v) dst[v] = cur[u][v];
            }
            const bool cl = clean_stage(s0);
#pragma unroll
            for (int q = 0; q < HPT; ++q) {
                const int h = t + q * nt;
                if (h < hcount) {
                    const int u = h / (2 * PAD);
                    const int hh = h - u * 2 * PAD;
                    long long c;
                    int uu;
                    halo_slot(h, uu, c);
                    const bool zero = cl && !periodic && (c < 0 || c >= a.nx);
                    lds[u * rowlen + (hh < PAD ? hh : W + hh)] = zero ? A(0) : hcur[q];
                }
            }
        }
        // next stage's loads overlap this stage's arithmetic
        if (clean) load_clean(s0 + G, nxt, hnxt);
        else if (s0 + G < niter) load_stage(s0 + G, nxt, hnxt);
        if constexpr (NWX > 1) {
            __syncthreads();
            const int nu = clean ? G : min(G, niter - s0);
#pragma unroll 1
            for (int u = 0; u < nu; ++u) {
                A x[XW];
                const A *lp = lds + u * rowlen + PAD + t * V - a.L;
#pragma unroll
                for (int k = 0; k < XW; ++k) x[k] = lp[k];
                consume(x, s0 + u, clean);
            }
        } else {
#pragma unroll
            for (int u = 0; u < G; ++u)
                if (clean || s0 + u < niter) consume(cur[u], s0 + u, clean);
        }
#pragma unroll
        for (int u = 0; u < G; ++u)
#pragma unroll
            for (int v = 0; v < V; ++v) cur[u][v] = nxt[u][v];
#pragma unroll
        for (int q = 0; q < (HPT > 0 ? HPT : 1); ++q) hcur[q] = hnxt[q];
    };

    int s0 = 0;
    while (s0 < niter && !clean_iter(s0)) {
        iteration(s0, false);
        s0 += G;
    }
    while (s0 < niter && clean_iter(s0)) {
        iteration(s0, true);
        s0 += G;
    }
    while (s0 < niter) {
        iteration(s0, false);
        s0 += G;
    }
}

template <typename T, int NWX, int NWY>
hipError_t launch_one(const Stencil2DArgs &a, int threads, hipStream_t s) {
    using A = typename St<T>::acc;
    constexpr int V = St<T>::V;
    const size_t lds = NWX > 1
        ? static_cast<size_t>(stage_rows<NWY>()) * (2 * halo_pad<NWX, V>() + threads * V) * sizeof(A)
        : 0;
    const int grid = a.nstrips * a.nchunks;
    hipLaunchKernelGGL((stencil2d_kernel<T, NWX, NWY>), dim3(grid), dim3(threads), lds, s, a);
    return hipGetLastError();
}

template <typename T>
hipError_t dispatch(int nwx, int nwy, const Stencil2DArgs &a, int threads, hipStream_t s) {
#define MXS_CASE(X, Y) \
    if (nwx == X && nwy == Y) return launch_one<T, X, Y>(a, threads, s);
    MXS_CASE(1, 1) MXS_CASE(3, 1) MXS_CASE(5, 1) MXS_CASE(9, 1) MXS_CASE(17, 1)
    MXS_CASE(1, 3) MXS_CASE(1, 5) MXS_CASE(1, 9) MXS_CASE(1, 17)
    MXS_CASE(3, 3) MXS_CASE(3, 5) MXS_CASE(3, 9)
    MXS_CASE(5, 3) MXS_CASE(5, 5) MXS_CASE(5, 9)
    MXS_CASE(9, 3) MXS_CASE(9, 5) MXS_CASE(9, 9)
#undef MXS_CASE
    return hipErrorInvalidValue;
}

// Reads a buffer once (grid-stride, 16-byte loads) and writes nothing back
// unless its words XOR to a fixed value (then one word of the same buffer,
// which only serves this kernel): the loads replace the contents of the
// memory-side cache with clean lines.
__global__ void __launch_bounds__(256) cache_flush_kernel(void *buf, size_t n16) {
    const gptr<const v4u_t> p = as_global(static_cast<const v4u_t *>(buf));
    uint32_t x = 0;
    for (size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n16;
         i += static_cast<size_t>(gridDim.x) * blockDim.x) {
        const v4u_t v = p[i];
        x ^= v.x ^ v.y ^ v.z ^ v.w;
    }
    if (x == 0x9e3779b9u) as_global(reinterpret_cast<uint32_t *>(buf))[0] = x;
}

}  // namespace

hipError_t launch_cache_flush(void *buf, size_t bytes, hipStream_t s) {
    hipLaunchKernelGGL(cache_flush_kernel, dim3(2048), dim3(256), 0, s, buf, bytes / 16);
    return hipGetLastError();
}

int bucket_width(int taps) {
    if (taps <= 1) return 1;
    if (taps <= 3) return 3;
    if (taps <= 5) return 5;
    if (taps <= 9) return 9;
    if (taps <= 17) return 17;
    return 0;
}

bool stencil2d_block_ok(int dtype, int nwx, int nwy, int block_rows) {
    if (nwx == 1 && nwy == 9) return dtype != BF16 && block_rows == 16;
    return (nwx == 1 || nwx == 3 || nwx == 5) && (nwy == 3 || nwy == 5) &&
           (block_rows == 8 || block_rows == 12 || block_rows == 16);
}

bool stencil2d_xshuffle_ok(int dtype, int nwx, int nwy, int left, int right, int block_rows) {
    const int V = dtype == F64 ? St<double>::V : dtype == F32 ? St<float>::V : St<bf16>::V;
    if (nwx == 1 || nwx / 2 > V || left != nwx / 2 || right != nwx / 2) return false;
    if (nwy == 1) return nwx <= 9 && (block_rows == 4 || block_rows == 8);
    return stencil2d_block_ok(dtype, nwx, nwy, block_rows);
}

size_t stencil2d_lds_bytes(int dtype, int nwx, int nwy, int threads, int block_rows, int xshuffle) {
    if (nwx <= 1 || xshuffle) return 0;
    const int V = dtype == F64 ? St<double>::V : dtype == F32 ? St<float>::V : St<bf16>::V;
    const int acc = dtype == F64 ? 8 : 4;
    const int pad = ((nwx - 1 + V - 1) / V) * V;
    const int g = block_rows ? block_rows : 4;
    (void)nwy;
    return static_cast<size_t>(g) * (2 * pad + threads * V) * acc;
}

hipError_t launch_stencil2d(int dtype, int nwx, int nwy, const Stencil2DArgs &a, int threads,
                            hipStream_t s) {
    if (!stencil2d_fits_launch(a, threads)) return hipErrorInvalidConfiguration;
    switch (a.block_rows ? dtype : dtype + 3) {
    case F64: return launch_stencil2d_block_f64(nwx, nwy, a, threads, s);
    case F32: return launch_stencil2d_block_f32(nwx, nwy, a, threads, s);
    case BF16: return launch_stencil2d_block_bf16(nwx, nwy, a, threads, s);
    case F64 + 3: return dispatch<double>(nwx, nwy, a, threads, s);
    case F32 + 3: return dispatch<float>(nwx, nwy, a, threads, s);
    case BF16 + 3: return dispatch<bf16>(nwx, nwy, a, threads, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace mxs
