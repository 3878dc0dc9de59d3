// Coarsening diagnostics of a Cahn-Hilliard state (Sec. 5.3):
//
//   s(t)  = 1 / (1 - <C^2>), <.> the spatial average by Simpson's rule;
//   k1(t) = sum_k |C^(k)|^2 / sum_k |k|^-1 |C^(k)|^2, over the nonzero
//           wavevectors of the grid's discrete Fourier transform.
//
// Simpson's rule on a periodic grid of N (even) nodes x_i = i h: the
// composite rule over [0, N h] with the end node identified with node 0
// gives node i the weight (2 h / 3) for even i and (4 h / 3) for odd i, so
// the average is (1 / (nx ny)) sum_ij a_i a_j C_ij^2 with a = 2/3, 4/3.
// Both sums are accumulated in double by fixed-order two-level reductions
// (deterministic).
//
// The transform: two real rows are transformed as one complex line and
// separated by symmetry, and only the columns 0 .. nx / 2 are kept and
// transformed (the spectrum of a real grid is Hermitian: the columns between
// count twice).  Lines are transformed in LDS by a self-sorting radix-4
// algorithm (Stockham; one radix-2 stage where log2 n is odd) with the
// roots of unity in an LDS table, computed once per workgroup.  A row
// workgroup also forms its rows' share of the Simpson sum; a column workgroup
// weights |C^|^2 by 1 and by 1/|k| and reduces both sums.  Grid sides must be
// powers of two, at most kDiagMaxSide.  At 512^2 FP64 the three kernels take
// 26 us where one line per workgroup with a sine and cosine per butterfly,
// full complex rows and separate Simpson kernels took 33 us; the serial chain
// of stages bounds them.
#include "diag.h"

#include <mutex>

namespace mxs {

// Scratch of the allocation-free diagnostics entry point: the transform grid
// (kNoAllocDiagPoints complex values), then the partial sums (ny + 2 nx
// doubles).  Every GPU the library runs on holds its own
// copy for the life of the process.  Host code never passes this name to a
// kernel: its device address comes from hipGetSymbolAddress, per device.
static __device__ __align__(256) double scratch[2 * kNoAllocDiagPoints + 3 * kDiagMaxSide + 8];

namespace {

template <typename T> __device__ __forceinline__ double load_f64(gptr<const T> p, long long i);
template <> __device__ __forceinline__ double load_f64<double>(gptr<const double> p, long long i) { return p[i]; }
template <> __device__ __forceinline__ double load_f64<float>(gptr<const float> p, long long i) { return p[i]; }
template <> __device__ __forceinline__ double load_f64<bf16>(gptr<const bf16> p, long long i) {
    return bf16_to_float(reinterpret_cast<gptr<const uint16_t>>(p)[i]);
}

// Sum of v over the workgroup, in a fixed order (tree over kDiagThreads).
__device__ double wg_sum(double v, double *red) {
    const int t = threadIdx.x;
    red[t] = v;
    __syncthreads();
    for (int h = kDiagThreads / 2; h > 0; h >>= 1) {
        if (t < h) red[t] += red[t + h];
        __syncthreads();
    }
    const double r = red[0];
    __syncthreads();
    return r;
}

// tw[m] = exp(-2 pi i m / n), m < n.
__device__ __forceinline__ void fill_roots(double2 *tw, int n) {
    for (int m = threadIdx.x; m < n; m += kDiagThreads) {
        double sn, cs;
        sincospi(-2.0 * m / n, &sn, &cs);
        tw[m] = make_double2(cs, sn);
    }
}

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// Transform `lines` lines of n = 2^logn >= 8 complex values in LDS, back to
// back in a, in natural order before and after: X_k = sum_m x_m exp(-2 pi i
// k m / n).  lines * n <= kDiagValues.  Every stage reads its inputs into
// registers before it writes its outputs over them.
__device__ __forceinline__ void fft_lines(double2 *a, const double2 *tw, int n, int logn, int lines) {
    constexpr int B4 = kDiagValues / 4 / kDiagThreads, B2 = 2 * B4;
    const int t = threadIdx.x;
    int ns = 1, lns = 0;   // transform length so far and its logarithm
    __syncthreads();
    for (; lns + 2 <= logn; ns *= 4, lns += 2) {
        const int q = n >> 2, lq = logn - 2, total = lines << lq;
        double2 v[B4][4];
#pragma unroll
        for (int b = 0; b < B4; ++b) {
            const int j = t + b * kDiagThreads;
            if (j < total) {
                const double2 *p = a + ((j >> lq) << logn);
                const int i = j & (q - 1), k = i & (ns - 1), step = k << (lq - lns);
                v[b][0] = p[i];
                v[b][1] = cmul(p[i + q], tw[step]);
                v[b][2] = cmul(p[i + 2 * q], tw[2 * step]);
                v[b][3] = cmul(p[i + 3 * q], tw[3 * step]);
            }
        }
        __syncthreads();
#pragma unroll
        for (int b = 0; b < B4; ++b) {
            const int j = t + b * kDiagThreads;
            if (j < total) {
                const int i = j & (q - 1), k = i & (ns - 1);
                double2 *o = a + ((j >> lq) << logn) + ((i - k) << 2) + k;
                const double2 x = v[b][0], y = v[b][1], z = v[b][2], w = v[b][3];
                const double2 s0 = make_double2(x.x + z.x, x.y + z.y), s1 = make_double2(x.x - z.x, x.y - z.y);
                const double2 s2 = make_double2(y.x + w.x, y.y + w.y), s3 = make_double2(y.x - w.x, y.y - w.y);
                o[0] = make_double2(s0.x + s2.x, s0.y + s2.y);
                o[ns] = make_double2(s1.x + s3.y, s1.y - s3.x);
                o[2 * ns] = make_double2(s0.x - s2.x, s0.y - s2.y);
                o[3 * ns] = make_double2(s1.x - s3.y, s1.y + s3.x);
            }
        }
        __syncthreads();
    }
    if (lns < logn) {
        const int h = n >> 1, lh = logn - 1, total = lines << lh;
        double2 v[B2][2];
#pragma unroll
        for (int b = 0; b < B2; ++b) {
            const int j = t + b * kDiagThreads;
            if (j < total) {
                const double2 *p = a + ((j >> lh) << logn);
                const int i = j & (h - 1);   // ns = h: output i of both halves
                v[b][0] = p[i];
                v[b][1] = cmul(p[i + h], tw[i]);
            }
        }
        __syncthreads();
#pragma unroll
        for (int b = 0; b < B2; ++b) {
            const int j = t + b * kDiagThreads;
            if (j < total) {
                const int i = j & (h - 1);
                double2 *o = a + ((j >> lh) << logn) + i;
                o[0] = make_double2(v[b][0].x + v[b][1].x, v[b][0].y + v[b][1].y);
                o[h] = make_double2(v[b][0].x - v[b][1].x, v[b][0].y - v[b][1].y);
            }
        }
        __syncthreads();
    }
}

// `lines` row pairs from pair lines * block on: the pairs' Simpson sums, and
// columns 0 .. nx / 2 of the transforms of both rows of every pair.
template <typename T>
__global__ void __launch_bounds__(kDiagThreads) fft_rows_kernel(const T *c, int nx, int lognx, int lines,
                                                                double2 *spec, int pitch, double *partial) {
    extern __shared__ double2 lds[];
    __shared__ double red[kDiagThreads];
    double2 *tw = lds + lines * nx;
    const int t = threadIdx.x;
    const long long row0 = 2LL * lines * blockIdx.x;
    const gptr<const T> src = as_global(c) + row0 * nx;
    fill_roots(tw, nx);
    double s = 0.0;
    for (int e = t; e < lines * nx; e += kDiagThreads) {
        const int pair = e >> lognx, i = e & (nx - 1);
        const long long o = (static_cast<long long>(pair) << (lognx + 1)) + i;
        const double u = load_f64<T>(src, o), v = load_f64<T>(src, o + nx);
        lds[e] = make_double2(u, v);
        s += ((i & 1) ? 4.0 / 3.0 : 2.0 / 3.0) * (2.0 / 3.0 * (u * u) + 4.0 / 3.0 * (v * v));
    }
    fft_lines(lds, tw, nx, lognx, lines);
    const gptr<double> o = as_global(reinterpret_cast<double *>(spec)) + 2 * row0 * pitch;
    const int nc = nx / 2 + 1;
    for (int pair = 0; pair < lines; ++pair) {
        const double2 *z = lds + (pair << lognx);
        const gptr<double> r = o + 4LL * pair * pitch;
        for (int k = t; k < nc; k += kDiagThreads) {
            const double2 x = z[k], y = z[(nx - k) & (nx - 1)];
            r[2 * k] = 0.5 * (x.x + y.x);                  // even row: (Z_k + conj Z_{n-k}) / 2
            r[2 * k + 1] = 0.5 * (x.y - y.y);
            r[2 * (pitch + k)] = 0.5 * (x.y + y.y);        // odd row: (Z_k - conj Z_{n-k}) / 2i
            r[2 * (pitch + k) + 1] = 0.5 * (y.x - x.x);
        }
    }
    const double tot = wg_sum(s, red);
    if (t == 0) partial[blockIdx.x] = tot;
}

// `lines` columns of the transformed rows from column lines * block on:
// transform, then their share of sum |X|^2 and sum |X|^2 / |k| (k = 0 left
// out), a column 0 < i < nx / 2 standing for column nx - i too.
__global__ void __launch_bounds__(kDiagThreads) fft_cols_kernel(const double2 *spec, int pitch, int nx, int ny,
                                                                int logny, int lines, double kx0, double ky0,
                                                                double *partial) {
    extern __shared__ double2 lds[];
    __shared__ double red[kDiagThreads];
    double2 *tw = lds + lines * ny;
    const int t = threadIdx.x;
    const int i0 = lines * blockIdx.x, nc = nx / 2 + 1;
    const gptr<const double> src = as_global(reinterpret_cast<const double *>(spec));
    fill_roots(tw, ny);
    for (int e = t; e < lines * ny; e += kDiagThreads) {
        const int j = e / lines, l = e - j * lines;        // columns fastest: neighbouring threads read one row
        const long long o = 2 * (static_cast<long long>(j) * pitch + min(i0 + l, nc - 1));
        lds[(l << logny) + j] = make_double2(src[o], src[o + 1]);
    }
    fft_lines(lds, tw, ny, logny, lines);
    double p = 0.0, q = 0.0;
    for (int e = t; e < lines * ny; e += kDiagThreads) {
        const int l = e >> logny, j = e & (ny - 1);
        const int mx = i0 + l, my = j <= ny / 2 ? j : j - ny;
        if (mx >= nc || (mx == 0 && my == 0)) continue;
        const double kx = kx0 * mx, ky = ky0 * my;
        const double2 x = lds[e];
        const double w = (mx == 0 || mx == nx / 2 ? 1.0 : 2.0) * (x.x * x.x + x.y * x.y);
        p += w;
        q += w / sqrt(kx * kx + ky * ky);
    }
    const double ps = wg_sum(p, red);
    const double qs = wg_sum(q, red);
    if (t == 0) {
        partial[2 * blockIdx.x] = ps;
        partial[2 * blockIdx.x + 1] = qs;
    }
}

// out[0] = the sum of the nr row partials, out[1] and out[2] = the sums of
// the nc pairs of column partials, each in a fixed order.
__global__ void __launch_bounds__(kDiagThreads) diag_final_kernel(const double *partial, int nr, int nc, double *out) {
    __shared__ double red[kDiagThreads];
    const int k = blockIdx.x;
    const int n = k == 0 ? nr : nc, stride = k == 0 ? 1 : 2;
    const double *p = k == 0 ? partial : partial + nr + (k - 1);
    double s = 0.0;
    for (int m = threadIdx.x; m < n; m += kDiagThreads) s += p[m * stride];
    const double tot = wg_sum(s, red);
    if (threadIdx.x == 0) out[k] = tot;
}

int log2_exact(int n) {
    int l = 0;
    while ((1 << l) < n) ++l;
    return (1 << l) == n ? l : -1;
}

template <typename T>
hipError_t diag_one(const DiagArgs &d, hipStream_t s) {
    const int lx = log2_exact(d.nx), ly = log2_exact(d.ny);
    // Row pairs per workgroup: 1024 values, one butterfly per thread and
    // stage.  Columns per workgroup: 2048 values, at most 4 columns (64-byte
    // pieces of a row; more columns would leave most CUs without a workgroup).
    const int pitch = (d.nx / 2 + 2) & ~1, ncols = d.nx / 2 + 1;
    int rl = 1, cl = 1;
    while (rl * 2 * d.nx <= 1024 && rl * 2 <= d.ny / 2) rl *= 2;
    while (cl < 4 && cl * 2 * d.ny <= 2048) cl *= 2;
    const int rblocks = d.ny / 2 / rl, cblocks = (ncols + cl - 1) / cl;
    hipLaunchKernelGGL((fft_rows_kernel<T>), dim3(rblocks), dim3(kDiagThreads), sizeof(double2) * d.nx * (rl + 1), s,
                       static_cast<const T *>(d.c), d.nx, lx, rl, d.spec, pitch, d.partial);
    hipLaunchKernelGGL(fft_cols_kernel, dim3(cblocks), dim3(kDiagThreads), sizeof(double2) * d.ny * (cl + 1), s, d.spec,
                       pitch, d.nx, d.ny, ly, cl, d.kx0, d.ky0, d.partial + rblocks);
    hipLaunchKernelGGL(diag_final_kernel, dim3(3), dim3(kDiagThreads), 0, s, d.partial, rblocks, cblocks, d.out);
    return hipGetLastError();
}

}  // namespace

bool diag_shape_ok(int nx, int ny) {
    return nx >= 8 && ny >= 8 && nx <= kDiagMaxSide && ny <= kDiagMaxSide && log2_exact(nx) >= 0 &&
           log2_exact(ny) >= 0;
}

hipError_t noalloc_diag_scratch(int nx, int ny, DiagArgs *d) {
    static std::mutex mu;
    static double *addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    double *base;
    {
        std::lock_guard<std::mutex> lock(mu);
        if (!addr[dev]) {
            void *p = nullptr;
            e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (e != hipSuccess) return e;
            addr[dev] = static_cast<double *>(p);
        }
        base = addr[dev];
    }
    d->spec = reinterpret_cast<double2 *>(base);
    d->partial = base + 2 * static_cast<size_t>(nx) * ny;
    return hipSuccess;
}

hipError_t launch_coarsening(int dtype, const DiagArgs &d, hipStream_t s) {
    if (!diag_shape_ok(d.nx, d.ny)) return hipErrorInvalidValue;
    switch (dtype) {
    case F64: return diag_one<double>(d, s);
    case F32: return diag_one<float>(d, s);
    case BF16: return diag_one<bf16>(d, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace mxs
