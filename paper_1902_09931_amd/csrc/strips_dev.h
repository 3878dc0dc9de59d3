// Device code of the column solves in one pass over memory: a workgroup
// holds a strip of CW columns, every row of it, in registers.
//
// Thread (c, s) of the workgroup holds L consecutive rows of column c,
// segment s: rows s L .. s L + L - 1.  Lane l of a wavefront is column l % CW
// of segment (64 / CW) w + l / CW, so a load instruction reads CW
// consecutive elements of 64 / CW rows.  Each direction of the cyclic
// recurrence (solve.h) takes two passes over the registers, as in the
// register line solver (wavelines.hip):
//   A. every thread runs the recurrence over its rows from a zero state; a
//      scan of the segments' end states within the wavefront (lane shuffles)
//      and a chain over the wavefronts' totals (LDS) give every segment the
//      zero-start state entering it and the state after the last row;
//   B. the cyclic closure gives the true state entering the column, and every
//      thread reruns its rows from its true incoming state.
// All powers of the companion matrix come from a table computed on the host.
#pragma once

#include "wave_dev.h"

namespace mxs {
namespace {

// Offsets, in matrices of 4 doubles, of the strip power table (SPW segments
// per wavefront, NW wavefronts): M^(k L) for k = 0 .. SPW; M^(w SPW L) for
// w < NW; the matrix that carries the closure state from the column's end to
// the segments of wavefront w, for w < NW; M^(rows of the last segment);
// M^(rows of the last wavefront that holds any); (I - M^ny)^{-1}.
template <int NT, int CW> struct StripTab {
    static constexpr int NW = NT / 64, SPW = 64 / CW;
    static constexpr int fw = SPW + 1, bwd = fw + NW, last = bwd + NW, tail = last + 1, cinv = tail + 1;
};

template <int BW> __device__ __forceinline__ S2 shfl_up_s(S2 v, int d) {
    return S2{__shfl_up(v.x, d, 64), BW == 2 ? __shfl_up(v.y, d, 64) : 0.0};
}
template <int BW> __device__ __forceinline__ S2 shfl_down_s(S2 v, int d) {
    return S2{__shfl_down(v.x, d, 64), BW == 2 ? __shfl_down(v.y, d, 64) : 0.0};
}

// xch: 2 NW CW pairs of doubles of LDS.
template <typename TR, typename TX, int BW, int EPI, int NT, int CW, int LMAX>
__device__ __forceinline__ void strip_block(const StripInst &I, const int strip, double2 *xch) {
    using Tab = StripTab<NT, CW>;
    constexpr int NW = NT / 64, SPW = 64 / CW;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int c = lane % CW, sl = lane / CW;
    const int L = I.L, ny = I.ny, nseg = I.nseg;
    const int seg = w * SPW + sl;
    const int wlast = (nseg - 1) / SPW;
    const int r0 = seg * L;
    const int cnt = min(max(ny - r0, 0), L);        // valid rows of the segment
    const bool whole = (w + 1) * SPW * L <= ny;     // every segment of the wavefront is full
    const int col = strip * CW + c;
    const bool valid = col < I.nx;
    const long long ld = I.ld;
    const double p1 = I.p1, p2 = I.p2;
    const cptr<double> tab = as_constant(I.tab);
    const long long base = valid ? col : I.nx - 1;

    // the segment's rows (rows past the end repeat the last one; their values are not used)
    TR raw[LMAX];
    {
        const gptr<const TR> rhs = as_global(static_cast<const TR *>(I.rhs)) + base;
        if (whole) {
            const gptr<const TR> p = rhs + r0 * ld;
#pragma unroll
            for (int j = 0; j < LMAX; ++j)
                if (j < L) raw[j] = gld<TR>(p, j * ld);
        } else {
#pragma unroll
            for (int j = 0; j < LMAX; ++j)
                if (j < L) raw[j] = gld<TR>(rhs, min(r0 + j, ny - 1) * ld);
        }
    }

    // ---- forward, pass A
    S2 e{0.0, 0.0};
    if (whole) {
#pragma unroll
        for (int j = 0; j < LMAX; ++j)
            if (j < L) e = rec<BW>(e, to_f64<TR>(raw[j]), p1, p2);
    } else {
#pragma unroll
        for (int j = 0; j < LMAX; ++j)
            if (j < L) e = keep_if<BW>(j < cnt, rec<BW>(e, to_f64<TR>(raw[j]), p1, p2), e);
    }
    S2 in;   // zero-start state entering the segment, from the wavefront's first segment
    {
        S2 s = e;
#pragma unroll
        for (int d = 1; d < SPW; d *= 2) {
            const S2 t = shfl_up_s<BW>(s, d * CW);
            const S2 u = mv_add<BW>(load_mat(tab + 4 * d), t, s);
            s = keep_if<BW>(sl >= d, u, s);
        }
        in = keep_if<BW>(sl > 0, shfl_up_s<BW>(s, CW), S2{0.0, 0.0});
        // the wavefront's total: the state after its last segment
        if (seg == min((w + 1) * SPW, nseg) - 1) {
            const S2 t = mv_add<BW>(load_mat(tab + 4 * (seg == nseg - 1 ? Tab::last : 1)), in, e);
            xch[w * CW + c] = make_double2(t.x, t.y);
        }
    }
    __syncthreads();
    {
        const Mat Mw = load_mat(tab + 4 * SPW);
        S2 f{0.0, 0.0}, mine{0.0, 0.0};
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            if (k <= wlast) {
                mine = keep_if<BW>(k == w, f, mine);
                const double2 t = xch[k * CW + c];
                f = mv_add<BW>(k == wlast ? load_mat(tab + 4 * Tab::tail) : Mw, f, S2{t.x, t.y});
            }
        }
        const S2 x0 = mv<BW>(load_mat(tab + 4 * Tab::cinv), f);
        // true state entering the wavefront, then the segment
        mine = mv_add<BW>(load_mat(tab + 4 * (Tab::fw + w)), x0, mine);
        in = mv_add<BW>(load_mat(tab + 4 * sl), mine, in);
    }

    // ---- forward, pass B
    double v[LMAX];
    {
        S2 s = in;
        if (whole) {
#pragma unroll
            for (int j = 0; j < LMAX; ++j)
                if (j < L) {
                    s = rec<BW>(s, to_f64<TR>(raw[j]), p1, p2);
                    v[j] = s.x;
                }
        } else {
#pragma unroll
            for (int j = 0; j < LMAX; ++j)
                if (j < L) {
                    s = rec<BW>(s, to_f64<TR>(raw[j]), p1, p2);
                    v[j] = j < cnt ? s.x : 0.0;
                }
        }
    }

    // ---- backward, pass A (rows past the end are zero and keep the zero state)
    e = S2{0.0, 0.0};
#pragma unroll
    for (int j = LMAX - 1; j >= 0; --j)
        if (j < L) e = rec<BW>(e, v[j], p1, p2);
    double2 *xb = xch + NW * CW;
    {
        S2 s = e;
#pragma unroll
        for (int d = 1; d < SPW; d *= 2) {
            const S2 t = shfl_down_s<BW>(s, d * CW);
            const S2 u = mv_add<BW>(load_mat(tab + 4 * d), t, s);
            s = keep_if<BW>(sl + d < SPW, u, s);
        }
        in = keep_if<BW>(sl < SPW - 1, shfl_down_s<BW>(s, CW), S2{0.0, 0.0});
        if (sl == 0) xb[w * CW + c] = make_double2(s.x, s.y);
    }
    __syncthreads();
    {
        const Mat Mw = load_mat(tab + 4 * SPW);
        S2 g{0.0, 0.0}, mine{0.0, 0.0};
#pragma unroll
        for (int k = NW - 1; k >= 0; --k) {
            if (k <= wlast) {
                mine = keep_if<BW>(k == w, g, mine);
                const double2 t = xb[k * CW + c];
                g = mv_add<BW>(Mw, g, S2{t.x, t.y});
            }
        }
        const S2 z0 = mv<BW>(load_mat(tab + 4 * Tab::cinv), g);
        mine = mv_add<BW>(load_mat(tab + 4 * (Tab::bwd + w)), z0, mine);
        // segments between this one and the state just formed
        const int up = min((w + 1) * SPW, nseg - 1) - 1 - seg;
        const S2 t = mv_add<BW>(load_mat(tab + 4 * max(up, 0)), mine, in);
        in = keep_if<BW>(seg == nseg - 1, z0, t);
    }

    // ---- backward, pass B, and the output (EPI 1: x = 2 cur - prev + v / K),
    // G rows at a time: their cur and prev values are requested together
    constexpr int G = LMAX < 8 ? LMAX : 8;
    const gptr<TX> x = as_global(static_cast<TX *>(I.x)) + base + r0 * ld;
    const gptr<const TX> cur = as_global(static_cast<const TX *>(I.cur)) + base;
    const gptr<const TX> prev = as_global(static_cast<const TX *>(I.prev)) + base;
    const double invK = I.invK;
    S2 s = in;
#pragma unroll
    for (int jg = LMAX - G; jg >= 0; jg -= G) {
        if (jg >= L) continue;
        double cb[G];
        if constexpr (EPI == 1) {
#pragma unroll
            for (int q = 0; q < G; ++q) {
                const long long o = min(r0 + min(jg + q, L - 1), ny - 1) * ld;
                cb[q] = 2.0 * to_f64<TX>(gld<TX>(cur, o)) - to_f64<TX>(gld<TX>(prev, o));
            }
        }
#pragma unroll
        for (int q = G - 1; q >= 0; --q) {
            const int j = jg + q;
            if (j < L) {
                if (whole) {
                    s = rec<BW>(s, v[j], p1, p2);
                } else {
                    s = keep_if<BW>(j < cnt, rec<BW>(s, v[j], p1, p2), s);
                }
                if (valid && j < cnt) gst<TX>(x, j * ld, from_f64<TX>(EPI == 1 ? cb[q] + s.x * invK : s.x * invK));
            }
        }
    }
}

}  // namespace
}  // namespace mxs
