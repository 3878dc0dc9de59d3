// Device code of the pentadiagonal line solver that spreads one line over LPR lanes, 16
// consecutive elements per lane: LPR = 16 or 32 lanes (2 or 4 lines share a
// wavefront), 64 (a wavefront) or 128 / 256 (2 or 4 wavefronts).  The method
// is the one of the register line solver (wavelines.hip): per direction a
// zero-start pass, a scan of the lane states, the cyclic closure and a rerun
// from the true states.  A lane holds 16 elements whatever the line's length,
// so that a long line takes more wavefronts instead of more registers.
#pragma once

#include "wave_dev.h"

namespace mxs {
namespace {

constexpr int kGroupE = 16;            // elements per lane
constexpr int kGroupLanes = 16;        // lanes of one scan group (a DPP row)
static_assert(kGroupE * kGroupLanes == kWaveBlock, "a scan group spans one table block");

struct LineCoef {
    double p1, p2;
    const double *pow;   // power table (solve.h)
};

// (I - m)^{-1}, m a power of the companion matrix
__device__ __forceinline__ Mat closure_mat(const Mat &m) {
    const double a = 1.0 - m.a, b = -m.b, c = -m.c, d = 1.0 - m.d;
    const double r = 1.0 / (a * d - b * c);
    return Mat{d * r, -b * r, -c * r, a * r};
}

// Orders LDS accesses between the lanes of a line.
template <int LPR> __device__ __forceinline__ void line_sync() {
    if constexpr (LPR <= 64) wave_sync();
    else __syncthreads();
}

// Solve the pentadiagonal line of n elements whose elements 16 li .. 16 li + 15 are in v
// (li = 0 .. LPR - 1 the lane's index in its line; elements past n are zero),
// leaving u / K times K in v, i.e. the solution before the scaling by 1/K.
// xch: the line's exchange space of 2 * max(1, LPR / 64) pairs of doubles (4
// pairs where LPR < 64).  Every lane of the wavefront is active; with LPR >
// 64 every thread of the workgroup calls this together.
template <int LPR>
__device__ __forceinline__ void group_solve(double (&v)[kGroupE], const int n, const int li, const LineCoef &co,
                                            double2 *xch) {
    constexpr int E = kGroupE, BW = 2;
    const int lane = threadIdx.x & 63;
    const int row = lane >> 4, p = lane & 15;
    const cptr<double> pw = as_constant(co.pow);
    const cptr<double> pb = pw + 4 * (kWaveBlock + 1);
    const double p1 = co.p1, p2 = co.p2;
    const int ll = (n - 1) / E;                         // lane of the last element
    const int cnt = min(max(n - E * li, 0), E);         // valid elements of the lane
    const int cl = n - E * ll;                          // valid elements of lane ll
    // the lanes of a wavefront that holds no partial lane need no selects
    const bool masked = cl < E && (LPR <= 64 || (li >> 6) == (ll >> 6));

    Mat K[4];   // M^E, M^2E, M^4E, M^8E: the row scan steps
#pragma unroll
    for (int i = 0; i < 4; ++i) K[i] = load_mat(pw + 4 * (E << i));
    const Mat Mrow = load_mat(pw + 4 * kWaveBlock);     // one row of 16 lanes
    const Mat Cn = closure_mat(pow_mat(pw, pb, n));

    // ---- forward, pass A
    S2 e{0.0, 0.0};
    if (!masked) {
#pragma unroll
        for (int j = 0; j < E; ++j) e = rec<BW>(e, v[j], p1, p2);
    } else {
#pragma unroll
        for (int j = 0; j < E; ++j) e = keep_if<BW>(j < cnt, rec<BW>(e, v[j], p1, p2), e);
    }
    S2 in;
    {
        S2 s = e;
        s = mv_add<BW>(K[0], dpp_s<0x111, BW>(s), s);
        s = mv_add<BW>(K[1], dpp_s<0x112, BW>(s), s);
        s = mv_add<BW>(K[2], dpp_s<0x114, BW>(s), s);
        s = mv_add<BW>(K[3], dpp_s<0x118, BW>(s), s);
        const S2 ex = dpp_s<0x111, BW>(s);              // zero-start state entering the lane, from its row
        const Mat Mp = load_mat(pw + 4 * (E * p));      // M^(E p)
        if constexpr (LPR >= 64) {
            constexpr int NW = LPR / 64;
            const int w = __builtin_amdgcn_readfirstlane(li >> 6);
            const int wl = ll >> 6;
            const S2 c1 = readlane_s<BW>(s, 15);
            const S2 c2 = mv_add<BW>(Mrow, c1, readlane_s<BW>(s, 31));
            const S2 c3 = mv_add<BW>(Mrow, c2, readlane_s<BW>(s, 47));
            in = mv_add<BW>(Mp, pick_row<BW>(row, S2{0.0, 0.0}, c1, c2, c3), ex);
            // the state after the wavefront's last element of the line
            S2 tot;
            if (w == wl) tot = mv_add<BW>(load_mat(pw + 4 * cl), readlane_s<BW>(in, ll & 63), readlane_s<BW>(e, ll & 63));
            else tot = mv_add<BW>(Mrow, c3, readlane_s<BW>(s, 63));
            S2 f = tot, pre{0.0, 0.0};
            if constexpr (NW > 1) {
                if (lane == 0) xch[w] = make_double2(tot.x, tot.y);
                __syncthreads();
                f = S2{0.0, 0.0};
#pragma unroll
                for (int k = 0; k < NW; ++k) {
                    if (k <= wl) {
                        if (k == w) pre = f;
                        const double2 t = xch[k];
                        f = mv_add<BW>(pow_mat(pw, pb, k == wl ? n - 64 * E * k : 64 * E), f, S2{t.x, t.y});
                    }
                }
            }
            const S2 x0 = mv<BW>(Cn, f);
            S2 c = x0;   // true state entering the wavefront
            if constexpr (NW > 1) c = mv_add<BW>(load_mat(pb + 4 * (64 * E / kWaveBlock * w)), x0, pre);
            in = mv_add<BW>(pow_mat(pw, pb, E * lane), c, in);
        } else {
            constexpr int G = LPR / 16;
            const int g = li >> 4, gl = ll >> 4;
            if (li == ll) {
                const S2 t = mv_add<BW>(load_mat(pw + 4 * cl), ex, e);
                xch[g] = make_double2(t.x, t.y);
            } else if (p == 15 && g < gl) {
                xch[g] = make_double2(s.x, s.y);
            }
            wave_sync();
            S2 f{0.0, 0.0}, pre{0.0, 0.0};
#pragma unroll
            for (int k = 0; k < G; ++k) {
                if (k <= gl) {
                    pre = keep_if<BW>(k == g, f, pre);
                    const double2 t = xch[k];
                    f = mv_add<BW>(load_mat(pw + 4 * (k == gl ? n - 16 * E * k : 16 * E)), f, S2{t.x, t.y});
                }
            }
            const S2 x0 = mv<BW>(Cn, f);
            const S2 c = G > 1 ? mv_add<BW>(load_mat(pb + 4 * g), x0, pre) : x0;
            in = mv_add<BW>(Mp, c, ex);
        }
    }

    // ---- forward, pass B (a lane past the end keeps the zero state and zero values)
    in = keep_if<BW>(cnt > 0, in, S2{0.0, 0.0});
    if (!masked) {
#pragma unroll
        for (int j = 0; j < E; ++j) {
            in = rec<BW>(in, v[j], p1, p2);
            v[j] = in.x;
        }
    } else {
#pragma unroll
        for (int j = 0; j < E; ++j) {
            in = rec<BW>(in, v[j], p1, p2);
            v[j] = j < cnt ? in.x : 0.0;
        }
    }

    // ---- backward, pass A (zero values above the line's end keep the zero state)
    e = S2{0.0, 0.0};
#pragma unroll
    for (int j = E - 1; j >= 0; --j) e = rec<BW>(e, v[j], p1, p2);
    {
        S2 s = e;
        s = mv_add<BW>(K[0], dpp_s<0x101, BW>(s), s);
        s = mv_add<BW>(K[1], dpp_s<0x102, BW>(s), s);
        s = mv_add<BW>(K[2], dpp_s<0x104, BW>(s), s);
        s = mv_add<BW>(K[3], dpp_s<0x108, BW>(s), s);
        const S2 ex = dpp_s<0x101, BW>(s);
        const Mat Mq = load_mat(pw + 4 * (E * (15 - p)));   // M^(E (15 - p))
        S2 g, above{0.0, 0.0};   // zero-start state after element 0; entering the lane's row or wavefront
        if constexpr (LPR >= 64) {
            constexpr int NW = LPR / 64;
            const int w = __builtin_amdgcn_readfirstlane(li >> 6);
            const int wl = ll >> 6;
            const S2 c2 = readlane_s<BW>(s, 48);
            const S2 c1 = mv_add<BW>(Mrow, c2, readlane_s<BW>(s, 32));
            const S2 c0 = mv_add<BW>(Mrow, c1, readlane_s<BW>(s, 16));
            const S2 tot = mv_add<BW>(Mrow, c0, readlane_s<BW>(s, 0));
            in = mv_add<BW>(Mq, pick_row<BW>(row, c0, c1, c2, S2{0.0, 0.0}), ex);
            g = tot;
            if constexpr (NW > 1) {
                double2 *xb = xch + NW;
                if (lane == 0) xb[w] = make_double2(tot.x, tot.y);
                __syncthreads();
                g = S2{0.0, 0.0};
                const Mat Mw = load_mat(pb + 4 * (64 * E / kWaveBlock));
#pragma unroll
                for (int k = NW - 1; k >= 0; --k) {
                    if (k <= wl) {
                        if (k == w) above = g;
                        const double2 t = xb[k];
                        g = mv_add<BW>(Mw, g, S2{t.x, t.y});
                    }
                }
                in = mv_add<BW>(pow_mat(pw, pb, E * (63 - lane)), above, in);
            }
        } else {
            constexpr int G = LPR / 16;
            double2 *xb = xch + G;
            const int gi = li >> 4, gl = ll >> 4;
            if (p == 0) xb[gi] = make_double2(s.x, s.y);
            wave_sync();
            g = S2{0.0, 0.0};
#pragma unroll
            for (int k = G - 1; k >= 0; --k) {
                if (k <= gl) {
                    above = keep_if<BW>(k == gi, g, above);
                    const double2 t = xb[k];
                    g = mv_add<BW>(Mrow, g, S2{t.x, t.y});
                }
            }
            in = G > 1 ? mv_add<BW>(Mq, above, ex) : ex;
        }
        // the closure state carried from the line's end over the elements above the lane
        const S2 z0 = mv<BW>(Cn, g);
        const int d = max(n - E * (li + 1), 0);
        in = mv_add<BW>(load_mat(pw + 4 * (d & (kWaveBlock - 1))), mv<BW>(load_mat(pb + 4 * (d / kWaveBlock)), z0), in);
    }

    // ---- backward, pass B
    if (!masked) {
#pragma unroll
        for (int j = E - 1; j >= 0; --j) {
            in = rec<BW>(in, v[j], p1, p2);
            v[j] = in.x;
        }
    } else {
#pragma unroll
        for (int j = E - 1; j >= 0; --j) {
            in = keep_if<BW>(j < cnt, rec<BW>(in, v[j], p1, p2), in);
            v[j] = in.x;
        }
    }
}

// Pairs of doubles of exchange space of one line.
template <int LPR> constexpr int kGroupXch = LPR < 64 ? 4 : 2 * (LPR / 64);

}  // namespace
}  // namespace mxs
