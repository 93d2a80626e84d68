// 2D levels of the scalar kinds: one wavefront per tile of 62 node columns and
// R node rows, no LDS and no barrier.
//
// Lane l owns node column xs + l - 1 (xs a multiple of 62) and evaluates the
// element column to its right; the corner values and the contributions of the
// neighbouring column cross by wavefront shifts (DPP), the row above's by a
// register carry.  Every element of the tile is evaluated once, against four
// times in the node-centric kernel, which was bound by that arithmetic (two
// square roots and two quotients per p = 1 element, eight exponentials per
// Bratu element); the halo costs (R + 1)/R in y and 64/62 in x.  All rows of
// the tile are loaded before the first element.  One FP64 Chebyshev step at
// 800^2: Bratu 37.2 -> 19.1 us (14.3 since its expm1 is a series), minimal
// surface 31.8 -> 12.3 us; at 1600^2 125 -> 53 (40) and 88 -> 36 us.
#pragma once
#include "stencil.hpp"

namespace jfnk {

constexpr int ROW2_COLS = 62;

template <int KIND, int MODE, typename T, typename TV, class Epi, int PF, int R>
__global__ __launch_bounds__(BLOCK) void k_row2(Grid g, Phys ph, const T *kap, const T *x, const TV *v, const T *Ax,
                                                FdStep fd, Epi epi, Red red, int strips, int tiles) {
    constexpr bool FD = MODE == M_FD_PLAIN || MODE == M_FD_DIFF;
    constexpr bool DIR = MODE != M_RESID;
    constexpr bool INV = KIND == JFNK_INVCOEF;
    constexpr bool PLAIN = MODE == M_FD_PLAIN;
    constexpr int NIN = Epi::NIN > 0 ? Epi::NIN : 1;
    constexpr bool VREG = DIR && Epi::VIN >= 0;
    const double eps = fd_eps_prepare(fd, epi);
    const bool zero_fd = FD && eps == 0.0;
    const T e = (T)eps, ie = PLAIN && eps > 0.0 ? (T)(1.0 / eps) : T(0), h = (T)g.h;
    double sums[Epi::NS > 0 ? Epi::NS : 1];
#pragma unroll
    for (int k = 0; k < (Epi::NS > 0 ? Epi::NS : 1); ++k) sums[k] = 0.0;
    const int lane = threadIdx.x & 63;
    const int nwaves = gridDim.x * (BLOCK / 64);
    for (int tile = blockIdx.x * (BLOCK / 64) + (threadIdx.x >> 6); tile < tiles; tile += nwaves) {
        const int X = (tile % strips) * ROW2_COLS - 1 + lane, y0 = (tile / strips) * R;
        const int Xc = min(max(X, 0), g.nx);
        const bool xdir = ((g.dir & JFNK_FACE_XLO) && X == 0) || ((g.dir & JFNK_FACE_XHI) && X == g.nx);
        const bool xfree = X == Xc && !xdir;
        auto ydir = [&](int Y) { return ((g.dir & JFNK_FACE_YLO) && Y == 0) || ((g.dir & JFNK_FACE_YHI) && Y == g.ny); };
        T px[R + 2], pv[R + 2], pk[R + 2], in[R][NIN], pax[R];
#pragma unroll
        for (int r = 0; r < R + 2; ++r) {
            const int Y = y0 - 1 + r, Yc = min(max(Y, 0), g.ny);
            const long long j = (long long)Yc * g.NX + Xc;
            px[r] = x[j];
            if constexpr (DIR) {
                const T d = (T)v[j];
                pv[r] = xfree && Y == Yc && !ydir(Y) ? d : T(0);
            }
            if constexpr (INV) pk[r] = kap[j];
        }
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const PtrAt at{(long long)min(y0 + k, g.ny) * g.NX + Xc};
            epi.template load<VREG>(at, in[k]);
            if constexpr (VREG) in[k][Epi::VIN] = pv[k + 1];
            pax[k] = PLAIN ? at.ld(Ax, 0) : T(0);
        }
        const bool own = lane >= 1 && lane <= ROW2_COLS && X <= g.nx;
        const bool col = X >= 0 && X < g.nx;
        T c0 = T(0), c1 = T(0);
        T xr = from_right(px[0]), vr = T(0), kr = T(0);
        if constexpr (DIR) vr = from_right(pv[0]);
        if constexpr (INV) kr = from_right(pk[0]);
#pragma unroll
        for (int r = 0; r <= R; ++r) {
            const int ey = y0 - 1 + r;
            const T xn = from_right(px[r + 1]);
            T vn = T(0), kn = T(0);
            if constexpr (DIR) vn = from_right(pv[r + 1]);
            if constexpr (INV) kn = from_right(pk[r + 1]);
            // an element outside the grid (copies of the edge) is selected away
            const bool on = col && ey >= 0 && ey < g.ny && !zero_fd;
            const T xe[1][4] = {{px[r], xr, px[r + 1], xn}};
            T ve[1][4] = {{T(0), T(0), T(0), T(0)}}, kp[4] = {T(0), T(0), T(0), T(0)}, r4[1][4];
            if constexpr (DIR) {
                ve[0][0] = pv[r]; ve[0][1] = vr; ve[0][2] = pv[r + 1]; ve[0][3] = vn;
            }
            if constexpr (INV) {
                kp[0] = pk[r]; kp[1] = kr; kp[2] = pk[r + 1]; kp[3] = kn;
            }
            elem_eval<2, KIND, MODE, T, 1, 4, PF>(xe, ve, kp, e, ph, h, r4);
#pragma unroll
            for (int a = 0; a < 4; ++a) r4[0][a] = on ? r4[0][a] : T(0);
            if (r >= 1) {      // node row r - 1 of the tile is complete
                const int Y = y0 + r - 1;
                T val[1] = {(c0 + r4[0][0]) + from_left(c1 + r4[0][1])};
                const bool dir = MODE != M_COEF && (xdir || ydir(Y));
                if constexpr (PLAIN) val[0] = (val[0] - pax[r - 1]) * ie;
                if (dir || zero_fd) val[0] = T(0);
                if (own && Y <= g.ny) epi.node(PtrAt{(long long)Y * g.NX + X}, val, dir, sums, in[r - 1]);
            }
            c0 = r4[0][2];
            c1 = r4[0][3];
            xr = xn; vr = vn; kr = kn;
        }
    }
    if constexpr (Epi::NS > 0) block_partials<Epi::NS>(sums, red);
}

}  // namespace jfnk
