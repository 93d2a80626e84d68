// 3D levels of the scalar kinds: one wavefront marches up in z over a tile of
// 62 node columns and R node rows in y, without LDS and without a barrier.
//
// The columns of all rows that are a multiple of R are numbered through
// (p = x + NX * group, group g owning the rows gR .. gR + R - 1), and lane l of
// a wave owns column 62 s + l - 1 of that numbering, so no lane idles at the
// end of a grid row.  A lane evaluates the element column to its right: the
// corner values of the next column and the contributions to it cross by
// wavefront shifts (DPP).  Infinities and NaN stay with the nodes of their own
// elements: where the next lane starts another group the element has corners
// far apart, and what it gives to either side is selected away at the node; in
// the rows off the grid the element is the mirror image of the one at the edge
// (its rows are loaded mirrored), so that the factor 0 that switches it off meets
// an infinity or a NaN only where that element has one.  The y neighbours of a node are
// summed in registers along the lane's R + 1 elements of a layer, the z
// neighbours by a register carry from layer to layer, so every element of a
// tile is evaluated once.  The planes z and z + 1 of the state (and direction
// and coefficient) stay in registers; plane z + 2 and the epilogue's inputs
// are loaded before the element work of layer z.
//
// The waves are independent: no barrier separates the loads of one from the
// arithmetic of another, and the corner values cost one lane shift instead of
// LDS writes and reads.  A block that spanned the whole x extent with two
// planes in LDS and two barriers per plane issued 774 VALU instructions per
// plane of 4 rows in the FP32 Chebyshev step (this kernel 656) and took, at
// 256^3, 141 us against 112 us here, 124 against 99 us for the FP64 residual
// (4.1 TB/s; a copy reaches 4.7 TB/s); a degree-4 FP64 smoother 143 against 98
// us at 128^3, 54 against 36 us at 64^3; in FP32 at 32^3 26 (node-centric)
// against 19 us.
#pragma once
#include "stencil_2d.hpp"

namespace jfnk {

// Most rows per wave (1, 2 and 4 are compiled): the FP64 Gauss-point element
// leaves no registers for 4 rows.
template <typename T, int KIND> constexpr int wave_rows_max = sizeof(T) == 8 && KIND == JFNK_PLAP_GAUSS ? 2 : 4;

struct WaveTile {
    int strips;      // waves along the numbered columns
    int ntz;         // z chunks
};

template <int KIND, int MODE, typename T, typename TV, class Epi, int PF, int R>
__global__ __launch_bounds__(BLOCK) void k_wave3(Grid g, Phys ph, const T *kap, const T *x, const TV *v, const T *Ax,
                                                 FdStep fd, Epi epi, Red red, WaveTile wt) {
    constexpr bool DIR = MODE != M_RESID;                            // has a direction v
    constexpr bool FD = MODE == M_FD_PLAIN || MODE == M_FD_DIFF;     // with a step eps
    constexpr bool INV = KIND == JFNK_INVCOEF;
    constexpr bool PLAIN = MODE == M_FD_PLAIN;
    constexpr bool VREG = DIR && Epi::VIN >= 0;
    constexpr int NIN = Epi::NIN > 0 ? Epi::NIN : 1;
    const double eps = fd_eps_prepare(fd, epi);
    const bool zero_fd = FD && eps == 0.0;
    const T e = (T)eps, ie = PLAIN && eps > 0.0 ? (T)(1.0 / eps) : T(0), h = (T)g.h;
    double sums[Epi::NS > 0 ? Epi::NS : 1];
#pragma unroll
    for (int k = 0; k < (Epi::NS > 0 ? Epi::NS : 1); ++k) sums[k] = 0.0;

    const int tiles = wt.strips * wt.ntz;
    int tile = __builtin_amdgcn_readfirstlane(xcd_tile(blockIdx.x, gridDim.x) * (BLOCK / 64) + (threadIdx.x >> 6));
    if (tile < tiles) do {
        const int lane = threadIdx.x & 63;
        const int chunk = tile / wt.strips;
        const int z0 = (int)((long long)chunk * g.NZ / wt.ntz), z1 = (int)((long long)(chunk + 1) * g.NZ / wt.ntz);
        const int p = (tile % wt.strips) * ROW2_COLS - 1 + lane;
        const int grp = p < 0 ? 0 : p / g.NX;
        const int X = p < 0 ? 0 : p - grp * g.NX, Y0 = grp * R;
        const bool in_ = p >= 0 && Y0 < g.NY;
        const bool xdir = ((g.dir & JFNK_FACE_XLO) && X == 0) || ((g.dir & JFNK_FACE_XHI) && X == g.nx);
        const int nxy = g.NX * g.NY;
        const bool xin = in_ && X < g.nx;       // the element column right of X exists
        // per-lane masks: fr[r] the direction is free in row Y0 - 1 + r, el[r] the
        // element row above that row exists, own[k] the lane stores row Y0 + k,
        // dr[k] that row's node is on a Dirichlet face in x or y
        unsigned col[R + 2];
        bool fr[R + 2], el[R + 1], own[R], dr[R];
#pragma unroll
        for (int r = 0; r < R + 2; ++r) {
            const int Y = Y0 - 1 + r, Ym = Y < 0 ? 1 : Y > g.ny ? max(2 * g.ny - Y, 0) : Y;
            col[r] = (unsigned)(Ym * g.NX + X);
            const bool yd = ((g.dir & JFNK_FACE_YLO) && Ym == 0) || ((g.dir & JFNK_FACE_YHI) && Ym == g.ny);
            fr[r] = in_ && !yd && !xdir;
            if (r <= R) el[r] = Y >= 0 && Y < g.ny;
            if (r >= 1 && r <= R) {
                own[r - 1] = in_ && lane >= 1 && lane <= ROW2_COLS && Y <= g.ny;
                dr[r - 1] = xdir || yd;
            }
        }
        auto zdir = [&](int z) { return ((g.dir & JFNK_FACE_ZLO) && z == 0) || ((g.dir & JFNK_FACE_ZHI) && z == g.nz); };
        // raw plane loads (clamped), and the masks applied when they are taken over
        auto fetch = [&](int z, T *px, TV *pv, T *pk) {
            const unsigned row = (unsigned)(min(max(z, 0), g.nz) * nxy);
#pragma unroll
            for (int r = 0; r < R + 2; ++r) {
                const BufAt at{row, col[r]};
                px[r] = at.ld(x, 0);
                if constexpr (DIR) pv[r] = at.ld(v, 0);
                if constexpr (INV) pk[r] = at.ld(kap, 0);
            }
        };
        T lx[R + 2], hx[R + 2], lk[R + 2], hk[R + 2], fx[R + 2], fk[R + 2];
        T lv[R + 2], hv[R + 2];
        TV fv[R + 2];
        auto take = [&](int z, T *px, T *pv, T *pk) {
            const bool zf = z >= 0 && z <= g.nz && !zdir(z);
#pragma unroll
            for (int r = 0; r < R + 2; ++r) {
                px[r] = fx[r];
                if constexpr (DIR) pv[r] = zf && fr[r] ? (T)fv[r] : T(0);
                if constexpr (INV) pk[r] = fk[r];
            }
        };
        T C0[R], C1[R], O[R], T1[R];
#pragma unroll
        for (int k = 0; k < R; ++k) C0[k] = C1[k] = O[k] = T1[k] = T(0);
        // element layer between the planes l and h; finishes the node rows of plane l
        auto layer = [&]() __attribute__((always_inline)) {
            T cx[4], cv[4], ck[4];
            auto row = [&](int r, T *ox, T *ov, T *ok) {
                ox[0] = lx[r]; ox[1] = from_right(lx[r]); ox[2] = hx[r]; ox[3] = from_right(hx[r]);
                if constexpr (DIR) { ov[0] = lv[r]; ov[1] = from_right(lv[r]); ov[2] = hv[r]; ov[3] = from_right(hv[r]); }
                if constexpr (INV) { ok[0] = lk[r]; ok[1] = from_right(lk[r]); ok[2] = hk[r]; ok[3] = from_right(hk[r]); }
            };
            row(0, cx, cv, ck);
            T pS0 = T(0), pS1 = T(0), pN0 = T(0), pN1 = T(0);
#pragma unroll
            for (int re = 0; re <= R; ++re) {
                T ux[4], uv[4], uk[4], r8[1][8];
                row(re + 1, ux, uv, uk);
                const T xe[1][8] = {{cx[0], cx[1], ux[0], ux[1], cx[2], cx[3], ux[2], ux[3]}};
                T ve[1][8], kp[8];
                if constexpr (DIR) {
                    const T w[8] = {cv[0], cv[1], uv[0], uv[1], cv[2], cv[3], uv[2], uv[3]};
#pragma unroll
                    for (int a = 0; a < 8; ++a) ve[0][a] = w[a];
                }
                if constexpr (INV) {
                    const T w[8] = {ck[0], ck[1], uk[0], uk[1], ck[2], ck[3], uk[2], uk[3]};
#pragma unroll
                    for (int a = 0; a < 8; ++a) kp[a] = w[a];
                }
                elem_eval<3, KIND, MODE, T, 1, 8, PF>(xe, ve, kp, e, ph, h, r8, el[re] ? T(1) : T(0));
                if (re >= 1) {
                    const int k = re - 1;
                    O[k] = C0[k] + (pS0 + r8[0][0]);
                    T1[k] = C1[k] + (pS1 + r8[0][1]);
                    C0[k] = pN0 + r8[0][4];
                    C1[k] = pN1 + r8[0][5];
                }
                pS0 = r8[0][2]; pS1 = r8[0][3]; pN0 = r8[0][6]; pN1 = r8[0][7];
#pragma unroll
                for (int c = 0; c < 4; ++c) { cx[c] = ux[c]; cv[c] = uv[c]; ck[c] = uk[c]; }
            }
        };
        fetch(z0 - 1, fx, fv, fk);
        take(z0 - 1, lx, lv, lk);
        fetch(z0, fx, fv, fk);
        take(z0, hx, hv, hk);
        fetch(z0 + 1, fx, fv, fk);
        if (z0 > 0 && !zero_fd) layer();
#pragma unroll
        for (int r = 0; r < R + 2; ++r) { lx[r] = hx[r]; lv[r] = hv[r]; lk[r] = hk[r]; }
        take(z0 + 1, hx, hv, hk);
        for (int z = z0; z < z1; ++z) {
            T in[R][NIN], pax[R];
            const unsigned prow = (unsigned)(z * nxy);
            if (z + 1 < z1) fetch(z + 2, fx, fv, fk);
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const BufAt at{prow, col[k + 1]};
                epi.template load<VREG>(at, in[k]);
                if constexpr (VREG) in[k][Epi::VIN] = lv[k + 1];
                pax[k] = PLAIN ? at.ld(Ax, 0) : T(0);
            }
            if (z < g.nz && !zero_fd) {
                layer();
            } else {
#pragma unroll
                for (int k = 0; k < R; ++k) { O[k] = C0[k]; T1[k] = C1[k]; }
            }
            const bool zd = zdir(z);
#pragma unroll
            for (int k = 0; k < R; ++k) {
                T val[1] = {(xin ? O[k] : T(0)) + from_left(xin ? T1[k] : T(0))};
                const bool dir = MODE != M_COEF && (zd || dr[k]);
                if constexpr (PLAIN) val[0] = (val[0] - pax[k]) * ie;
                if (dir || zero_fd) val[0] = T(0);
                if (own[k]) epi.node(BufAt{prow, col[k + 1]}, val, dir, sums, in[k]);
            }
#pragma unroll
            for (int r = 0; r < R + 2; ++r) { lx[r] = hx[r]; lv[r] = hv[r]; lk[r] = hk[r]; }
            if (z + 1 < z1) take(z + 2, hx, hv, hk);
        }
        // only the residual's waves walk over several tiles (WAVE_BLOCKS_MAX); as
        // a loop in the FD modes this cost 20% (branches where masks were)
        if constexpr (MODE != M_RESID) break;
        tile += gridDim.x * (BLOCK / 64);
    } while (tile < tiles);
    if constexpr (Epi::NS > 0) block_partials<Epi::NS>(sums, red);
}

}  // namespace jfnk
