// Neo-Hookean levels in two kernels: k_nh_elem evaluates every element once
// and writes its corner contributions, summed over the two elements that meet
// in x, to the level's scratch; k_nh_node adds the (up to) four sums of a node
// and applies the epilogue.
//
// The node-centric kernel evaluates each element from all of its 8 corners,
// 64 Gauss points per node, and is bound by that arithmetic.  The exchange
// costs 12 values per element written and read back (about 100 MB each way
// in FP64 at 256 x 64 x 64, which the 256 MB last-level cache holds).  A tile
// that keeps its sums on the chip would evaluate halo elements again: with
// one block per CU at that size 1.6 to 1.9 times the elements.
//
// 256 x 64 x 64, against the node-centric kernel: F(u) FP64 1018 -> 97 us,
// J^T lam 1680 -> 132 us, a Chebyshev step FP32 950 -> 140 us, FP64 2220 ->
// 275 us; at 128 x 32 x 32 a step FP32 195 -> 30 us, FP64 386 -> 47 us.
#pragma once
#include <type_traits>

#include "stencil.hpp"

namespace jfnk {

// Row layout of the scratch: rows (ey + ny ez) of nx + 1 node sums, and the
// seams: past 256 elements in x a row is split over several blocks, and the
// last element of a block leaves its right part in the row's seam entry.
// Entry e of row w and part p = (ay + 2 az) * 3 + component is at
// (p * rows + w) * pitch + e.
struct NhParts {
    int rows, pitch;       // ny nz; nx + 1 + seams
    int chunks;            // blocks per row (1 up to 256 elements)
    int per;               // rows per block
    int threads;
    int blocks;
    size_t entries() const { return (size_t)12 * rows * pitch; }
};
constexpr int NH_BLOCK = 256;
inline NhParts nh_parts(const Grid &g) {
    NhParts p;
    p.rows = g.ny * g.nz;
    p.chunks = (g.nx + NH_BLOCK - 1) / NH_BLOCK;
    p.pitch = g.nx + 1 + (p.chunks - 1);
    p.per = p.chunks > 1 ? 1 : NH_BLOCK / g.nx;
    p.threads = p.chunks > 1 ? NH_BLOCK : (p.per * g.nx + 63) / 64 * 64;
    p.blocks = p.chunks > 1 ? p.rows * p.chunks : (p.rows + p.per - 1) / p.per;
    return p;
}

// The element vector as it stands: no product of its last step is fused into
// the sums that follow, so every kernel forms the same bits from it.
template <typename T> __device__ __forceinline__ void nh_settle(T (*r)[8]) {
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int a = 0; a < 8; ++a) asm volatile("" : "+v"(r[c][a]));
}

// Elements up to which eight lanes share an element (k_nh_elem8).
constexpr long long NH_SPLIT_MAX = 32768;
inline bool nh_split(const Grid &g) { return (long long)g.nx * g.ny * g.nz <= NH_SPLIT_MAX; }
// scratch entries of a level
inline size_t nh_entries(const Grid &g) {
    const size_t e = nh_parts(g).entries(), c = (size_t)24 * g.nx * g.ny * g.nz;
    return nh_split(g) && c > e ? c : e;
}

template <int MODE, typename T, typename TV>
__global__ __launch_bounds__(NH_BLOCK) void k_nh_elem(Grid g, Phys ph, const T *x, const TV *v, FdStep fd, NhParts pt,
                                                      T *w) {
    constexpr bool DIR = MODE != M_RESID;
    __shared__ T sh[12][NH_BLOCK];
    const double eps = fd.eps();
    if ((MODE == M_FD_PLAIN || MODE == M_FD_DIFF) && eps == 0.0) return;     // every product is 0
    const int t = threadIdx.x;
    int row, ex;
    if (pt.chunks > 1) {
        row = blockIdx.x / pt.chunks;
        ex = (blockIdx.x % pt.chunks) * NH_BLOCK + t;
    } else {
        const int k = t / g.nx;
        row = blockIdx.x * pt.per + k;
        ex = t - k * g.nx;
        if (k >= pt.per) row = pt.rows;
    }
    const bool live = row < pt.rows && ex < g.nx;
    const int ey = live ? row % g.ny : 0, ez = live ? row / g.ny : 0;
    T r[3][8];
    if (live) {
        T xe[3][8], ve[3][8];
        bool free_[3][2];       // [axis][side]: the corner's side of the cell is off the Dirichlet faces
        free_[0][0] = !((g.dir & JFNK_FACE_XLO) && ex == 0);
        free_[0][1] = !((g.dir & JFNK_FACE_XHI) && ex + 1 == g.nx);
        free_[1][0] = !((g.dir & JFNK_FACE_YLO) && ey == 0);
        free_[1][1] = !((g.dir & JFNK_FACE_YHI) && ey + 1 == g.ny);
        free_[2][0] = !((g.dir & JFNK_FACE_ZLO) && ez == 0);
        free_[2][1] = !((g.dir & JFNK_FACE_ZHI) && ez + 1 == g.nz);
        const long long j0 = node_index(g, ex, ey, ez);
        const long long sy = g.NX, sz = (long long)g.NX * g.NY;
#pragma unroll
        for (int a = 0; a < 8; ++a) {
            const long long j = j0 + (a & 1) + ((a >> 1) & 1) * sy + ((a >> 2) & 1) * sz;
            const bool fr = free_[0][a & 1] && free_[1][(a >> 1) & 1] && free_[2][(a >> 2) & 1];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                xe[c][a] = x[c * g.nn + j];
                if constexpr (DIR) {
                    const T d = (T)v[c * g.nn + j];
                    ve[c][a] = fr ? d : T(0);
                }
            }
        }
        nh_elem<MODE, T>(xe, ve, (T)eps, ph, (T)g.h, r);
        nh_settle(r);
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int c = 0; c < 3; ++c) sh[p * 3 + c][t] = r[c][2 * p + 1];
    }
    __syncthreads();
    if (!live) return;
    const bool left = ex > 0 && t > 0;        // the element to the left is thread t - 1
    const size_t part = (size_t)pt.rows * pt.pitch;
    T *wr = w + (size_t)row * pt.pitch;
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const int k = p * 3 + c;
            T *wk = wr + k * part;
            const T l = left ? sh[k][t - 1] : T(0);
            wk[ex] = r[c][2 * p] + l;
            if (ex + 1 == g.nx) wk[g.nx] = r[c][2 * p + 1];
            else if (t == NH_BLOCK - 1 && pt.chunks > 1) wk[g.nx + 1 + ex / NH_BLOCK] = r[c][2 * p + 1];
        }
}

// Small levels: eight lanes per element, one per Gauss point, so that the
// launch is not one thread's chain of 8 points.  The lanes exchange halves of
// their 24 corner contributions (mirror images within 8 lanes, then the lane
// pairs 1 and 2 apart), after which lane l holds the element's sum at corner
// 4 l2 + 2 l0 + l1 (l = l0 + 2 l1 + 4 l2).  Entry (corner * 3 + component) of
// element e is at entry * ne + e.  The sums are kept in FP64 on FP32 levels
// too, as the wavefront-per-node kernel does.
template <int CTRL, int N> __device__ __forceinline__ void exchange_half(double *r, bool up) {
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const double keep = up ? r[k + N] : r[k], send = up ? r[k] : r[k + N];
        r[k] = keep + dpp_mov<CTRL>(send);
    }
}
template <int MODE, typename T, typename TV>
__global__ __launch_bounds__(NH_BLOCK) void k_nh_elem8(Grid g, Phys ph, const T *x, const TV *v, FdStep fd, double *w) {
    constexpr bool DIR = MODE != M_RESID;
    const double eps = fd.eps();
    if ((MODE == M_FD_PLAIN || MODE == M_FD_DIFF) && eps == 0.0) return;
    const int ne = g.nx * g.ny * g.nz;
    const int t = blockIdx.x * NH_BLOCK + threadIdx.x;
    const int el = min(t >> 3, ne - 1), gq = t & 7;      // lanes past the level repeat its last element
    unsigned q, rx, q2, ry;
    udivmod((unsigned)el, (unsigned)g.nx, 1.0 / g.nx, q, rx);
    udivmod(q, (unsigned)g.ny, 1.0 / g.ny, q2, ry);
    const int ex = (int)rx, ey = (int)ry, ez = (int)q2;
    T xe[3][8], ve[3][8], r8[3][8];
#pragma unroll
    for (int a = 0; a < 8; ++a) {
        const int ax = ex + (a & 1), ay = ey + ((a >> 1) & 1), az = ez + ((a >> 2) & 1);
        const long long j = node_index(g, ax, ay, az);
        const bool dj = DIR && is_dirichlet(g, ax, ay, az);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            xe[c][a] = x[c * g.nn + j];
            ve[c][a] = T(0);
            if constexpr (DIR) {
                const T d = (T)v[c * g.nn + j];
                ve[c][a] = dj ? T(0) : d;
            }
            if constexpr (MODE == M_FD_PLAIN) xe[c][a] += (T)eps * ve[c][a];
            r8[c][a] = T(0);
        }
    }
    if constexpr (MODE == M_FD_DIFF) nh_point_fd<T>(xe, ve, (T)eps, ph, (T)g.h, gq, r8);
    else if constexpr (MODE == M_VJP) nh_point_jvp<T>(xe, ve, ph, (T)g.h, gq, r8);
    else nh_point<T>(xe, ph, (T)g.h, gq, r8);
    double r[24];
#pragma unroll
    for (int a = 0; a < 8; ++a)
#pragma unroll
        for (int c = 0; c < 3; ++c) r[3 * a + c] = (double)r8[c][a];
    exchange_half<0x141, 12>(r, (gq & 4) != 0);      // row_half_mirror: lane 7 - l
    exchange_half<0xB1, 6>(r, (gq & 1) != 0);        // lane ^ 1
    exchange_half<0x4E, 3>(r, (gq & 2) != 0);        // lane ^ 2
    if ((t >> 3) < ne) {
        const int a = (gq & 4) + 2 * (gq & 1) + ((gq >> 1) & 1);
#pragma unroll
        for (int c = 0; c < 3; ++c) w[(size_t)(3 * a + c) * ne + el] = r[c];
    }
}

// EIGHT: w holds the corner contributions of every element (k_nh_elem8)
template <int MODE, bool EIGHT, typename T, class Epi>
__global__ __launch_bounds__(BLOCK) void k_nh_node(Grid g, const std::conditional_t<EIGHT, double, T> *w, NhParts pt, const T *Ax, FdStep fd, Epi epi,
                                                   Red red) {
    constexpr bool FD = MODE == M_FD_PLAIN || MODE == M_FD_DIFF;
    const double eps = fd_eps_prepare(fd, epi);
    const T ie = MODE == M_FD_PLAIN && eps > 0.0 ? (T)(1.0 / eps) : T(0);
    double sums[Epi::NS > 0 ? Epi::NS : 1];
#pragma unroll
    for (int k = 0; k < (Epi::NS > 0 ? Epi::NS : 1); ++k) sums[k] = 0.0;
    const size_t part = (size_t)pt.rows * pt.pitch;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < g.nn; i += stride) {
        int X, Y, Z;
        node_coords(g, i, X, Y, Z);
        const bool dir = is_dirichlet(g, X, Y, Z);
        T in[Epi::NIN * 3 > 0 ? Epi::NIN * 3 : 1];
        const PtrAt at{i};
        epi.load(at, in);
        T val[3] = {T(0), T(0), T(0)};
        if (EIGHT && !dir && !(FD && eps == 0.0)) {
            const int ne = g.nx * g.ny * g.nz;
            double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
            for (int a = 0; a < 8; ++a) {
                const int ex = X - (a & 1), ey = Y - ((a >> 1) & 1), ez = Z - ((a >> 2) & 1);
                const bool in_ = ex >= 0 && ex < g.nx && ey >= 0 && ey < g.ny && ez >= 0 && ez < g.nz;
                const int el = in_ ? (ez * g.ny + ey) * g.nx + ex : 0;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const double p = (double)w[(size_t)(3 * a + c) * ne + el];
                    s[c] += in_ ? p : 0.0;
                }
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) val[c] = (T)s[c];
        }
        if (!EIGHT && !dir && !(FD && eps == 0.0)) {
            // the element rows around the node: it lies on side ay, az of row (Y - ay, Z - az)
            const bool seam = pt.chunks > 1 && X > 0 && X < g.nx && X % NH_BLOCK == 0;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const int ey = Y - (p & 1), ez = Z - (p >> 1);
                if (ey < 0 || ey >= g.ny || ez < 0 || ez >= g.nz) continue;
                const auto *wr = w + (size_t)(p * 3) * part + (size_t)(ez * g.ny + ey) * pt.pitch;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    val[c] += (T)wr[c * part + X];
                    if (seam) val[c] += (T)wr[c * part + g.nx + X / NH_BLOCK];
                }
            }
        }
        if constexpr (MODE == M_FD_PLAIN) {
            if (!dir && eps != 0.0) {
#pragma unroll
                for (int c = 0; c < 3; ++c) val[c] = (val[c] - Ax[c * g.nn + i]) * ie;
            }
        }
        epi.node(at, val, dir, sums, in);
    }
    if constexpr (Epi::NS > 0) block_partials<Epi::NS>(sums, red);
}

// Node values of the Neo-Hookean kind with one wavefront per node: lane l
// evaluates Gauss point l & 7 of element l >> 3 around the node (the
// element whose corner l >> 3 the node is), and the wave sums the 64 parts
// by DPP in a fixed order.  One launch for the smallest levels: every point is
// evaluated 8 times over, but in parallel.  Every lane of a wave walks the same
// nodes, so the sums are wave-uniform; lane 0 applies the epilogue.
template <int MODE, typename T, typename TV, class Epi>
__global__ __launch_bounds__(BLOCK) void k_node_nh(Grid g, Phys ph, const T *x, const TV *v, const T *Ax,
                                                   FdStep fd, Epi epi, Red red) {
    constexpr int NC = 3;
    const double eps = fd_eps_prepare(fd, epi);
    double sums[Epi::NS > 0 ? Epi::NS : 1];
#pragma unroll
    for (int k = 0; k < (Epi::NS > 0 ? Epi::NS : 1); ++k) sums[k] = 0.0;
    const long long nn = g.nn;
    const int lane = threadIdx.x & 63;
    const int el = lane >> 3, gq = lane & 7;
    const long long wave = ((long long)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const long long nwaves = ((long long)gridDim.x * blockDim.x) >> 6;
    const T h = (T)g.h, e = (T)eps;
    for (long long i = wave; i < nn; i += nwaves) {
        int X, Y, Z;
        node_coords(g, i, X, Y, Z);
        const bool dir = is_dirichlet(g, X, Y, Z);
        const bool eval = !dir && !(MODE != M_RESID && eps == 0.0);
        const int ex = X - (el & 1), ey = Y - ((el >> 1) & 1), ez = Z - ((el >> 2) & 1);
        const bool inside = eval && ex >= 0 && ex < g.nx && ey >= 0 && ey < g.ny && ez >= 0 && ez < g.nz;
        T c3[NC] = {T(0), T(0), T(0)};
        if (inside) {
            T xe[NC][8], ve[NC][8], r8[NC][8];
#pragma unroll
            for (int a = 0; a < 8; ++a) {
                const int ax = ex + (a & 1), ay = ey + ((a >> 1) & 1), az = ez + ((a >> 2) & 1);
                const long long j = node_index(g, ax, ay, az);
                const bool dj = (MODE != M_RESID) && is_dirichlet(g, ax, ay, az);
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    xe[c][a] = x[c * nn + j];
                    ve[c][a] = (MODE == M_RESID || dj) ? T(0) : (T)v[c * nn + j];
                    r8[c][a] = T(0);
                }
            }
            if constexpr (MODE == M_FD_DIFF) {
                nh_point_fd<T>(xe, ve, e, ph, h, gq, r8);
            } else if constexpr (MODE == M_FD_PLAIN) {
                T w[NC][8];
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int a = 0; a < 8; ++a) w[c][a] = xe[c][a] + e * ve[c][a];
                nh_point<T>(w, ph, h, gq, r8);
            } else {
                nh_point<T>(xe, ph, h, gq, r8);
            }
#pragma unroll
            for (int a = 0; a < 8; ++a)
                if (a == el) {
#pragma unroll
                    for (int c = 0; c < NC; ++c) c3[c] = r8[c][a];
                }
        }
        T val[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            double s = (double)c3[c];
            if constexpr (sizeof(T) == 4) {
                val[c] = (T)wave_sum(s);
                continue;
            }
            // FP64: the 8 points of an element, then the elements in corner
            // order, as k_nh_elem8 and k_nh_node add them (the residual without
            // scratch has the same bits)
            s += dpp_mov<0x141>(s);
            s += dpp_mov<0xB1>(s);
            s += dpp_mov<0x4E>(s);
            double sum = 0.0;
#pragma unroll
            for (int a = 0; a < 8; ++a) sum += read_lane(s, 8 * a);
            val[c] = (T)sum;
        }
        if (lane == 0) {
            if constexpr (MODE == M_FD_PLAIN) {
                if (eval) {
                    const T ie = (T)(1.0 / eps);
#pragma unroll
                    for (int c = 0; c < NC; ++c) val[c] = (val[c] - Ax[c * nn + i]) * ie;
                }
            }
            T in[Epi::NIN * NC > 0 ? Epi::NIN * NC : 1];
            const PtrAt at{i};
            epi.load(at, in);
            epi.node(at, val, dir, sums, in);
        }
    }
    if constexpr (Epi::NS > 0) block_partials<Epi::NS>(sums, red);
}

// The residual without scratch (jfnk_residual_static) on large levels: a
// thread per node, its 8 elements evaluated one after the other and summed in
// the order of k_nh_elem and k_nh_node, so both give the same bits.
template <typename T, class Epi>
__global__ __launch_bounds__(BLOCK) void k_nh_direct(Grid g, Phys ph, const T *x, NhParts pt, Epi epi, Red red) {
    double sums[1] = {0.0};
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < g.nn; i += stride) {
        int X, Y, Z;
        node_coords(g, i, X, Y, Z);
        const bool dir = is_dirichlet(g, X, Y, Z);
        const bool seam = pt.chunks > 1 && X > 0 && X < g.nx && X % NH_BLOCK == 0;
        T val[3] = {T(0), T(0), T(0)}, l[3] = {T(0), T(0), T(0)};
        for (int e = 0; e < 8 && !dir; ++e) {
            // element on side ax = e & 1 of the node in row (Y - ay, Z - az): corner e of it
            const int ex = X - (e & 1), ey = Y - ((e >> 1) & 1), ez = Z - (e >> 2);
            T c3[3] = {T(0), T(0), T(0)};
            const bool row = ey >= 0 && ey < g.ny && ez >= 0 && ez < g.nz, in_ = row && ex >= 0 && ex < g.nx;
            if (in_) {
                T xe[3][8], r[3][8];
#pragma unroll
                for (int a = 0; a < 8; ++a) {
                    const long long j = node_index(g, ex + (a & 1), ey + ((a >> 1) & 1), ez + ((a >> 2) & 1));
#pragma unroll
                    for (int c = 0; c < 3; ++c) xe[c][a] = x[c * g.nn + j];
                }
                nh_elem<M_RESID, T>(xe, xe, T(0), ph, (T)g.h, r);
                nh_settle(r);
#pragma unroll
                for (int a = 0; a < 8; ++a)
                    if (a == e) {
#pragma unroll
                        for (int c = 0; c < 3; ++c) c3[c] = r[c][a];
                    }
            }
            if (!row) continue;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                if (!(e & 1)) {
                    l[c] = c3[c];                      // the element to the right: its left part
                } else if (seam) {
                    val[c] += l[c] + T(0);
                    val[c] += c3[c];
                } else {
                    val[c] += X == g.nx ? c3[c] : l[c] + c3[c];
                }
            }
        }
        T in[3];
        const PtrAt at{i};
        epi.load(at, in);
        epi.node(at, val, dir, sums, in);
    }
    block_partials<1>(sums, red);
}

}  // namespace jfnk
