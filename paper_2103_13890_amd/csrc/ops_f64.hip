// FP64 element sums outside the stencil launchers: the energy.
#include "stencil_nh.hpp"
#include "ops.hpp"

namespace jfnk {

size_t nh_scratch_entries(const Grid &g) { return nh_entries(g); }

// ---- energy: sum over elements of Psi_e(u) ----------------------------------
template <int DIM, int KIND>
__global__ __launch_bounds__(BLOCK) void k_energy(Grid g, Phys ph, const double *u, Red red, double *out) {
    constexpr int NV = Cell<DIM>::NV;
    constexpr int NC = (KIND == JFNK_NEOHOOKE) ? 3 : 1;
    const long long ne = (long long)g.nx * g.ny * (DIM == 3 ? g.nz : 1);
    double sum[1] = {0.0};
    const long long stride = (long long)gridDim.x * blockDim.x;
    const double rnx = 1.0 / g.nx, rny = 1.0 / g.ny;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < ne; e += stride) {
        unsigned q, r, q2, r2;
        udivmod((unsigned)e, (unsigned)g.nx, rnx, q, r);
        udivmod(q, (unsigned)g.ny, rny, q2, r2);
        const int ex = (int)r, ey = (int)r2, ez = (int)q2;
        double w[NC][NV];
#pragma unroll
        for (int a = 0; a < NV; ++a) {
            const long long j = node_index(g, ex + (a & 1), ey + ((a >> 1) & 1), ez + ((a >> 2) & 1));
#pragma unroll
            for (int c = 0; c < NC; ++c) w[c][a] = u[c * g.nn + j];
        }
        if constexpr (KIND == JFNK_NEOHOOKE) sum[0] += elem_neohooke_energy<double>(w, ph, g.h);
        else sum[0] += elem_scalar_energy<DIM, KIND, double>(w[0], ph, g.h);
    }
    block_partials<1>(sum, red);
}

void op_energy(const Exec &ex, const Grid &g, const Phys &ph, const double *u, double *out) {
    const long long ne = (long long)g.nx * g.ny * (g.dim == 3 ? g.nz : 1);
    const int nb = node_blocks(ne);
    if (ph.kind == JFNK_BRATU && g.dim == 2) k_energy<2, JFNK_BRATU><<<nb, BLOCK, 0, ex.st>>>(g, ph, u, ex.red, out);
    else if (ph.kind == JFNK_BRATU) k_energy<3, JFNK_BRATU><<<nb, BLOCK, 0, ex.st>>>(g, ph, u, ex.red, out);
    else if (ph.kind == JFNK_PLAP && g.dim == 2) k_energy<2, JFNK_PLAP><<<nb, BLOCK, 0, ex.st>>>(g, ph, u, ex.red, out);
    else if (ph.kind == JFNK_PLAP) k_energy<3, JFNK_PLAP><<<nb, BLOCK, 0, ex.st>>>(g, ph, u, ex.red, out);
    else if (ph.kind == JFNK_NEOHOOKE) k_energy<3, JFNK_NEOHOOKE><<<nb, BLOCK, 0, ex.st>>>(g, ph, u, ex.red, out);
    else if (ph.kind == JFNK_PLAP_GAUSS && g.dim == 2)
        k_energy<2, JFNK_PLAP_GAUSS><<<nb, BLOCK, 0, ex.st>>>(g, ph, u, ex.red, out);
    else if (ph.kind == JFNK_PLAP_GAUSS) k_energy<3, JFNK_PLAP_GAUSS><<<nb, BLOCK, 0, ex.st>>>(g, ph, u, ex.red, out);
    finish<1>(ex.st, ex.red, nb, FinStore<1>{out});
}

}  // namespace jfnk
