// Viscous stress of the liquid (eq. stressTensor) in the mixture fluxes (gfx950).
//
// T = mu (grad u + grad u^T - 2/3 div(u) I) enters the momentum flux as -T and the energy flux as -T.u
// (eq. euler_transport).  It is a separate pass that runs after a stage kernel when the problem is
// viscous, so the stage kernels carry no code for it: every owned cell forms the viscous fluxes through
// its 2 ndim faces from the velocities of the stage's input state (the primitive scratch P), by
// second-order central differences at the face -- normal derivatives from the two cells beside it,
// transverse derivatives as the mean of those two cells' central differences, face velocity the mean
// of the two cells' -- and adds scale * (F_lo - F_hi)/dx to the momentum and energy the stage wrote
// (scale = b dt of the RK combine, 1 for a right-hand side).  Mirrored ghost cells negate the velocity
// component along the mirrored direction.
#pragma once

#include "device_common.hpp"
#include "ee_kernels.hpp"

namespace bub {

// qo (momentum and energy) += scale * viscous rates of every cell; scale = b * (*dtp), or 1 when dtp is null.
// A thread loads the velocities of its cell's neighbourhood once (3, 9 or, without the corners, 19 cells, each
// coordinate through the ghost-cell map once) and forms the fluxes of its 2 ndim faces from them in registers, every
// index known at compile time.  The form before loaded each face's six or ten cells for itself through run-time axes
// and divided 64-bit indices: 600 x 150 cells 12.3 to 4.9 us, of which a launch is about 4.
template <int D>
__global__ void __launch_bounds__(256) k_viscous(const double *__restrict__ P, double *__restrict__ qo, Grid g,
                                                 double mu, const double *__restrict__ dtp, double b)
{
    const double scale = dtp ? b * *dtp : 1.0;
    const long long N = g.N;
    constexpr int NY = D > 1 ? 3 : 1, NZ = D > 2 ? 3 : 1;
    for (long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x; c < N; c += (long long)gridDim.x * blockDim.x) {
        const unsigned row = (unsigned)c / (unsigned)g.n[0];
        const int co[3] = {(int)((unsigned)c - row * (unsigned)g.n[0]), D > 2 ? (int)(row % (unsigned)g.n[1]) : (int)row,
                           D > 2 ? (int)(row / (unsigned)g.n[1]) : 0};
        // the cells at -1, 0 and +1 along each axis, and whether they are mirrored there
        int at[3][3];
        bool fl[3][3];
#pragma unroll
        for (int e = 0; e < 3; ++e)
#pragma unroll
            for (int o = 0; o < 3; ++o) {
                at[e][o] = co[e];
                fl[e][o] = false;
                if (e < D && o != 1) at[e][o] = map_coord(co[e] + o - 1, g.n[e], g.bc[e], fl[e][o]);
            }
        double u[NZ][NY][3][D];
#pragma unroll
        for (int k = 0; k < NZ; ++k)
#pragma unroll
            for (int j = 0; j < NY; ++j)
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const int o[3] = {i, D > 1 ? j : 1, D > 2 ? k : 1};
                    if (o[0] != 1 && o[1] != 1 && o[2] != 1) continue;
                    const long long gi = (long long)at[0][o[0]] +
                                         (long long)g.n[0] * ((long long)at[1][o[1]] + (long long)g.n[1] * at[2][o[2]]);
#pragma unroll
                    for (int v = 0; v < D; ++v) {
                        const double x = P[(long long)(PL<D>::U + v) * N + gi];
                        u[k][j][i][v] = fl[v][o[v]] ? -x : x;
                    }
                }
        double L[D + 1];
#pragma unroll
        for (int k = 0; k <= D; ++k) L[k] = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            double F[2][D + 1];   // through the lower and the upper face of direction d
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                // velocity component v of the cell left (side 0) or right of the face, `oe` along axis e
                auto vel = [&](int side, int e, int oe, int v) {
                    int o[3] = {1, 1, 1};
                    o[d] = s + side;
                    if (e >= 0) o[e] = 1 + oe;
                    return u[D > 2 ? o[2] : 0][D > 1 ? o[1] : 0][o[0]][v];
                };
                double gr[D][D];   // gr[k][e] = d u_k / d x_e at the face
#pragma unroll
                for (int k = 0; k < D; ++k)
#pragma unroll
                    for (int e = 0; e < D; ++e)
                        gr[k][e] = e == d ? (vel(1, -1, 0, k) - vel(0, -1, 0, k)) * g.inv_dx[d]
                                          : ((vel(0, e, 1, k) - vel(0, e, -1, k)) + (vel(1, e, 1, k) - vel(1, e, -1, k))) *
                                                (0.25 * g.inv_dx[e]);
                double div = 0.0;
#pragma unroll
                for (int e = 0; e < D; ++e) div += gr[e][e];
                double work = 0.0;
#pragma unroll
                for (int k = 0; k < D; ++k) {
                    const double T = mu * (gr[d][k] + gr[k][d] - (k == d ? (2.0 / 3.0) * div : 0.0));
                    F[s][k] = -T;
                    work += T * 0.5 * (vel(0, -1, 0, k) + vel(1, -1, 0, k));
                }
                F[s][D] = -work;
            }
#pragma unroll
            for (int k = 0; k <= D; ++k) L[k] += (F[0][k] - F[1][k]) * g.inv_dx[d];
        }
#pragma unroll
        for (int k = 0; k < D; ++k) qo[(long long)(1 + k) * N + c] += scale * L[k];
        qo[(long long)(D + 1) * N + c] += scale * L[D];
    }
}

}  // namespace bub
