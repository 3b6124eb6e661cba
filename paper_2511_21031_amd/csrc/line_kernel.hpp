// The RK-stage kernel of 1D grids: one wavefront per tile of 63 cells and group of bins (gfx950).
//
// Lane l holds cell x0 + l of the tile and computes the face at its low side; lane 63 computes only the last
// cell's high face, and a cell takes its high face's flux from the next lane.  What a tile costs here is its
// latency, not its throughput (a 1D grid has a few dozen tiles): the mixture face of a lane is one long
// chain, then come the group's bins, a face each.  So a workgroup is one wave, which needs no barrier (LDS
// operations of a wave complete in order), an owned cell stays in its lane's registers, and the bins are
// spread over as many waves as there are pairs of them.  Against a tile of 255 cells on four waves: right-hand
// side of 400 cells x 11 bins 12.7 to 11.0 us (primitive pass included), split mixed step of 2000 cells x 31
// bins 78 to 68 us.
#pragma once

#include "stage_kernel.hpp"

namespace bub {

// Order of a wave's LDS writes and the reads of other lanes' values that follow (no instruction).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The value of the next lane (lane 63: zero).
__device__ __forceinline__ double next_lane(double x)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    const unsigned lo = __builtin_amdgcn_update_dpp(0u, (unsigned)b, 0x130, 0xf, 0xf, true);
    const unsigned hi = __builtin_amdgcn_update_dpp(0u, (unsigned)(b >> 32), 0x130, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ float next_lane(float x)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), 0x130, 0xf, 0xf, true));
}

// A launch of the kernel: RK stage, RK stage with the primitive pass of its result, right-hand side.
enum LineMode : int { LM_RK = 0, LM_FUSE = 1, LM_RHS = 2 };

constexpr int LINE_TX = 63;        // cells of a tile
constexpr int LINE_SLOTS = 72;     // staged cells -3 .. 65, and a slot for lanes without a halo cell

// SRC: the bubble sources are in the stage; UN: the combine reads u^n.
template <typename TF, int CT, int MODE, bool SRC, bool UN>
__global__ void __launch_bounds__(64) k_line(StageArgs A, Grid g, Phys ph, Bins bins)
{
    constexpr bool TR = CT == CT_TRANSFER, FUSE = MODE == LM_FUSE, RHS = MODE == LM_RHS;
    constexpr int NP = TR ? 2 : 1, NF = 2 * NP, NCF = 4;
    using PT = Pair<TF>;
    __shared__ PT s_q[NP][LINE_SLOTS];
    const int b = blockIdx.x;
    const int item = (b & 7) * A.nblk_per_xcd + (b >> 3);
    if (item >= A.nitems) return;
    const int tile = item / A.ngroups, grp = item - tile * A.ngroups;
    const int b0 = grp * A.bpg, b1 = b0 + A.bpg < bins.nb ? b0 + A.bpg : bins.nb;
    const bool core_out = grp == 0;
    const int lane = threadIdx.x;
    const long long N = g.N;
    const int nb = bins.nb, nx = g.n[0];
    const int x0 = tile * LINE_TX;
    const bool act = lane < LINE_TX && x0 + lane < nx;
    bool dum = false;
    const long long c = map_coord(x0 + lane, nx, g.bc[0], dum);
    // one x-halo cell (columns -3, -2, -1, 64, 65) for each of the first five lanes
    const int hx = lane < 3 ? lane - 3 : 61 + lane;
    const long long ch = lane < 5 ? map_coord(x0 + hx, nx, g.bc[0], dum) : c;
    const int hslot = lane < 5 ? hx + 3 : LINE_SLOTS - 1;

    // ---- loads of the first bin, ahead of the mixture face ----
    double raw[NF], raw_h[NF], un[NF];
    auto load = [&](int ib) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const long long o = (long long)(4 + f * nb + ib) * N;
            raw[f] = A.qk[o + c];
            raw_h[f] = A.qk[o + ch];
            if constexpr (UN) un[f] = A.qn[o + c];
        }
    };
    load(b0);

    // ---- mixture face and update of the owned cell ----
    TF F[NCF], coef, Lc[NCF];
    bool right, ok;
    {
        long long c6[6];
        bool fx6[6];
#pragma unroll
        for (int o = 0; o < 6; ++o) {
            fx6[o] = false;
            c6[o] = map_coord(x0 + lane - 3 + o, nx, g.bc[0], fx6[o]);
        }
        core_face<1, 0, TF>([&](int v, int o) { return (TF)A.P[(long long)v * N + c6[o]]; }, fx6, ph, F, coef, right, ok);
    }
#pragma unroll
    for (int v = 0; v < NCF; ++v) Lc[v] = div_add(true, TF(0), F[v], next_lane(F[v]), (TF)g.inv_dx[0]);
    const double dt = RHS ? 0.0 : *A.dtp;
    [[maybe_unused]] double new_rho = 0.0, new_a = 0.0, wcfl = 0.0;
    [[maybe_unused]] bool new_bad = false;
    if (core_out && act) {
        double nq[NCF];
#pragma unroll
        for (int v = 0; v < NCF; ++v) {
            const long long o = (long long)v * N + c;
            double Lv = (double)Lc[v];
            if (v == 3 && SRC) Lv = add_plain(Lv, A.P[(long long)PL<1>::SA * N + c]);
            if constexpr (RHS) {
                A.qo[o] = Lv;
            } else {
                double r = rk_combine(A.b, dt, Lv, A.qk[o]);
                if constexpr (UN) r = fma(A.a, A.qn[o], r);
                A.qo[o] = r;
                nq[v] = r;
            }
        }
        if constexpr (FUSE) {
            const CellCore<1> k = cell_core<1>(nq[0], &nq[1], nq[2], nq[3], ph);
            A.Pout[(long long)PL<1>::RHO * N + c] = nq[0];
            A.Pout[(long long)PL<1>::U * N + c] = k.u[0];
            A.Pout[(long long)PL<1>::PLQ * N + c] = k.pl;
            A.Pout[(long long)PL<1>::A * N + c] = nq[3];
            new_rho = nq[0];
            new_a = nq[3];
            new_bad = k.bad;
            if (A.cfl) wcfl = (fabs(k.u[0]) + k.cs) * g.inv_dx[0];
        }
    }
    const double n = A.P[(long long)PL<1>::N * N + c], nh = A.P[(long long)PL<1>::N * N + ch];
    const double in = n > 0.0 ? frcp(n) : 0.0, in_h = nh > 0.0 ? frcp(nh) : 0.0;
    [[maybe_unused]] double pl = 0.0, irhol = 0.0, ic = 0.0;
    if constexpr (SRC) {
        pl = A.P[(long long)PL<1>::PLQ * N + c];
        irhol = frcp(A.P[(long long)PL<1>::RHO * N + c] / (1.0 - A.P[(long long)PL<1>::A * N + c]));
        ic = frcp(sqrt(ph.gamma * (pl + ph.pi_inf) * irhol));
    }
    // the upwind stencil in the staged cells: first slot and signed stride; a face that takes cell values
    // reads its upwind cell five times
    int st = lane + (right ? 5 : 0), sd = right ? -1 : 1;
    if (!ok) st += 2 * sd, sd = 0;

    // ---- bins ----
    [[maybe_unused]] BinSums acc;
    acc.bad = nb;
    for (int ib = b0; ib < b1; ++ib) {
        const double r0 = bins.r0[ib], pg0 = bins.pg0[ib];
        auto put = [&](int slot, const double (&x)[NF], double inv) {
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                PT v;   // cells without bubbles take the bin's equilibrium values
                v.a = (TF)(inv > 0.0 ? x[2 * p] * inv : (p == 0 ? r0 : bins.pb0[ib]));
                v.b = (TF)(inv > 0.0 ? x[2 * p + 1] * inv : (p == 0 ? 0.0 : bins.mv0[ib]));
                s_q[p][slot] = v;
            }
        };
        put(lane + 3, raw, in);
        put(hslot, raw_h, in_h);
        double own[NF], own_un[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            own[f] = raw[f];
            own_un[f] = un[f];
        }
        if (ib + 1 < b1) load(ib + 1);
        wave_sync();
        TF W[NF], c2[NF];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            PT e[5];
#pragma unroll
            for (int o = 0; o < 5; ++o) e[o] = s_q[p][st + o * sd];
            W[2 * p] = weno5(e[0].a, e[1].a, e[2].a, e[3].a, e[4].a);
            W[2 * p + 1] = weno5(e[0].b, e[1].b, e[2].b, e[3].b, e[4].b);
            c2[2 * p] = e[2].a;
            c2[2 * p + 1] = e[2].b;
        }
        wave_sync();   // the next bin's staging writes follow these reads
        const bool cell = !ok || !(W[0] > TF(0));
        double L[NF], out[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const TF Fb = coef * (cell ? c2[f] : W[f]);
            L[f] = (double)div_add(true, TF(0), Fb, next_lane(Fb), (TF)g.inv_dx[0]);
        }
        if constexpr (SRC) {
            if (n > 0.0) {   // Keller--Miksis in FP64 from the FP64 state of the owned cell
                const double R = own[0] * in, V = own[1] * in;
                L[0] = fma(n, V, L[0]);
                if constexpr (TR) {
                    const double pb = own[2] * in, mv = own[3] * in;
                    double pdot, mdot;
                    contents_rates(ph, R, V, pb, mv, bins.mg[ib], pdot, mdot);
                    L[1] = fma(n, km_rddot_pb(ph, R, V, pb, pdot, pl, irhol, ic), L[1]);
                    L[2] = fma(n, pdot, L[2]);
                    L[3] = fma(n, mdot, L[3]);
                } else {
                    L[1] = fma(n, km_rddot_t<pw_of(CT)>(ph, R, V, r0, pg0, pl, irhol, ic, nullptr), L[1]);
                }
            }
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            out[f] = L[f];
            if constexpr (!RHS) out[f] = rk_combine(A.b, dt, L[f], own[f]);
            if constexpr (UN) out[f] = fma(A.a, own_un[f], out[f]);
        }
        if constexpr (FUSE) {
            if constexpr (TR) bin_add_tr(acc, ib, out[0], out[1], out[2], bins.w[ib], nb);
            else bin_add<pw_of(CT)>(acc, ib, out[0], out[1], bins.w[ib], pg0, r0, nb, ph, nullptr);
        }
        if (act) {
#pragma unroll
            for (int f = 0; f < NF; ++f) A.qo[(long long)(4 + f * nb + ib) * N + c] = out[f];
        }
    }
    if constexpr (FUSE) {
        // the primitive pass of the new state for the owned cell (same arithmetic as k_prim)
        if (act) {
            const CellBins m = cell_bins<CT>(new_rho, new_a, acc, ph, bins);
            A.Pout[(long long)PL<1>::N * N + c] = m.n;
            A.Pout[(long long)PL<1>::B * N + c] = m.B;
            A.Pout[(long long)PL<1>::SA * N + c] = m.Sa;
            const bool bad = new_bad || !(m.B == m.B) || !(m.n == m.n);
            if (new_a > 0.0 && acc.bad < nb) raise_error(A.sc, E_NEGR, c, acc.bad);
            else if (bad) raise_error(A.sc, E_NONFINITE, c, -1);
        }
        if (A.cfl) wmax_post(wcfl, A.sc);
    }
}

}  // namespace bub
