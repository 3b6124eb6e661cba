// The RK-stage kernel of 2D and 3D grids for polytropic air and transfer contents (gfx950).
//
// The tiling of stage_kernel.hpp with balanced tiles only ((TX+1) TY TZ <= BLOCK and so on: one face per
// thread and direction, one cell per thread).  In 2D it is bound by FP64 vector work, and by the power that
// takes (the clock falls as the vector units fill), so it is arranged for fewer instructions per bin:
//  * the mode (RK stage, with or without the primitive pass of its result, right-hand side), the sources
//    and the u^n term are template parameters, and air's power is straight-line code, so a bin's work is;
//  * a bin's R and Rdot are staged as one (R, Rdot) pair per cell: a face reads its stencil with five 16-byte
//    LDS reads and posts one pair of fluxes; in 2D a cell is staged once, in one plane of rows;
//  * a face's stencil address and signed stride and its flux coefficient stay in registers.
// 1024^2 x 31 bins FP64, RK stage with the primitive pass, 16 x 15 tile: 2.37e8 to 2.05e8 vector instructions,
// 0.718 to 0.633 ms (mixed 0.643 to 0.570); 256^3 x 21 FP64, 8 x 8 x 3: 11.8 to 10.6 ms.  Two bins between the
// same two barriers needed 151 registers instead of 126 (three waves per SIMD, not four): 0.664 ms.
#pragma once

#include "stage_kernel.hpp"

namespace bub {

enum TileMode : int { TM_RK = 0, TM_FUSE = 1, TM_RHS = 2 };

// 2D: cells and halos of a tile in one plane of rows (corners unused); 3D: a line array per direction.
template <int D, int TX, int TY, int TZ>
struct TileLds {
    using G = Geo<D, TX, TY, TZ>;
    static constexpr int ROW = TX + 6;
    static constexpr int CELLS = D == 2 ? ROW * (TY + 6) : G::L;
    static constexpr int NL = D == 2 ? 1 : 3;   // slots of an owned cell
    // slot of local cell (i, j, k) in the array that the faces of direction d read
    template <int d>
    __host__ __device__ static int slot(int i, int j, int k)
    {
        if constexpr (D == 2) return (j + 3) * ROW + i + 3;
        else return G::template lidx<d>(i, j, k);
    }
    template <int d>
    __host__ __device__ static constexpr int stride()
    {
        return D == 2 ? (d == 0 ? 1 : ROW) : G::LSTRIDE[d];
    }
};

template <int D, int TX, int TY, int TZ, int BLOCK, typename TF, int CT, int MODE, bool SRC, bool UN>
__global__ void __launch_bounds__(BLOCK) k_tile(StageArgs A, Grid g, Phys ph, Bins bins)
{
    using G = Geo<D, TX, TY, TZ>;
    using S = TileLds<D, TX, TY, TZ>;
    using PT = Pair<TF>;
    static_assert(G::FX <= BLOCK && G::FY <= BLOCK && G::FZ <= BLOCK && G::T <= BLOCK, "balanced tiles");
    constexpr bool TR = CT == CT_TRANSFER, FUSE = MODE == TM_FUSE, RHS = MODE == TM_RHS;
    constexpr int T = G::T, C = G::C, NCF = G::NCF, NP = TR ? 2 : 1, NF = 2 * NP;
    constexpr int CPT = (C + BLOCK - 1) / BLOCK, NL = S::NL;
    constexpr int QCELLS = S::CELLS + 1;        // and a slot that takes what no face reads
    // the bins' staged pairs and fluxes; the mixture fluxes use the same space before them
    constexpr int QBYTES = NP * QCELLS * (int)sizeof(PT), FBYTES = NP * D * BLOCK * (int)sizeof(PT);
    constexpr int CBYTES = NCF * D * BLOCK * (int)sizeof(TF);
    constexpr int BYTES = QBYTES + FBYTES > CBYTES ? QBYTES + FBYTES : CBYTES;
    __shared__ __align__(16) char s_mem[BYTES];
    PT *s_q = reinterpret_cast<PT *>(s_mem);             // [NP][QCELLS]
    PT *s_f = reinterpret_cast<PT *>(s_mem + QBYTES);    // [NP][D][BLOCK]
    TF *s_c = reinterpret_cast<TF *>(s_mem);             // [NCF][D][BLOCK]
    // the epilogue's bin sums of the slots that are done (an owned cell's are its thread's)
    __shared__ double s_tot[FUSE ? 5 : 1][FUSE ? T : 1];

    // XCD-aware order: consecutive items (and the bin groups of a tile) land on the same XCD
    const int item = (int)(blockIdx.x & 7) * A.nblk_per_xcd + (int)(blockIdx.x >> 3);
    if (item >= A.nitems) return;
    const int tile = item / A.ngroups, grp = item - tile * A.ngroups;
    const int b0 = grp * A.bpg, b1 = b0 + A.bpg < bins.nb ? b0 + A.bpg : bins.nb;
    const bool core_out = grp == 0;
    const int tx = tile % A.ntile[0], ty = (tile / A.ntile[0]) % A.ntile[1], tz = tile / (A.ntile[0] * A.ntile[1]);
    const int x0 = tx * TX, y0 = ty * G::TY, z0 = tz * G::TZ;
    const long long N = g.N;
    const int nb = bins.nb, tid = threadIdx.x;

    // ---- staged cells of this thread: global index, 1/n, LDS slots (slot 0 is the owned cell's) ----
    unsigned st_g[CPT];
    double st_in[CPT];
    int st_l[CPT][NL];
    bool some = false;   // a staged cell without bubbles
#pragma unroll
    for (int r = 0; r < CPT; ++r) {
        const int ci = tid + r * BLOCK, cc = ci < C ? ci : 0;
        int i, j, k;
        const int h = G::cdecode(cc, i, j, k);
        bool f = false;
        const int gx = map_coord(x0 + i, g.n[0], g.bc[0], f), gy = map_coord(y0 + j, g.n[1], g.bc[1], f);
        const int gz = D > 2 ? map_coord(z0 + k, g.n[2], g.bc[2], f) : 0;
        st_g[r] = (unsigned)gx + (unsigned)g.n[0] * ((unsigned)gy + (unsigned)g.n[1] * (unsigned)gz);
        const double n = A.P[(long long)PL<D>::N * N + st_g[r]];
        st_in[r] = n > 0.0 ? frcp(n) : 0.0;
        some = some || !(n > 0.0);
        const bool live = ci < C;
        if constexpr (D == 2) {
            st_l[r][0] = live ? S::template slot<0>(i, j, k) : S::CELLS;
        } else {
            st_l[r][0] = live && (h == 0 || h < 0) ? S::template slot<0>(i, j, k) : S::CELLS;
            st_l[r][NL > 1 ? 1 : 0] = live && (h == 1 || h < 0) ? S::template slot<1>(i, j, k) : S::CELLS;
            st_l[r][NL > 2 ? 2 : 0] = live && (h == 2 || h < 0) ? S::template slot<(D > 2 ? 2 : 0)>(i, j, k) : S::CELLS;
        }
    }
    const bool anyzero = __ballot(some) != 0ull;   // (per wave: each wave stages its own cells)

    double raw[NF][CPT];   // the next bin's values, loaded a bin ahead
    auto load = [&](int ib) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const double *p = A.qk + (long long)(D + 3 + f * nb + ib) * N;
#pragma unroll
            for (int r = 0; r < CPT; ++r) raw[f][r] = p[st_g[r]];
        }
    };

    // ---- mixture faces, one per thread and direction ----
    TF cf[D];
    int fa[D];   // stencil of the face's upwind side: LDS cell of its first entry | signed stride << 16
    auto core = [&](auto dtag) {
        constexpr int d = decltype(dtag)::value;
        constexpr int BX = G::template BX<d>(), BY = G::template BY<d>();
        constexpr int FD = d == 0 ? G::FX : (d == 1 ? G::FY : G::FZ);
        const int t = tid < FD ? tid : 0;
        const int fi = t % BX, fj = (t / BX) % BY, fk = t / (BX * BY);
        const int lc[3] = {fi, fj, fk}, org[3] = {x0, y0, z0};
        unsigned gi6[6];
        bool fl6[6], fo = false;
        int gt[3];
#pragma unroll
        for (int e = 0; e < 3; ++e) gt[e] = (e < D && e != d) ? map_coord(org[e] + lc[e], g.n[e], g.bc[e], fo) : 0;
#pragma unroll
        for (int o = 0; o < 6; ++o) {
            fl6[o] = false;
            int cc[3] = {gt[0], gt[1], gt[2]};
            cc[d] = map_coord(org[d] + lc[d] - 3 + o, g.n[d], g.bc[d], fl6[o]);
            gi6[o] = (unsigned)cc[0] + (unsigned)g.n[0] * ((unsigned)cc[1] + (unsigned)g.n[1] * (unsigned)cc[2]);
        }
        TF F[NCF];
        bool right, ok;
        core_face<D, d, TF>([&](int v, int o) { return (TF)A.P[(long long)v * N + gi6[o]]; }, fl6, ph, F, cf[d], right,
                            ok);
#pragma unroll
        for (int v = 0; v < NCF; ++v) s_c[(v * D + d) * BLOCK + tid] = F[v];
        int p[3] = {fi, fj, fk};
        p[d] -= 3;
        constexpr int st = S::template stride<d>();
        int at = S::template slot<d>(p[0], p[1], p[2]) + (right ? 5 * st : 0), sd = right ? -st : st;
        if (!ok) at += 2 * sd, sd = 0;   // a face that takes cell values reads its upwind cell five times
        fa[d] = (sd << 16) | at;
    };
    core(std::integral_constant<int, 0>{});
    core(std::integral_constant<int, 1>{});
    if constexpr (D > 2) core(std::integral_constant<int, (D > 2 ? 2 : 0)>{});
    load(b0);
    __syncthreads();

    // ---- owned cell: mixture update ----
    const int oc = tid < T ? tid : 0;
    const int li = oc % TX, lj = (oc / TX) % G::TY, lk = oc / (TX * G::TY);
    const bool act = tid < T && x0 + li < g.n[0] && y0 + lj < g.n[1] && (D < 3 || z0 + lk < g.n[2]);
    const long long c = (long long)(x0 + li) + (long long)g.n[0] * ((long long)(y0 + lj) + (long long)g.n[1] * (z0 + lk));
    int flo[3], fhi[3];
    flo[0] = li + (TX + 1) * (lj + G::TY * lk);
    fhi[0] = flo[0] + 1;
    flo[1] = li + TX * (lj + (G::TY + 1) * lk);
    fhi[1] = flo[1] + TX;
    flo[2] = li + TX * (lj + G::TY * lk);
    fhi[2] = flo[2] + TX * G::TY;
    const double dt = RHS ? 0.0 : *A.dtp;
    [[maybe_unused]] double new_rho = 0.0, new_a = 0.0, wcfl = 0.0;
    [[maybe_unused]] bool new_bad = false;
    [[maybe_unused]] double own_n = 0.0, own_pl = 0.0, own_irhol = 1.0, own_ic = 1.0;
    if (act) {
        if (core_out) {
            double nq[NCF];
#pragma unroll
            for (int v = 0; v < NCF; ++v) {
                TF Lc = TF(0);
#pragma unroll
                for (int d = 0; d < D; ++d)
                    Lc = div_add(d == 0, Lc, s_c[(v * D + d) * BLOCK + flo[d]], s_c[(v * D + d) * BLOCK + fhi[d]],
                                 (TF)g.inv_dx[d]);
                const long long o = (long long)v * N + c;
                double Lv = (double)Lc;
                if (v == D + 2 && SRC) Lv = add_plain(Lv, A.P[(long long)PL<D>::SA * N + c]);
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
                const CellCore<D> k = cell_core<D>(nq[0], &nq[1], nq[D + 1], nq[D + 2], ph);
                A.Pout[(long long)PL<D>::RHO * N + c] = nq[0];
#pragma unroll
                for (int d = 0; d < D; ++d) A.Pout[(long long)(PL<D>::U + d) * N + c] = k.u[d];
                A.Pout[(long long)PL<D>::PLQ * N + c] = k.pl;
                A.Pout[(long long)PL<D>::A * N + c] = nq[D + 2];
                new_rho = nq[0];
                new_a = nq[D + 2];
                new_bad = k.bad;
                if (A.cfl) {
#pragma unroll
                    for (int d = 0; d < D; ++d) wcfl = dmax(wcfl, (fabs(k.u[d]) + k.cs) * g.inv_dx[d]);
                }
            }
        }
        if constexpr (SRC) {
            own_n = A.P[(long long)PL<D>::N * N + c];
            own_pl = A.P[(long long)PL<D>::PLQ * N + c];
            own_irhol = frcp(A.P[(long long)PL<D>::RHO * N + c] / (1.0 - A.P[(long long)PL<D>::A * N + c]));
            own_ic = frcp(sqrt(ph.gamma * (own_pl + ph.pi_inf) * own_irhol));
        }
    }
    __syncthreads();   // the mixture fluxes' space is the bins' from here

    // ---- bins ----
    // The fused epilogue adds the bins up as the primitive pass of this grid does, whose A.slots threads a cell take
    // the bins slot, slot + slots, ..., so it walks them in that order (one slot: in plain order) and puts a slot's
    // sums by when it is done.
    [[maybe_unused]] BinSums acc;
    acc.bad = nb;
    [[maybe_unused]] int bad = nb, slot = 0;
    const int slots = FUSE ? A.slots : 1;
    int next = b0;
#pragma unroll 1
    for (int it = b0; it < b1; ++it) {
        const int ib = next;
        next = ib + slots;
        bool turn = false;   // the slot's last bin
        if constexpr (FUSE) {
            if (next >= b1) {
                turn = true;
                next = ++slot;
            }
        }
        const double r0 = bins.r0[ib], pg0 = bins.pg0[ib];
#pragma unroll
        for (int r = 0; r < CPT; ++r)
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                PT v;
                v.a = (TF)(raw[2 * p][r] * st_in[r]);
                v.b = (TF)(raw[2 * p + 1][r] * st_in[r]);
                if (anyzero) {   // cells without bubbles take the bin's equilibrium values
                    v.a = st_in[r] > 0.0 ? v.a : (TF)(p == 0 ? r0 : bins.pb0[ib]);
                    v.b = st_in[r] > 0.0 ? v.b : (TF)(p == 0 ? 0.0 : bins.mv0[ib]);
                }
#pragma unroll
                for (int l = 0; l < NL; ++l) s_q[p * QCELLS + st_l[r][l]] = v;
            }
        double own[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) own[f] = raw[f][0];
        __syncthreads();
        [[maybe_unused]] double un[NF];
        if constexpr (UN) {
#pragma unroll
            for (int f = 0; f < NF; ++f) un[f] = A.qn[(long long)(D + 3 + f * nb + ib) * N + st_g[0]];
        }
        if (it + 1 < b1) load(next);
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int at = fa[d] & 0xffff, sd = fa[d] >> 16;
            TF W[NF], c2[NF];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const PT *q = s_q + p * QCELLS + at;
                PT e[5];
#pragma unroll
                for (int o = 0; o < 5; ++o) e[o] = q[o * sd];
                W[2 * p] = weno5(e[0].a, e[1].a, e[2].a, e[3].a, e[4].a);
                W[2 * p + 1] = weno5(e[0].b, e[1].b, e[2].b, e[3].b, e[4].b);
                c2[2 * p] = e[2].a;
                c2[2 * p + 1] = e[2].b;
            }
            // (in FP64 five equal entries reconstruct to themselves exactly)
            bool cell = !(W[0] > TF(0));
            if constexpr (sizeof(TF) == 4) cell = cell || sd == 0;
#pragma unroll
            for (int p = 0; p < NP; ++p)
                s_f[(p * D + d) * BLOCK + tid] = PT{cf[d] * (cell ? c2[2 * p] : W[2 * p]),
                                                    cf[d] * (cell ? c2[2 * p + 1] : W[2 * p + 1])};
        }
        __syncthreads();
        if (act) {
            double L[NF], out[NF];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                TF La = TF(0), Lb = TF(0);
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    const PT *q = s_f + (p * D + d) * BLOCK;
                    const PT lo = q[flo[d]], hi = q[fhi[d]];
                    La = div_add(d == 0, La, lo.a, hi.a, (TF)g.inv_dx[d]);
                    Lb = div_add(d == 0, Lb, lo.b, hi.b, (TF)g.inv_dx[d]);
                }
                L[2 * p] = (double)La;
                L[2 * p + 1] = (double)Lb;
            }
            if constexpr (SRC) {
                // Keller--Miksis in FP64 from the FP64 state of the owned cell
                const double R = own[0] * st_in[0], V = own[1] * st_in[0];
                double Q[NF];
                Q[0] = V;
                if constexpr (TR) {
                    const double pb = own[2] * st_in[0], mv = own[3] * st_in[0];
                    contents_rates(ph, R, V, pb, mv, bins.mg[ib], Q[2], Q[3]);
                    Q[1] = km_rddot_pb(ph, R, V, pb, Q[2], own_pl, own_irhol, own_ic);
                } else {
                    Q[1] = km_rddot_t<pw_of(CT)>(ph, R, V, r0, pg0, own_pl, own_irhol, own_ic, nullptr);
                }
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    const double Ls = fma(own_n, Q[f], L[f]);
                    L[f] = !anyzero || own_n > 0.0 ? Ls : L[f];
                }
            }
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                out[f] = L[f];
                if constexpr (!RHS) out[f] = rk_combine(A.b, dt, L[f], own[f]);
                if constexpr (UN) out[f] = fma(A.a, un[f], out[f]);
            }
            if constexpr (FUSE) {
                if constexpr (TR) bin_add_tr(acc, ib, out[0], out[1], out[2], bins.w[ib], nb);
                else bin_add<pw_of(CT)>(acc, ib, out[0], out[1], bins.w[ib], pg0, r0, nb, ph, nullptr);
            }
#pragma unroll
            for (int f = 0; f < NF; ++f) A.qo[(long long)(D + 3 + f * nb + ib) * N + c] = out[f];
            if constexpr (FUSE) {
                if (turn && it + 1 < b1) {
                    double *v[5] = {&acc.s3, &acc.s2, &acc.s21, &acc.s32, &acc.sp};
#pragma unroll
                    for (int k = 0; k < 5; ++k) {
                        s_tot[k][oc] = slot > 1 ? s_tot[k][oc] + *v[k] : *v[k];
                        *v[k] = 0.0;
                    }
                    bad = acc.bad < bad ? acc.bad : bad;
                    acc.bad = nb;
                }
            }
        }
        // the next bin is staged only after every thread has passed the barrier above, and its fluxes are
        // posted only after the barrier that follows its staging
    }
    if constexpr (FUSE) {
        // the primitive pass of the new state for the owned cell (same arithmetic as k_prim)
        if (act) {
            if (slot > 1) {
                acc.s3 = s_tot[0][oc] + acc.s3;
                acc.s2 = s_tot[1][oc] + acc.s2;
                acc.s21 = s_tot[2][oc] + acc.s21;
                acc.s32 = s_tot[3][oc] + acc.s32;
                acc.sp = s_tot[4][oc] + acc.sp;
                acc.bad = acc.bad < bad ? acc.bad : bad;
            }
            const CellBins m = cell_bins<CT>(new_rho, new_a, acc, ph, bins);
            A.Pout[(long long)PL<D>::N * N + c] = m.n;
            A.Pout[(long long)PL<D>::B * N + c] = m.B;
            A.Pout[(long long)PL<D>::SA * N + c] = m.Sa;
            const bool bad = new_bad || !(m.B == m.B) || !(m.n == m.n);
            if (new_a > 0.0 && acc.bad < nb) raise_error(A.sc, E_NEGR, c, acc.bad);
            else if (bad) raise_error(A.sc, E_NONFINITE, c, -1);
        }
        if (A.cfl) wmax_post(wcfl, A.sc);
    }
}

}  // namespace bub
