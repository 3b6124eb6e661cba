// The fused RK-stage kernel of the ensemble-averaged model (gfx950).
//
// One workgroup owns a tile of cells.  It computes the WENO5 + HLLC flux of the
// mixture on every face of the tile (all directions), then streams the bins
// one at a time through LDS: stage R = nR/n and Rdot = nRdot/n of the tile and
// its 3-cell halos, reconstruct the upwind side of every face (the passive
// HLLC flux of a bin variable needs only that side), difference the fluxes,
// add the Keller--Miksis source of the owned cell and write the RK combine.
// The next bin's global loads are in flight while the current bin is
// reconstructed.
//
// TF is the reconstruction precision: double (plain FP64) or float (the mixed
// form: reconstruction, Riemann solver and flux differences in FP32; the
// primitive pass, moments, Keller--Miksis and the RK combine stay FP64).
#pragma once

#include <type_traits>

#include "device_common.hpp"
#include "ee_kernels.hpp"
#include "stage_args.hpp"

namespace bub {

// Tile geometry.  Faces of direction d form the box (T + e_d).  The "cross"
// region holds the tile plus 3-cell halos along each active direction; bins
// are staged into one "line" array per direction d, of extent T_d + 6 along d
// and T_e across, so every face stencil is affine (constant stride).
template <int D, int TX_, int TY_, int TZ_>
struct Geo {
    static constexpr int TX = TX_, TY = (D > 1 ? TY_ : 1), TZ = (D > 2 ? TZ_ : 1);
    static constexpr int T = TX * TY * TZ;
    static constexpr int FX = (TX + 1) * TY * TZ;
    static constexpr int FY = D > 1 ? TX * (TY + 1) * TZ : 0;
    static constexpr int FZ = D > 2 ? TX * TY * (TZ + 1) : 0;
    static constexpr int F = FX + FY + FZ;
    static constexpr int OFF[3] = {0, FX, FX + FY};
    static constexpr int HX = 3 * TY * TZ, HY = D > 1 ? 3 * TX * TZ : 0, HZ = D > 2 ? 3 * TX * TY : 0;
    static constexpr int C = T + 2 * (HX + HY + HZ);
    static constexpr int NC = D + 5;   // reconstructed core primitives
    static constexpr int NCF = D + 3;  // core fluxes: mass, momentum, energy, alpha
    // line arrays
    static constexpr int LX = (TX + 6) * TY * TZ;
    static constexpr int LY = D > 1 ? TX * (TY + 6) * TZ : 0;
    static constexpr int LZ = D > 2 ? TX * TY * (TZ + 6) : 0;
    static constexpr int LOFF[3] = {0, LX, LX + LY};
    static constexpr int L = LX + LY + LZ;
    static constexpr int LSTRIDE[3] = {1, TX, TX * TY};

    template <int d>
    static constexpr int BX() { return TX + (d == 0); }
    template <int d>
    static constexpr int BY() { return TY + (d == 1); }

    // line-array index of local cell (i,j,k) in the array of direction d
    // (coordinate d may lie in [-3, T_d + 3))
    template <int d>
    __host__ __device__ static inline int lidx(int i, int j, int k)
    {
        if (d == 0) return LOFF[0] + (k * TY + j) * (TX + 6) + (i + 3);
        if (d == 1) return LOFF[1] + (k * (TY + 6) + (j + 3)) * TX + i;
        return LOFF[2] + ((k + 3) * TY + j) * TX + i;
    }

    // local coordinates of cross-region index ci; returns the halo direction
    // (0,1,2) or -1 for a core cell
    __host__ __device__ static inline int cdecode(int ci, int &i, int &j, int &k)
    {
        if (ci < T) {
            i = ci % TX;
            j = (ci / TX) % TY;
            k = ci / (TX * TY);
            return -1;
        }
        ci -= T;
        if (ci < 2 * HX) {
            int hi = ci >= HX;
            if (hi) ci -= HX;
            int r = ci / 3;
            i = (ci % 3) + (hi ? TX : -3);
            j = r % TY;
            k = r / TY;
            return 0;
        }
        ci -= 2 * HX;
        if (ci < 2 * HY) {
            int hi = ci >= HY;
            if (hi) ci -= HY;
            i = ci % TX;
            int r = ci / TX;
            j = (r % 3) + (hi ? TY : -3);
            k = r / 3;
            return 1;
        }
        ci -= 2 * HY;
        int hi = ci >= HZ;
        if (hi) ci -= HZ;
        i = ci % TX;
        j = (ci / TX) % TY;
        k = (ci / (TX * TY)) + (hi ? TZ : -3);
        return 2;
    }
};

// LDS needs of one tile: coef[F] and scr[SCR] of TF, flag[F] bytes; a bin's R and Rdot have a line array and a face
// array each.
template <int D, int TX_, int TY_, int TZ_, typename TF>
struct StageLds {
    using G = Geo<D, TX_, TY_, TZ_>;
    // line arrays of R and Rdot are LP apart, a multiple of 64 elements, so one paired LDS
    // access (64-element stride form) serves both
    static constexpr int LP = (G::L + 63) / 64 * 64;
    static constexpr int SCR = (G::NCF * G::F > 2 * LP + 2 * G::F) ? G::NCF * G::F : 2 * LP + 2 * G::F;
    static constexpr int BYTES = (G::F + SCR) * (int)sizeof(TF) + G::F;
};

// Two bin variables of a cell or a face, staged and read as one.
template <typename TF>
struct alignas(2 * sizeof(TF)) Pair {
    TF a, b;
};

// Mixture face between the cells f-1 and f of direction d: WENO5 of the primitives (ld(v, o): primitive v of
// cell f - 3 + o; fl6: that cell is a mirrored ghost, whose normal velocity changes sign), admissibility
// check, HLLC.  F_: the mixture fluxes; a bin variable's flux is coef times its value on the upwind side
// (right: the cell f's side), coef = n_K (u_K + fac); ok false: the face takes cell values.
template <int D, int d, typename TF, typename Ld>
__device__ __forceinline__ void core_face(Ld &&ld, const bool (&fl6)[6], const Phys &ph, TF (&F_)[D + 3], TF &coef,
                                          bool &right, bool &ok)
{
    constexpr int NC = D + 5;
    const TF pinf = (TF)ph.pi_inf, gpi = (TF)ph.gpi, igm1 = (TF)ph.inv_gm1, gam = (TF)ph.gamma;
    TF WL[NC], WR[NC], WcL[NC], WcR[NC];
#pragma unroll
    for (int v = 0; v < NC; ++v) {
        TF s[6];
#pragma unroll
        for (int o = 0; o < 6; ++o) s[o] = ld(v, o);
        if (v == 1 + d) {
#pragma unroll
            for (int o = 0; o < 6; ++o) s[o] = fl6[o] ? -s[o] : s[o];
        }
        weno5_pair(s, WL[v], WR[v]);
        WcL[v] = s[2];
        WcR[v] = s[3];
    }
    constexpr int iPL = D + 1, iA = D + 2, iN = D + 3, iB = D + 4;
    ok = WL[0] > TF(0) && WR[0] > TF(0) && WL[iA] >= TF(0) && WL[iA] < TF(1) && WR[iA] >= TF(0) &&
         WR[iA] < TF(1) && WL[iN] >= TF(0) && WR[iN] >= TF(0) && WL[iPL] + pinf > TF(0) &&
              WR[iPL] + pinf > TF(0);
    if (!ok) {
#pragma unroll
        for (int v = 0; v < NC; ++v) {
            WL[v] = WcL[v];
            WR[v] = WcR[v];
        }
    }
    // HLLC (Davis speeds, Toro contact speed, difference-form star flux)
    TF pK[2], EK[2], cK[2];
    const TF *Ws[2] = {WL, WR};
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const TF *Wk = Ws[s];
        TF a = Wk[iA], oma = TF(1) - a;
        TF u2 = TF(0);
#pragma unroll
        for (int e = 0; e < D; ++e) u2 += Wk[1 + e] * Wk[1 + e];
        pK[s] = oma * Wk[iPL] + a * Wk[iB];
        EK[s] = oma * (Wk[iPL] + gpi) * igm1 + TF(0.5) * Wk[0] * u2;
        cK[s] = tsqrt(gam * (Wk[iPL] + pinf) * oma * trcp(Wk[0]));
    }
    TF uL = WL[1 + d], uR = WR[1 + d];
    TF SL = dmin(uL - cK[0], uR - cK[1]);
    TF SR = dmax(uL + cK[0], uR + cK[1]);
    TF mL = WL[0] * (SL - uL), mR = WR[0] * (SR - uR);
    TF Ss = tdiv(pK[1] - pK[0] + uL * mL - uR * mR, mL - mR);
    int side, star;
    if (SL >= TF(0)) { side = 0; star = 0; }
    else if (Ss >= TF(0)) { side = 0; star = 1; }
    else if (SR > TF(0)) { side = 1; star = 1; }
    else { side = 1; star = 0; }
    const TF *WK = side ? WR : WL;
    TF SK = side ? SR : SL;
    TF un = WK[1 + d], rk = WK[0], pk = side ? pK[1] : pK[0], ek = side ? EK[1] : EK[0];
    TF fac = star ? tdiv(SK * (Ss - un), SK - Ss) : TF(0);
    F_[0] = rk * un + fac * rk;
#pragma unroll
    for (int e = 0; e < D; ++e)
        F_[1 + e] = rk * un * WK[1 + e] + (e == d ? pk : TF(0)) + fac * rk * (e == d ? SK : WK[1 + e]);
    F_[D + 1] = (ek + pk) * un + fac * (ek + pk + rk * Ss * (SK - un));
    F_[D + 2] = WK[iA] * un + fac * WK[iA];
    coef = WK[iN] * (un + fac);
    right = side;
}

// The work of one tile (every thread of the workgroup calls it).  FUSE: the epilogue carries the
// primitive pass of the state it writes (A.Pout, A.cfl).
template <int D, int TX_, int TY_, int TZ_, int BLOCK, typename TF, bool FUSE, int CT>
// Bins b0 <= ib < b1 are this workgroup's; core_out: it also writes the mixture variables
// (exactly one workgroup per tile does).
__device__ __forceinline__ void stage_tile(const StageArgs &A, const Grid &g, const Phys &ph, const Bins &bins,
                                           int tile, int b0, int b1, bool core_out, TF *__restrict__ s_coef,
                                           TF *__restrict__ s_scr, unsigned char *__restrict__ s_flag,
                                           double *__restrict__ s_out, const double *__restrict__ s_pp)
{
    using G = Geo<D, TX_, TY_, TZ_>;
    constexpr int T = G::T, F = G::F, C = G::C, NCF = G::NCF;
    constexpr int PW = pw_of(CT);
    constexpr int CPT = (C + BLOCK - 1) / BLOCK;  // cross cells staged per thread
    const int tx = tile % A.ntile[0];
    const int ty = (tile / A.ntile[0]) % A.ntile[1];
    const int tz = tile / (A.ntile[0] * A.ntile[1]);
    const int x0 = tx * G::TX, y0 = ty * G::TY, z0 = tz * G::TZ;
    const long long N = g.N;
    const int nb = bins.nb;
    const int tid = threadIdx.x;

    // ---- per-thread staging plan: global index, 1/n and line-array slots of its cross cells ----
    unsigned st_g[CPT];
    double st_in[CPT];
    int st_l[CPT][D];
#pragma unroll
    for (int r = 0; r < CPT; ++r) {
        int ci = tid + r * BLOCK;
        st_g[r] = 0;
        st_in[r] = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) st_l[r][d] = -1;
        if (ci < C) {
            int i, j, k;
            int h = G::cdecode(ci, i, j, k);
            bool f = false;
            int gx = map_coord(x0 + i, g.n[0], g.bc[0], f);
            int gy = D > 1 ? map_coord(y0 + j, g.n[1], g.bc[1], f) : 0;
            int gz = D > 2 ? map_coord(z0 + k, g.n[2], g.bc[2], f) : 0;
            unsigned gi = (unsigned)gx + (unsigned)g.n[0] * ((unsigned)gy + (unsigned)g.n[1] * (unsigned)gz);
            st_g[r] = gi;
            double n = A.P[PL<D>::N * N + gi];
            st_in[r] = n > 0.0 ? frcp(n) : 0.0;
            if (h == 0 || h < 0) st_l[r][0] = G::template lidx<0>(i, j, k);
            if (D > 1 && (h == 1 || h < 0)) st_l[r][D > 1 ? 1 : 0] = G::template lidx<(D > 1 ? 1 : 0)>(i, j, k);
            if (D > 2 && (h == 2 || h < 0)) st_l[r][D > 2 ? 2 : 0] = G::template lidx<(D > 2 ? 2 : 0)>(i, j, k);
        }
    }

    // ---- core faces: WENO5 of the mixture primitives, HLLC ----
    TF *s_cf = s_scr;  // [NCF][F]
    auto core_faces = [&](auto dtag) {
        constexpr int d = decltype(dtag)::value;
        constexpr int BX = G::template BX<d>(), BY = G::template BY<d>();
        constexpr int FD = (d == 0) ? G::FX : (d == 1 ? G::FY : G::FZ);
        for (int t = tid; t < FD; t += BLOCK) {
            int fi = t % BX, fj = (t / BX) % BY, fk = t / (BX * BY);
            int lc[3] = {fi, fj, fk};
            int org[3] = {x0, y0, z0};
            // global index of the 6 cells along d (positions f-3 .. f+2)
            unsigned gi6[6];
            bool fl6[6];
            {
                bool fo = false;
                int gt[3];
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    gt[e] = (e < D && e != d) ? map_coord(org[e] + lc[e], g.n[e], g.bc[e], fo) : 0;
#pragma unroll
                for (int o = 0; o < 6; ++o) {
                    bool f = false;
                    int gd = map_coord(org[d] + lc[d] - 3 + o, g.n[d], g.bc[d], f);
                    int cc[3] = {gt[0], gt[1], gt[2]};
                    cc[d] = gd;
                    gi6[o] = (unsigned)cc[0] + (unsigned)g.n[0] * ((unsigned)cc[1] + (unsigned)g.n[1] * (unsigned)cc[2]);
                    fl6[o] = f;
                }
            }
            TF F_[NCF], coef;
            bool right, ok;
            core_face<D, d, TF>([&](int v, int o) { return (TF)A.P[(long long)v * N + gi6[o]]; }, fl6, ph, F_, coef,
                                right, ok);
            const int slot = G::OFF[d] + t;
#pragma unroll
            for (int v = 0; v < NCF; ++v) s_cf[v * F + slot] = F_[v];
            s_coef[slot] = coef;
            s_flag[slot] = (unsigned char)((right ? 1 : 0) | (ok ? 0 : 2));
        }
    };
    core_faces(std::integral_constant<int, 0>{});
    if (D > 1) core_faces(std::integral_constant<int, (D > 1 ? 1 : 0)>{});
    if (D > 2) core_faces(std::integral_constant<int, (D > 2 ? 2 : 0)>{});

    // first bin's global loads go out while the core faces finish
    const int iNR = D + 3, iNV = D + 3 + nb;
    double pre_r[CPT], pre_v[CPT];
#pragma unroll
    for (int r = 0; r < CPT; ++r) {
        bool ok = tid + r * BLOCK < C;
        pre_r[r] = ok ? A.qk[(long long)(iNR + b0) * N + st_g[r]] : 0.0;
        pre_v[r] = ok ? A.qk[(long long)(iNV + b0) * N + st_g[r]] : 0.0;
    }
    __syncthreads();

    // ---- own cell: core divergence, sources, RK combine ----
    const bool own = tid < T;
    int ci_ = own ? tid : 0;
    int li = ci_ % G::TX, lj = (ci_ / G::TX) % G::TY, lk = ci_ / (G::TX * G::TY);
    const bool active = own && (x0 + li < g.n[0]) && (D < 2 || y0 + lj < g.n[1]) && (D < 3 || z0 + lk < g.n[2]);
    const long long gc = (long long)(x0 + li) + (long long)g.n[0] * ((long long)(y0 + lj) + (long long)g.n[1] * (z0 + lk));
    int flo[3], fhi[3];
    {
        // face slots of the own cell: lo face has the cell's coordinate, hi face +1 along d
        flo[0] = G::OFF[0] + li + (G::TX + 1) * (lj + G::TY * lk);
        fhi[0] = flo[0] + 1;
        flo[1] = D > 1 ? G::OFF[1] + li + G::TX * (lj + (G::TY + 1) * lk) : 0;
        fhi[1] = flo[1] + G::TX;
        flo[2] = D > 2 ? G::OFF[2] + li + G::TX * (lj + G::TY * lk) : 0;
        fhi[2] = flo[2] + G::TX * G::TY;
    }
    const double dt = A.rhs_mode ? 0.0 : *A.dtp;
    double own_n = 0.0, own_in = 0.0, own_pl = 0.0, own_irhol = 1.0, own_ic = 1.0;
    // fused primitive pass: the owned cell's new rho and alpha, admissibility, wave speed, bin sums
    constexpr bool fuse = FUSE;
    double new_rho = 0.0, new_a = 0.0, wcfl = 0.0;
    bool new_bad = false;
    BinSums acc;
    acc.bad = nb;
    if (active && core_out) {
        TF Lc[NCF];
#pragma unroll
        for (int v = 0; v < NCF; ++v) {
            TF acc = TF(0);
#pragma unroll
            for (int d = 0; d < D; ++d)
                acc = div_add(d == 0, acc, s_cf[v * F + flo[d]], s_cf[v * F + fhi[d]], (TF)g.inv_dx[d]);
            Lc[v] = acc;
        }
        double nq[NCF];
#pragma unroll
        for (int v = 0; v < NCF; ++v) {
            long long o = (long long)v * N + gc;
            double Lv = (double)Lc[v];
            if (v == D + 2 && A.sources) Lv = add_plain(Lv, A.P[PL<D>::SA * N + gc]);
            if (A.rhs_mode) A.qo[o] = Lv;
            else {
                double r = rk_combine(A.b, dt, Lv, A.qk[o]);
                if (A.a != 0.0) r = fma(A.a, A.qn[o], r);
                A.qo[o] = r;
                nq[v] = r;
            }
        }
        if constexpr (fuse) {
            const CellCore<D> k = cell_core<D>(nq[0], &nq[1], nq[D + 1], nq[D + 2], ph);
            A.Pout[PL<D>::RHO * N + gc] = nq[0];
#pragma unroll
            for (int d = 0; d < D; ++d) A.Pout[(PL<D>::U + d) * N + gc] = k.u[d];
            A.Pout[PL<D>::PLQ * N + gc] = k.pl;
            A.Pout[PL<D>::A * N + gc] = nq[D + 2];
            new_rho = nq[0];
            new_a = nq[D + 2];
            new_bad = k.bad;
            if (A.cfl) {
#pragma unroll
                for (int d = 0; d < D; ++d) wcfl = dmax(wcfl, (fabs(k.u[d]) + k.cs) * g.inv_dx[d]);
            }
        }
    }
    if (active) {
        own_n = A.P[PL<D>::N * N + gc];
        own_in = own_n > 0.0 ? frcp(own_n) : 0.0;
        own_pl = A.P[PL<D>::PLQ * N + gc];
        double a = A.P[PL<D>::A * N + gc];
        double rhol = A.P[PL<D>::RHO * N + gc] / (1.0 - a);
        own_irhol = frcp(rhol);
        own_ic = frcp(sqrt(ph.gamma * (own_pl + ph.pi_inf) * own_irhol));
    }
    __syncthreads();  // s_cf is reused below

    // ---- bins, one at a time: stage -> faces -> cells; next bin's loads overlap the faces ----
    // The owned cell is slot 0 of this thread's staging plan (cross index tid < T), so its own
    // bin values of u^(k) arrive with the staging loads; its u^n values are fetched one bin ahead too.
    const bool own_un = active && !A.rhs_mode && A.a != 0.0;
    double pre_nr = own_un ? A.qn[(long long)(iNR + b0) * N + gc] : 0.0;
    double pre_nv = own_un ? A.qn[(long long)(iNV + b0) * N + gc] : 0.0;
    constexpr int LP = StageLds<D, TX_, TY_, TZ_, TF>::LP;
    TF *s_R = s_scr, *s_V = s_scr + LP, *s_fR = s_scr + 2 * LP, *s_fV = s_scr + 2 * LP + F;
    // In 3D the owned cell's two results of a bin wait in this thread's own s_out slots and go
    // to HBM one bin late, ahead of the next bin's loads, so that the wait for those loads at
    // the next staging does not also wait for stores issued just before it (measured: 1-3 %
    // faster in 3D; in 2D the extra registers cost a wave per SIMD, so it stores at once).
    constexpr bool DEFER = D == 3;
    for (int ib = b0; ib < b1; ++ib) {
        const double r0 = bins.r0[ib], pg0 = bins.pg0[ib];
        const double own_r = pre_r[0], own_v = pre_v[0], own_nr = pre_nr, own_nv = pre_nv;
#pragma unroll
        for (int r = 0; r < CPT; ++r) {
            if (tid + r * BLOCK < C) {
                double in = st_in[r];
                TF Rv = (TF)(in > 0.0 ? pre_r[r] * in : r0);
                TF Vv = (TF)(in > 0.0 ? pre_v[r] * in : 0.0);
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    int l = st_l[r][d];
                    if (l >= 0) {
                        s_R[l] = Rv;
                        s_V[l] = Vv;
                    }
                }
            }
        }
        __syncthreads();
        if (DEFER && active && ib > b0) {
            A.qo[(long long)(iNR + ib - 1) * N + gc] = s_out[tid];
            A.qo[(long long)(iNV + ib - 1) * N + gc] = s_out[BLOCK + tid];
        }
        if (ib + 1 < b1) {
            if (own_un) {
                pre_nr = A.qn[(long long)(iNR + ib + 1) * N + gc];
                pre_nv = A.qn[(long long)(iNV + ib + 1) * N + gc];
            }
#pragma unroll
            for (int r = 0; r < CPT; ++r) {
                bool ok = tid + r * BLOCK < C;
                pre_r[r] = ok ? A.qk[(long long)(iNR + ib + 1) * N + st_g[r]] : 0.0;
                pre_v[r] = ok ? A.qk[(long long)(iNV + ib + 1) * N + st_g[r]] : 0.0;
            }
        }
        auto bin_faces = [&](auto dtag) {
            constexpr int d = decltype(dtag)::value;
            constexpr int BX = G::template BX<d>(), BY = G::template BY<d>();
            constexpr int FD = (d == 0) ? G::FX : (d == 1 ? G::FY : G::FZ);
            constexpr int S = G::LSTRIDE[d];
            for (int t = tid; t < FD; t += BLOCK) {
                int fi = t % BX, fj = (t / BX) % BY, fk = t / (BX * BY);
                const int slot = G::OFF[d] + t;
                unsigned fl = s_flag[slot];
                bool right = fl & 1;
                // cells f-3 .. f+2 along d start at the face's own coordinates in the line array
                int p[3] = {fi, fj, fk};
                p[d] -= 3;
                const int base = G::template lidx<d>(p[0], p[1], p[2]);
                // upwind side only: L reads cells f-3..f+1, R the mirrored f+2..f-2 (a signed stride)
                const int st = right ? base + 5 * S : base;
                const int sd = right ? -S : S;
                TF rr[5], vv[5];
#pragma unroll
                for (int o = 0; o < 5; ++o) {
                    rr[o] = s_R[st + o * sd];
                    vv[o] = s_V[st + o * sd];
                }
                TF RK, VK;
                if (fl & 2) {
                    RK = rr[2];
                    VK = vv[2];
                } else {
                    RK = weno5(rr[0], rr[1], rr[2], rr[3], rr[4]);
                    VK = weno5(vv[0], vv[1], vv[2], vv[3], vv[4]);
                    if (!(RK > TF(0))) {
                        RK = rr[2];
                        VK = vv[2];
                    }
                }
                TF cf = s_coef[slot];
                s_fR[slot] = cf * RK;
                s_fV[slot] = cf * VK;
            }
        };
        bin_faces(std::integral_constant<int, 0>{});
        if (D > 1) bin_faces(std::integral_constant<int, (D > 1 ? 1 : 0)>{});
        if (D > 2) bin_faces(std::integral_constant<int, (D > 2 ? 2 : 0)>{});
        __syncthreads();
        if (active) {
            TF LRf = TF(0), LVf = TF(0);
#pragma unroll
            for (int d = 0; d < D; ++d) {
                LRf = div_add(d == 0, LRf, s_fR[flo[d]], s_fR[fhi[d]], (TF)g.inv_dx[d]);
                LVf = div_add(d == 0, LVf, s_fV[flo[d]], s_fV[fhi[d]], (TF)g.inv_dx[d]);
            }
            double LR = (double)LRf, LV = (double)LVf;
            const double xr0 = own_r, xv0 = own_v;   // u^(k) of bin ib at the owned cell
            if (A.sources && own_n > 0.0) {
                // Keller--Miksis in FP64 from the FP64 state of the owned cell
                double own_R = xr0 * own_in, own_V = xv0 * own_in;
                LR = fma(own_n, own_V, LR);
                LV = fma(own_n, km_rddot_t<PW>(ph, own_R, own_V, r0, pg0, own_pl, own_irhol, own_ic, s_pp), LV);
            }
            double xr = LR, xv = LV;
            if (!A.rhs_mode) {
                xr = rk_combine(A.b, dt, LR, xr0);
                xv = rk_combine(A.b, dt, LV, xv0);
                if (A.a != 0.0) {
                    xr = fma(A.a, own_nr, xr);   // u^n of bin ib at the owned cell
                    xv = fma(A.a, own_nv, xv);
                }
            }
            if constexpr (fuse) {
                bin_add<PW>(acc, ib, xr, xv, bins.w[ib], pg0, r0, nb, ph, s_pp);
            }
            if constexpr (DEFER) {
                s_out[tid] = xr;
                s_out[BLOCK + tid] = xv;
            } else {
                A.qo[(long long)(iNR + ib) * N + gc] = xr;
                A.qo[(long long)(iNV + ib) * N + gc] = xv;
            }
        }
        // the next bin's staging writes s_R/s_V only after every thread passed the barrier above,
        // and s_fR/s_fV are rewritten only after the next staging barrier.
    }
    if (DEFER && active && b1 > b0) {
        A.qo[(long long)(iNR + b1 - 1) * N + gc] = s_out[tid];
        A.qo[(long long)(iNV + b1 - 1) * N + gc] = s_out[BLOCK + tid];
    }
    if constexpr (fuse) {
        // the primitive pass of the new state for the owned cell (same arithmetic as k_prim)
        if (active) {
            const CellBins m = cell_bins<CT>(new_rho, new_a, acc, ph, bins);
            A.Pout[PL<D>::N * N + gc] = m.n;
            A.Pout[PL<D>::B * N + gc] = m.B;
            A.Pout[PL<D>::SA * N + gc] = m.Sa;
            const bool bad = new_bad || !(m.B == m.B) || !(m.n == m.n);
            if (new_a > 0.0 && acc.bad < nb) raise_error(A.sc, E_NEGR, gc, acc.bad);
            else if (bad) raise_error(A.sc, E_NONFINITE, gc, -1);
        }
        if (A.cfl) wmax_post(wcfl, A.sc);
    }
    __syncthreads();  // a following tile on this workgroup may reuse the LDS at once
}

// The LDS arrays of one stage workgroup, declared in the kernel that uses them.
#define BUB_STAGE_SHARED(D, TX_, TY_, TZ_, BLOCK, TF)                                   \
    __shared__ TF s_coef[Geo<D, TX_, TY_, TZ_>::F];                                       \
    __shared__ TF s_scr[StageLds<D, TX_, TY_, TZ_, TF>::SCR];                             \
    __shared__ unsigned char s_flag[Geo<D, TX_, TY_, TZ_>::F];                            \
    __shared__ double s_out[D == 3 ? 2 * BLOCK : 1]; /* 3D: results stored one bin late */ \
    __shared__ double s_pp[PPOW_N];                  /* constants of the polytropic power */ \
    if (threadIdx.x < PPOW_N) s_pp[threadIdx.x] = PPOW_TABLE[threadIdx.x]; /* read after the tile's barriers */

// Work item `item` (a tile, or one bin group of a tile) of a stage.
template <int D, int TX_, int TY_, int TZ_, int BLOCK, typename TF, bool FUSE, int CT>
__device__ __forceinline__ void stage_item(const StageArgs &A, const Grid &g, const Phys &ph, const Bins &bins,
                                           int item, TF *__restrict__ s_coef, TF *__restrict__ s_scr,
                                           unsigned char *__restrict__ s_flag, double *__restrict__ s_out,
                                           const double *__restrict__ s_pp)
{
    const int tile = item / A.ngroups, grp = item - tile * A.ngroups;
    const int b0 = grp * A.bpg, b1 = b0 + A.bpg < bins.nb ? b0 + A.bpg : bins.nb;
    stage_tile<D, TX_, TY_, TZ_, BLOCK, TF, FUSE, CT>(A, g, ph, bins, tile, b0, b1, grp == 0, s_coef, s_scr, s_flag,
                                                      s_out, s_pp);
}

// Wavefronts a SIMD that the register allocation of a stage kernel keeps room for.  The unfused 1D and 2D kernels of
// the mixed form with the fifth-root power fit 96 VGPRs without spilling and run five (2D: 4 % faster stage than at
// four); the FP64 ones, the fused ones and those of the other contents would spill.  The 3D kernels of the mixed form
// sit at the edge of three wavefronts (168 VGPRs), those of 512 threads of four (128), where a CU's second workgroup
// hangs on it; none spills.  Microseconds a step, left to itself and held: general power 112^3 x 11 3068 and 2466,
// 8 x 8 x 7 tiles of kappa = 5/3 84^3 x 5 719 and 561.
template <int D, int BLOCK, typename TF, bool FUSE, int CT>
__host__ __device__ constexpr int stage_waves()
{
    if (sizeof(TF) != 4) return 1;
    if (D == 3) return BLOCK == 512 ? 4 : 3;
    return !FUSE && CT == CT_FIFTHS ? 5 : 1;
}

template <int D, int TX_, int TY_, int TZ_, int BLOCK, typename TF, bool FUSE, int CT>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(stage_waves<D, BLOCK, TF, FUSE, CT>()))) k_stage(StageArgs A, Grid g, Phys ph, Bins bins)
{
    BUB_STAGE_SHARED(D, TX_, TY_, TZ_, BLOCK, TF)
    // XCD-aware order: consecutive items land on the same XCD (blocks are dealt round-robin), and
    // the bin groups of a tile are consecutive items, so they share that XCD's L2.
    const int b = blockIdx.x;
    const int item = (b & 7) * A.nblk_per_xcd + (b >> 3);
    if (item >= A.nitems) return;
    stage_item<D, TX_, TY_, TZ_, BLOCK, TF, FUSE, CT>(A, g, ph, bins, item, s_coef, s_scr, s_flag, s_out, s_pp);
}

}  // namespace bub
