// Host rules of the stage launches: workgroups per tile (bin groups), and whether a stage carries the primitive pass
// of the state it writes.  Plain functions of sizes, so that the measurements they were fitted to can be held against
// them without a GPU.
#pragma once

namespace bub {

// What a stage of nw workgroups of `waves` wavefronts takes on 256 CUs when each does `bins` bins, in units of one
// bin of a workgroup alone (1.35 us in 2D): the mixture faces cost about ten bins, whatever the tiles; a CU's second
// workgroup (of four wavefronts) hides in the first one's waits for the most part, `second`, and k take k times
// `share`.  Fitted to 60 to 1056 tiles of 2D with 5 to 31 bins, and to 3D boxes of 26^3 to 80^3; FP32 fluxes (light)
// leave more room.
inline double stage_cost(long long nw, int waves, double bins, double second, double share)
{
    const long long k = (nw + 255) / 256 * ((waves + 3) / 4);
    return (10.0 + bins) * (k == 1 ? 1.0 : k == 2 ? second : share * (double)k);
}

inline double group_cost(long long nw, int waves, int bins, bool light)
{
    return light ? stage_cost(nw, waves, bins, 1.2, 0.43) : stage_cost(nw, waves, bins, 1.3, 0.6);
}

// Bin groups: small grids give each tile several workgroups (a range of bins each) where the cheaper bins outweigh
// the repeated mixture faces (group_cost).  About 1024 workgroups, the rule before, was too many: a viscous step of
// 600 x 150 x 5 with 3, 2, 1 groups 185, 164, 158 us, of 300 x 100 x 31 with 8, 4, 3 groups 190, 179, 170, of
// 150 x 80 x 31 with 16, 4, 3 groups 152, 135, 145.  In 1D a mixture face has one direction and a tile few halo cells,
// so a repeat costs less, and the nearest number to 1024 workgroups of four wavefronts is best (kappa = 5/3 FP64:
// 60000 x 31 with 2, 4, 5 groups 149, 138, 137 us, 100000 x 31 with 1, 3 237, 188, 250000 x 11 with 1, 2 193, 211;
// 1 % behind the best number on average, 11 % at worst, where group_cost is 6 and 53 %).
// forced: the caller's number (0: by this rule).
// Returns the bins per group; *groups receives the workgroups per tile.
inline int bins_per_group(int ndim, long long ntiles, int waves, int nb, bool light, int forced, int *groups)
{
    int ng = forced;
    if (ng <= 0 && ndim == 1) {
        const int cap = (nb + 1) / 2;
        const long long load = ntiles * waves, want = (4096 + load / 2) / load;
        ng = want < 1 ? 1 : want > cap ? cap : (int)want;
    } else if (ng <= 0) {
        ng = 1;
        double best = group_cost(ntiles, waves, nb, light);
        const int cap = (nb + 1) / 2;   // at least two bins per group
        for (int g = 2; g <= cap && ntiles * (g - 1) < 1024; ++g) {
            const double t = group_cost(ntiles * g, waves, (nb + g - 1) / g, light);
            if (t < best) best = t, ng = g;
        }
    }
    if (ng > nb) ng = nb;
    const int bpg = (nb + ng - 1) / ng;
    *groups = (nb + bpg - 1) / bpg;
    return bpg;
}

// Whether the registers of the balanced-tile kernel that carries the pass and the sources cost more than the pass:
// FP32 fluxes in 3D, where they take a wavefront a SIMD, and with workgroups of eight wavefronts a CU's second
// workgroup.  Apart over fused, us a step of 8 x 8 x 7 tiles: 64^3 x 1 185 / 192, x 5 243 / 262, x 31 750 / 841,
// 84^3 x 5 485 / 561, 112^3 x 11 1719 / 1852, 160^3 x 11 4983 / 5344 (40^3 x 11, the one size that loses, 162 / 150).
inline bool fused_starves(int ndim, bool light, bool sources) { return ndim == 3 && light && sources; }

// Whether a 2D or 3D grid of fewer than 2^19 cells is better off with one workgroup per tile that carries the
// primitive pass than with its bins in groups and a pass of its own (five bins and 10,000 cells a bin).  In 3D with
// FP32 fluxes the eight wavefronts of a tile alone on its CU hide less (1.6).  In 2D with FP32 fluxes a CU holds four
// fused workgroups but five plain ones, so between 1024 and 1280 tiles the fused launch alone has a second round
// (500^2 x 31, 1088 tiles: 466 us apart, 498 fused; 520 x 530 x 31, 1188 tiles: 485 and 529).
// Held against 188 measured steps the form it takes is at worst 8 % behind the other, 2 % or more behind it for
// 150 x 140 x 11 mixed and 280 x 250 x 21 FP64 only; without the last two terms it was up to 13 % behind.
inline bool fused_pays(int ndim, long long cells, long long ntiles, int waves, int nb, bool light, bool sources)
{
    if (ndim == 1 || fused_starves(ndim, light, sources)) return false;
    int groups;
    const int bpg = bins_per_group(ndim, ntiles, waves, nb, light, 0, &groups);
    const bool box = ndim == 3 && light;
    double fused = stage_cost(ntiles, waves, (light ? 1.1 : 1.2) * nb, box ? 1.6 : 1.3, box ? 0.51 : light ? 0.53 : 0.6);
    const long long load = ntiles * waves / 4;
    if (light && !box && load > 1024 && load <= 1280) fused *= 1.15;
    return fused < group_cost(ntiles * groups, waves, bpg, light) + 5.0 + (double)cells / 10000.0;
}

}  // namespace bub
