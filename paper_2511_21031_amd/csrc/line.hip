// Launches of the 1D stage kernel (line_kernel.hpp).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "line.hpp"
#include "line_kernel.hpp"

namespace bub {

namespace {

template <typename TF, int CT>
void launch(const bub_ctx *c, const StageArgs &A, hipStream_t s)
{
    const dim3 grid(8u * (unsigned)A.nblk_per_xcd), block(64);
    auto go = [&](auto mode, auto src, auto un) {
        hipLaunchKernelGGL((k_line<TF, CT, decltype(mode)::value, decltype(src)::value, decltype(un)::value>), grid,
                           block, 0, s, A, c->g, c->ph, c->bt);
    };
    const std::false_type no;
    const std::true_type yes;
    auto stage = [&](auto mode) {
        if (A.a != 0.0) A.sources ? go(mode, yes, yes) : go(mode, no, yes);
        else A.sources ? go(mode, yes, no) : go(mode, no, no);
    };
    const std::integral_constant<int, LM_RHS> rhs;
    if (A.rhs_mode) A.sources ? go(rhs, yes, no) : go(rhs, no, no);
    else if (A.Pout) stage(std::integral_constant<int, LM_FUSE>{});
    else stage(std::integral_constant<int, LM_RK>{});
}

template <int CT>
void launch_prec(const bub_ctx *c, const StageArgs &A, hipStream_t s)
{
    if (c->opts.precision == BUB_PREC_MIXED) launch<float, CT>(c, A, s);
    else launch<double, CT>(c, A, s);
}

}  // namespace

bool line_ok(const bub_ctx *c)
{
    if (c->ndim != 1) return false;
    return c->opts.contents == BUB_CONTENTS_TRANSFER || (c->ph.pw_c == 5 && c->ph.pw_d == 4);
}

// Bins are spread over waves until the chip has two waves per SIMD (2048), at least two bins to a wave: each
// wave repeats the tile's mixture face, which costs as much as seven bins.
int line_grouping(const bub_ctx *c, int *ntiles, int *groups)
{
    *ntiles = (int)((c->N + LINE_TX - 1) / LINE_TX);
    int ng = c->bin_groups;
    if (ng <= 0) {
        constexpr int target = 2048;
        ng = *ntiles >= target ? 1 : (target + *ntiles - 1) / *ntiles;
        const int cap = (c->nb + 1) / 2;
        if (ng > cap) ng = cap;
    }
    if (ng < 1) ng = 1;
    if (ng > c->nb) ng = c->nb;
    const int bpg = (c->nb + ng - 1) / ng;
    *groups = (c->nb + bpg - 1) / bpg;
    return bpg;
}

int launch_line(const bub_ctx *c, StageArgs A, hipStream_t s)
{
    A.bpg = line_grouping(c, &A.ntiles, &A.ngroups);
    A.ntile[0] = A.ntiles;
    A.ntile[1] = A.ntile[2] = 1;
    if (A.Pout && A.ngroups != 1) return BUB_EINVAL;   // the fused epilogue needs every bin of a cell
    A.nitems = A.ntiles * A.ngroups;
    A.nblk_per_xcd = (A.nitems + 7) / 8;
    if (c->opts.contents == BUB_CONTENTS_TRANSFER) launch_prec<CT_TRANSFER>(c, A, s);
    else launch_prec<CT_AIR>(c, A, s);
    return hipGetLastError() == hipSuccess ? BUB_OK : BUB_EHIP;
}

}  // namespace bub
