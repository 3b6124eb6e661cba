// Launches of the balanced-tile stage kernels (tile_kernel.hpp).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "tile.hpp"
#include "tile_kernel.hpp"

namespace bub {

namespace {

template <int D, int TX, int TY, int TZ, int BLOCK, typename TF, int CT>
void launch(const bub_ctx *c, const StageArgs &A, hipStream_t s)
{
    const dim3 grid(8u * (unsigned)A.nblk_per_xcd), block(BLOCK);
    auto go = [&](auto mode, auto src, auto un) {
        hipLaunchKernelGGL((k_tile<D, TX, TY, TZ, BLOCK, TF, CT, decltype(mode)::value, decltype(src)::value,
                                   decltype(un)::value>),
                           grid, block, 0, s, A, c->g, c->ph, c->bt);
    };
    const std::false_type no;
    const std::true_type yes;
    auto stage = [&](auto mode) {
        if (A.a != 0.0) A.sources ? go(mode, yes, yes) : go(mode, no, yes);
        else A.sources ? go(mode, yes, no) : go(mode, no, no);
    };
    const std::integral_constant<int, TM_RHS> rhs;
    if (A.rhs_mode) A.sources ? go(rhs, yes, no) : go(rhs, no, no);
    else if (A.Pout) stage(std::integral_constant<int, TM_FUSE>{});
    else stage(std::integral_constant<int, TM_RK>{});
}

template <int D, int TX, int TY, int TZ, int BLOCK, int CT>
int launch_prec(const bub_ctx *c, const StageArgs &A, hipStream_t s)
{
    if (c->opts.precision == BUB_PREC_MIXED) launch<D, TX, TY, TZ, BLOCK, float, CT>(c, A, s);
    else launch<D, TX, TY, TZ, BLOCK, double, CT>(c, A, s);
    return hipGetLastError() == hipSuccess ? BUB_OK : BUB_EHIP;
}

}  // namespace

bool tile_ok(const bub_ctx *c, int shape)
{
    if (c->opts.contents == BUB_CONTENTS_TRANSFER) return (c->ndim == 2 && shape == 5) || (c->ndim == 3 && shape == 3);
    if (c->ph.pw_c != 5 || c->ph.pw_d != 4) return false;
    return (c->ndim == 2 && (shape == 4 || shape == 5)) || (c->ndim == 3 && (shape == 3 || shape == 4));
}

int launch_tile(const bub_ctx *c, int shape, const StageArgs &A, hipStream_t s)
{
    const bool tr = c->opts.contents == BUB_CONTENTS_TRANSFER;
    if (c->ndim == 2) {
        if (tr) return launch_prec<2, 16, 15, 1, 256, CT_TRANSFER>(c, A, s);
        if (shape == 5) return launch_prec<2, 16, 15, 1, 256, CT_AIR>(c, A, s);
        return launch_prec<2, 32, 15, 1, 512, CT_AIR>(c, A, s);
    }
    if (tr) return launch_prec<3, 8, 8, 3, 256, CT_TRANSFER>(c, A, s);
    if (shape == 3) return launch_prec<3, 8, 8, 3, 256, CT_AIR>(c, A, s);
    return launch_prec<3, 8, 8, 7, 512, CT_AIR>(c, A, s);
}

}  // namespace bub
