// The balanced-tile stage kernels of 2D and 3D grids (tile_kernel.hpp): when they apply, their launch.
#pragma once

#include "ctx.hpp"
#include "stage_args.hpp"

namespace bub {

// Whether the stage shape (index into the per-dimension list) has this kernel for the context: the balanced
// shapes, with polytropic air (its power is straight-line code) or transfer contents.
bool tile_ok(const bub_ctx *c, int shape);

// One stage or right-hand side; the caller fills A with the decomposition of that shape.
int launch_tile(const bub_ctx *c, int shape, const StageArgs &A, hipStream_t s);

}  // namespace bub
