// The one-wave-per-tile stage kernel of 1D grids: when it applies, its decomposition, its launch.
#pragma once

#include "ctx.hpp"
#include "stage_args.hpp"

namespace bub {

// Whether the context's stages can run it: 1D, polytropic air (its power is straight-line code) or transfer
// contents.
bool line_ok(const bub_ctx *c);

// Tiles and waves per tile (bin groups); returns the bins per group.
int line_grouping(const bub_ctx *c, int *ntiles, int *groups);

// One stage or right-hand side (the caller fills the state pointers and the combine of A).
int launch_line(const bub_ctx *c, StageArgs A, hipStream_t s);

}  // namespace bub
