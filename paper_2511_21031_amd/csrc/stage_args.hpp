// Arguments of a stage kernel launch.
#pragma once

#include "device_common.hpp"

namespace bub {

// RK combine: out = a * un + b * (uk + dt * L); a == 0 skips un.  RHS mode writes L.
struct StageArgs {
    const double *qk;   // u^(k): stencil source
    const double *qn;   // u^n (own cell only), may equal qk or be null when a == 0
    double *qo;         // output
    const double *P;    // primitive scratch of qk
    const double *dtp;  // device step (RK mode)
    double a, b;
    int rhs_mode;       // 1: write L instead of the combine
    int sources;        // 0: leave bubble source terms out (split mode flux part)
    int ntile[3];
    int nblk_per_xcd;
    int ntiles;
    int ngroups;        // workgroups per tile, each taking a contiguous range of bpg bins
    int bpg;            // bins per group (ngroups * bpg >= nb)
    int nitems;         // ntiles * ngroups
    // Fused primitive pass (RK mode, one workgroup per tile): the epilogue writes the primitives of
    // the state it produces into Pout (the layout of P; must not be P) and, with cfl set, posts that
    // state's wave-speed maximum.  Null Pout: the next stage needs a primitive pass of its own.
    double *Pout;
    int slots;          // threads per cell of the grid's primitive pass, whose order of bins the epilogue keeps
    int cfl;
    Scalars *sc;        // error word and wave-speed maxima of the context
};

}  // namespace bub
