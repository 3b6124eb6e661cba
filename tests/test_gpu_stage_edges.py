"""Right-hand sides and steps of the stage kernels at the sizes where their tilings can go wrong: just below, at and
just above one and two tiles, the smallest grids, cells without bubbles, every kind of end, both contents.

The oracle is the reference; the tolerance is that of the other right-hand-side tests (rounding of face fluxes,
1e-12 of the flux-divergence scale).  Steps of different shapes have to agree bit for bit.
"""
import dataclasses

import numpy as np
import pytest

import workloads as W
from tests.parity import flux_scale, perturb_bins, rhs_err

pytestmark = pytest.mark.gpu
RHS_TOL = 1e-12

LINE = [((3,), 1), ((62,), 0), ((63,), 1), ((64,), 2), ((126,), 0), ((127,), 2), ((190,), 1)]


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.fixture(scope="module")
def bub(torch):
    import paper_2511_21031_amd as B
    B.lib()
    return B


def _case(n, bc, contents, nb):
    case = W.random_smooth(len(n), n, 1e-4, nb, seed=31 + sum(n), bc=bc)
    if contents:
        case = dataclasses.replace(case, gas=dict(W.AIR_WITH_VAPOUR), contents=dict(W.AIR_VAPOUR))
    return case


def _state(orc, pb, case, bubbles_everywhere=True):
    if not bubbles_everywhere:   # a stretch of pure liquid that starts and ends inside tiles
        a = case.prim[case.ndim + 2]
        a[len(a) // 3:len(a) // 2] = 0.0
    return perturb_bins(orc.init_state(pb, case.prim), case.ndim, case.nb, seed=6)


def _check(torch, bub, orc, n, bc, contents, nb, everywhere):
    case = _case(n, bc, contents, nb)
    pb = orc.problem_from_case(case)
    q = _state(orc, pb, case, everywhere)
    ref = orc.rhs(pb, q)
    ctx = bub.context_from_case(case)
    qg = torch.from_numpy(q).cuda()
    err = rhs_err(ctx.rhs_stage(qg).cpu().numpy(), ref, flux_scale(orc, pb, q))
    assert err.max() < RHS_TOL, (n, bc, err)
    assert ctx.last_error()[0] == 0


@pytest.mark.parametrize("contents", [False, True])
@pytest.mark.parametrize("n,bc", LINE)
def test_line_tiles(torch, bub, orc, n, bc, contents):
    _check(torch, bub, orc, n, bc, contents, 5, everywhere=bc != 0)


def test_large_1d_grid_carries_its_primitives(torch, bub):
    """2^19 cells: the wave tiles' stages write the next state's primitives; bitwise the tiles of 255 cells."""
    case = W.random_smooth(1, ((1 << 19) + 5,), 1e-4, 3, seed=44)
    outs = []
    for tile in (3, 0):
        ctx = bub.context_from_case(case)
        ctx.tile = tile
        q = ctx.init_state(torch.from_numpy(case.prim).cuda())
        ctx.rk3_steps(q, ctx.new_work(), 2)
        assert ctx.last_error()[0] == 0
        outs.append(q)
    assert torch.equal(outs[0], outs[1])


PLANE = [((16, 15), 0), ((17, 16), 1), ((15, 14), 2), ((32, 30), 1), ((33, 31), 0), ((3, 3), 1), ((2, 40), 0), ((49, 7), 2)]
BOX = [((8, 8, 3), 0), ((9, 9, 4), 1), ((7, 7, 2), 2), ((16, 8, 7), 1), ((17, 10, 8), 0), ((3, 3, 3), 1)]


@pytest.mark.parametrize("contents", [False, True])
@pytest.mark.parametrize("n,bc", PLANE + BOX)
def test_balanced_tiles(torch, bub, orc, n, bc, contents):
    _check(torch, bub, orc, n, bc, contents, 5 if len(n) == 2 else 3, everywhere=bc != 0)


@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("n", [(19, 22, 9), (30, 14, 13), (8, 25, 7)])
def test_liquid_tiles_inside_the_grid(torch, bub, orc, bc, n):
    """Liquid right-hand side of grids that have tiles away from every end (staged without the ghost map) next to
    tiles that reach one, and of one that has none.  The bound is that of the other liquid right-hand sides: 1e-12
    of the flux-divergence scale."""
    rng = np.random.default_rng(5)
    N, dx = int(np.prod(n)), 1e-4
    prim = np.empty((5, N))
    prim[0] = 1000.0 + 5.0 * rng.standard_normal(N)
    prim[1:4] = 3.0 * rng.standard_normal((3, N))
    prim[4] = 1e5 + 3e4 * rng.standard_normal(N)
    alpha, rate = 0.01 * rng.random(N), 20.0 * rng.standard_normal(N)
    pb = orc.problem(3, n, (dx,) * 3, ((bc, bc),) * 3, 1)
    ctx = bub.Context(3, n, (dx,) * 3, ((bc, bc),) * 3, 1)
    ql = orc.el_liquid_state(pb, prim)
    ref = orc.el_rhs(pb, ql, alpha, rate)
    got = ctx.lagrangian_rhs(torch.from_numpy(ql).cuda(), torch.from_numpy(np.vstack([alpha, rate])).cuda()).cpu().numpy()
    scale = np.abs(ref).max(axis=1) + 1500.0 / dx * np.abs(ql).max(axis=1)
    scale[1:4] += np.abs(prim[4]).max() / dx
    err = np.abs(got - ref).max(axis=1) / scale
    assert err.max() < 1e-12, err


@pytest.mark.parametrize("contents", [False, True])
@pytest.mark.parametrize("n,nb", [(8191, 31), (8192, 31), (16383, 9), (16384, 17), (60, 17), (40, 7)])
def test_threads_per_cell_of_the_passes(torch, bub, orc, n, nb, contents):
    """Primitive passes with 8, 16 and 32 threads a cell, on both sides of the sizes where the number changes, bins
    that fill the threads and bins that do not: the sources of the right-hand side come from their sums."""
    _check(torch, bub, orc, (n,), 0, contents, nb, everywhere=True)


CARRY = [((211, 203), 11, False, False), ((211, 203), 11, True, False), ((127, 190), 5, False, True), ((331, 320), 31, False, False),
         ((41, 40, 39), 11, False, False), ((41, 40, 39), 11, True, False), ((64, 33, 30), 5, False, True)]


@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("n,nb,mixed,contents", CARRY)
def test_stages_of_small_grids_that_carry_their_primitives(torch, bub, n, nb, mixed, contents, split):
    """Grids whose primitive pass takes two to eight threads a cell: a stage that carries it adds the bins up in that
    pass's order.  Three steps in one call, bitwise those with the bins in two groups and a pass of their own."""
    case = _case(n, 1, contents, nb)
    outs = []
    for groups in (0, 2):
        ctx = bub.context_from_case(case, precision=bub.PREC_MIXED if mixed else bub.PREC_FP64,
                                    bubble_mode=bub.BUBBLES_SPLIT if split else bub.BUBBLES_UNSPLIT)
        ctx.set_bin_groups(groups)
        q = ctx.init_state(torch.from_numpy(case.prim).cuda())
        ctx.rk3_steps(q, ctx.new_work(), 3)
        assert ctx.last_error()[0] == 0
        outs.append(q)
    assert torch.equal(outs[0], outs[1])
