"""GPU parity of the Strang-split bubble sub-stepper (Sec. 3) against the CPU oracle.

Adaptive accept/reject decisions are taken in floating point on both sides, so
a (cell, bin) whose error estimate sits at the tolerance may take a different
number of sub-steps on the two sides.  Items with equal sub-step counts must
agree to 1e-8 relative; the others to 10 * rtol; the count of diverging items
is printed.
"""
import numpy as np
import pytest

import workloads as W
from tests.parity import flux_scale, oracle_split_step, perturb_bins, rel_err, rhs_err

pytestmark = pytest.mark.gpu
RTOL = 1e-4


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


def _gpu(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _compare_advance(q_gpu, q_ref, ns_gpu, ns_ref, ndim, nb):
    """Per-item comparison of (nR, nRdot) after a bubble half-step; returns the diverging fraction."""
    i0 = ndim + 3
    same = ns_gpu == ns_ref                         # [nb][N]
    for blk in (slice(i0, i0 + nb), slice(i0 + nb, i0 + 2 * nb)):
        g, r = q_gpu[blk], q_ref[blk]
        rel = np.abs(g - r) / np.abs(r).max(axis=1, keepdims=True)
        assert rel[same].max(initial=0.0) < 1e-8, rel[same].max()
        assert rel[~same].max(initial=0.0) < 10 * RTOL
    # alpha: rescaled by the cell's M3 ratio
    ra = np.abs(q_gpu[ndim + 2] - q_ref[ndim + 2]) / np.abs(q_ref[ndim + 2]).max()
    cell_same = same.all(axis=0)
    assert ra[cell_same].max(initial=0.0) < 1e-8
    assert ra.max() < 10 * RTOL
    return 1.0 - same.mean()


def _split_trajectory(torch, bub, orc, case, steps):
    """Both sides step `case` in split mode with the oracle's steps; returns the GPU and oracle states and
    the number of (cell, bin, half-step) sub-step counts that differed between the two sides."""
    pb = orc.problem_from_case(case, split=1)
    q_ref = orc.init_state(pb, case.prim)
    ctx = bub.context_from_case(case, bubble_mode=bub.BUBBLES_SPLIT)
    q = ctx.init_state(_gpu(torch, case.prim))
    work = ctx.new_work()
    ns = torch.zeros((2, case.nb, case.ncells), dtype=torch.int32, device="cuda")
    ctx.substep_counts(ns)
    diverged = 0
    for _ in range(steps):
        dt = orc.cfl_dt(pb, q_ref)
        ns_ref = oracle_split_step(orc, pb, q_ref, dt)
        ctx.rk3_step(q, work, dt)
        diverged += int((ns.cpu().numpy() != ns_ref).sum())
    ctx.substep_counts(None)
    assert ctx.last_error()[0] == 0
    return pb, q.cpu().numpy(), q_ref, diverged


def _judge_split(orc, pb, got, q_ref, diverged, tag):
    """1e-8 on every field when no sub-step decision differed anywhere in the run, else 10 rtol."""
    err = rel_err(got, q_ref)
    mg, mr = orc.moments(pb, got), orc.moments(pb, q_ref)
    e_p, e_a = rel_err(mg[6], mr[6]), rel_err(mg[1], mr[1])
    print(f"{tag}: diverging sub-step counts {diverged}; max field err {err.max():.3e}, p {e_p:.3e}, "
          f"alpha {e_a:.3e}")
    if diverged == 0:
        assert err.max() < 1e-8
    else:
        assert err.max() < 10 * RTOL
        assert e_p < 1e-6 and e_a < 10 * RTOL


@pytest.mark.parametrize("amp", [3.0, 10.0])
def test_bubble_advance_matches_oracle(torch, bub, orc, amp):
    case = W.c3(n=12, nb=5, amp_atm=amp, width=4e-4)
    pb = orc.problem_from_case(case, split=1)
    q = perturb_bins(orc.init_state(pb, case.prim), 3, 5, seed=8, amp_r=0.02, vel=0.05)
    tau = 0.5 * orc.cfl_dt(pb, q)
    q_ref = q.copy()
    ns_ref = orc.bubble_advance(pb, q_ref, tau)
    ctx = bub.context_from_case(case, bubble_mode=bub.BUBBLES_SPLIT)
    qg = _gpu(torch, q)
    ns = torch.zeros((5, case.ncells), dtype=torch.int32, device="cuda")
    ctx.bubble_advance(qg, tau, ns)
    assert ctx.last_error()[0] == 0
    frac = _compare_advance(qg.cpu().numpy(), q_ref, ns.cpu().numpy(), ns_ref, 3, 5)
    print(f"amp {amp} atm: sub-steps per item {ns_ref.mean():.2f} (max {ns_ref.max()}), diverging items {frac:.2e}")
    assert ns_ref.max() > 1


def test_split_trajectory_3d_pulse(torch, bub, orc):
    """A 10 atm spherical pulse that collapses bubbles: unsplit RK3 fails, split mode advances."""
    case = W.c3(n=24, nb=5, width=6e-4)
    pb, got, q_ref, diverged = _split_trajectory(torch, bub, orc, case, 8)
    _judge_split(orc, pb, got, q_ref, diverged, "split 3D pulse 24^3 nb 5, 8 steps")


def test_full_size_3d_sampled(torch, bub, orc):
    """256^3 with 21 bins: flux-part RHS and bubble half-step at sampled cells, plus one full split step."""
    case = W.c3()
    pb = orc.problem_from_case(case)
    qh = perturb_bins(orc.init_state(pb, case.prim), 3, 21, seed=9, amp_r=0.02, vel=0.05)
    n = 256
    rng = np.random.default_rng(6)
    pick = list(rng.integers(0, n ** 3, 120))
    for x, y, z in [(0, 0, 0), (n - 1, n - 1, n - 1), (128, 128, 128), (7, 8, 4), (8, 7, 3), (255, 0, 129)]:
        pick.append((z * n + y) * n + x)
    cells = np.array(pick, dtype=np.int64)
    # (a) RHS of the unsplit context at the sampled cells
    ctx = bub.context_from_case(case)
    qg = _gpu(torch, qh)
    rhs = ctx.rhs_stage(qg)
    ref = orc.rhs_cells(pb, qh, cells)
    got = rhs[:, torch.from_numpy(cells).cuda()].cpu().numpy()
    assert rhs_err(got, ref.T, flux_scale(orc, pb, qh)).max() < 1e-12
    del rhs
    # (b) bubble half-step: cells are independent, so the oracle advances just the sampled cells
    tau = 0.5 * orc.cfl_dt(pb, qh)
    sub = np.ascontiguousarray(qh[:, cells])
    # a K x 1 x 1 grid with the 3D slot layout holds the sampled cells (periodic, never coupled here)
    pb1 = orc.problem(3, (len(cells), 1, 1), (1e-4, 1e-4, 1e-4), ((0, 0), (0, 0), (0, 0)), 21, sigma_ln=0.3,
                      split=1)
    ns_ref = orc.bubble_advance(pb1, sub, tau)
    ctxs = bub.context_from_case(case, bubble_mode=bub.BUBBLES_SPLIT)
    ns = torch.zeros((21, case.ncells), dtype=torch.int32, device="cuda")
    ctxs.bubble_advance(qg, tau, ns)
    assert ctxs.last_error()[0] == 0
    ci = torch.from_numpy(cells).cuda()
    frac = _compare_advance(qg[:, ci].cpu().numpy(), sub, ns[:, ci].cpu().numpy(), ns_ref, 3, 21)
    print("256^3 sampled bubble half-step: diverging items", frac)
    # (c) one full split step of the whole grid: no device error; mass and energy are conserved
    #     by the flux part in the reflective box and left unchanged by the bubble part
    work = ctxs.new_work()
    tot0 = torch.stack([qg[0].sum(), qg[4].sum()])
    ctxs.rk3_step(qg, work)
    assert ctxs.last_error()[0] == 0
    tot = torch.stack([qg[0].sum(), qg[4].sum()])
    scale = torch.stack([qg[0].abs().sum(), qg[4].abs().sum()])
    assert ((tot - tot0).abs() / scale).max().item() < 1e-12


def _serving_requests():
    """A 1D and a 2D request of the serving stream, at test size (reflective box, Gaussian pulse)."""
    one = W.c5_stream(count=4, seed=3, scale=0.05)[0]
    two = [r for r in W.c5_stream(count=24, seed=7, scale=0.05) if r.ndim == 2][0]
    return {"1d": W.request_case(one), "2d": W.request_case(two)}


@pytest.mark.parametrize("kind", ["1d", "2d"])
def test_split_trajectory_1d_2d_requests(torch, bub, orc, kind):
    case = _serving_requests()[kind]
    pb, got, q_ref, diverged = _split_trajectory(torch, bub, orc, case, 6)
    _judge_split(orc, pb, got, q_ref, diverged, f"split {kind} {case.n} nb {case.nb}, 6 steps")


@pytest.mark.parametrize("contents", [False, True])
@pytest.mark.parametrize("n", [(130,), (300, 260), (520, 515), (84, 84, 84)])
def test_steps_in_one_call_are_single_steps(n, contents):
    """Split mode: a call of several steps takes the next step's primitives and wave speeds from the closing bubble
    half-step, single steps from the primitive pass: the same bits, with one to eight threads per cell."""
    import dataclasses

    import torch
    import paper_2511_21031_amd as bub
    case = W.random_smooth(len(n), n, 1e-4, 3, seed=51, bc=1, amp_atm=2.0)
    if contents:
        case = dataclasses.replace(case, gas=dict(W.AIR_WITH_VAPOUR), contents=dict(W.AIR_VAPOUR))
    outs = []
    for calls in ((3,), (1, 1, 1)):
        ctx = bub.context_from_case(case, bubble_mode=bub.BUBBLES_SPLIT)
        q = ctx.init_state(torch.from_numpy(case.prim).cuda())
        work = ctx.new_work()
        for k in calls:
            ctx.rk3_steps(q, work, k)
        assert ctx.last_error()[0] == 0
        outs.append(q)
    assert torch.equal(outs[0], outs[1])


@pytest.mark.gpu
@pytest.mark.parametrize("n,nb", [(8191, 31), (8192, 21), (16383, 9), (60, 17)])
def test_half_steps_of_many_threads_per_cell(orc, n, nb):
    """Half-steps with 16 and 32 threads a cell, on both sides of the sizes where the number changes, against the
    oracle (the bound of the other half-steps), and in a call of several steps against single steps (the same bits)."""
    import torch
    import paper_2511_21031_amd as bub
    case = W.random_smooth(1, (n,), 1e-4, nb, seed=52, bc=1, amp_atm=1.0)
    pb = orc.problem_from_case(case, split=1)
    q0 = perturb_bins(orc.init_state(pb, case.prim), 1, nb, seed=8, amp_r=0.02, vel=0.05)
    tau = 0.5 * orc.cfl_dt(pb, q0)
    q_ref = q0.copy()
    ns_ref = orc.bubble_advance(pb, q_ref, tau)
    ctx = bub.context_from_case(case, bubble_mode=bub.BUBBLES_SPLIT)
    qg = _gpu(torch, q0)
    ns = torch.zeros((nb, n), dtype=torch.int32, device="cuda")
    ctx.bubble_advance(qg, tau, ns)
    assert ctx.last_error()[0] == 0
    _compare_advance(qg.cpu().numpy(), q_ref, ns.cpu().numpy(), ns_ref, 1, nb)
    outs = []
    for calls in ((3,), (1, 1, 1)):
        ctx = bub.context_from_case(case, bubble_mode=bub.BUBBLES_SPLIT)
        q = ctx.init_state(torch.from_numpy(case.prim).cuda())
        work = ctx.new_work()
        for k in calls:
            ctx.rk3_steps(q, work, k)
        assert ctx.last_error()[0] == 0
        outs.append(q)
    assert torch.equal(outs[0], outs[1])
