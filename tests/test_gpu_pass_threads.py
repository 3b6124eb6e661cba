"""The primitive pass that half-steps and stages carry, at every number of threads a cell that the grid's own pass can
take (one to 32; the host-side check `threads` holds these sizes to those numbers), bitwise against separate passes."""
import dataclasses

import pytest

import workloads as W

pytestmark = pytest.mark.gpu


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


def _case(n, nb, contents):
    case = W.random_smooth(len(n), n, 1e-4, nb, seed=61 + sum(n), bc=1, amp_atm=0.2)
    if contents:
        case = dataclasses.replace(case, gas=dict(W.AIR_WITH_VAPOUR), contents=dict(W.AIR_VAPOUR))
    return case


def _steps(torch, bub, case, calls, profile=False, **kw):
    groups = kw.pop("groups", 0)
    ctx = bub.context_from_case(case, **kw)
    ctx.set_bin_groups(groups)
    q = ctx.init_state(torch.from_numpy(case.prim).cuda())
    work = ctx.new_work()
    ctx.profile(profile)
    for k in calls:
        ctx.rk3_steps(q, work, k)
    passes = ctx.profile_read(1)[1] if profile else None
    assert ctx.last_error()[0] == 0
    return q, passes


# threads a cell -> sizes
SPLIT = [(1, (700, 760), 3), (2, (600, 500), 5), (4, (150, 140), 5), (8, (150, 150), 7), (16, (100, 100), 17), (32, (45, 40), 31),
         (32, (1800,), 31)]


@pytest.mark.parametrize("contents", [False, True])
@pytest.mark.parametrize("threads,n,nb", SPLIT)
def test_half_steps_carry_the_pass(torch, bub, threads, n, nb, contents):
    """Three split steps in one call, whose half-steps make the next pass, and in three calls, each with its own."""
    case = _case(n, nb, contents)
    one, _ = _steps(torch, bub, case, (3,), bubble_mode=bub.BUBBLES_SPLIT)
    three, _ = _steps(torch, bub, case, (1, 1, 1), bubble_mode=bub.BUBBLES_SPLIT)
    assert torch.equal(one, three)


# threads a cell, sizes, contents: grids below 2^19 cells whose stages carry the pass
CARRY = [(2, (600, 500), 5, False), (2, (600, 500), 5, True), (4, (150, 140), 5, False), (8, (211, 203), 11, False),
         (8, (200, 190), 11, True), (8, (32, 32, 30), 11, False)]


@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("threads,n,nb,contents", CARRY)
def test_stages_carry_the_pass(torch, bub, threads, n, nb, contents, split):
    """Three steps in one call against separate passes (the bins in two groups).  The first step's pass is the only one
    of its own, or in split mode none after it."""
    case = _case(n, nb, contents)
    mode = bub.BUBBLES_SPLIT if split else bub.BUBBLES_UNSPLIT
    fused, passes = _steps(torch, bub, case, (3,), profile=True, bubble_mode=mode)
    apart, more = _steps(torch, bub, case, (3,), profile=True, bubble_mode=mode, groups=2)
    assert passes == 1 and more == (7 if split else 9)
    assert torch.equal(fused, apart)


@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("n", [(160, 150), (30, 29, 28)])
def test_one_bin_carries_the_pass(torch, bub, n, mixed, split):
    """One bin on two threads a cell, the second without any: the stages of a context with memory of its own carry the
    pass (but for mixed boxes with sources); one on the caller's buffer has no room for it."""
    case = _case(n, 1, False)
    kw = dict(bubble_mode=bub.BUBBLES_SPLIT if split else bub.BUBBLES_UNSPLIT, profile=True,
              precision=bub.PREC_MIXED if mixed else bub.PREC_FP64)
    own, passes = _steps(torch, bub, case, (3,), **kw)
    buf, more = _steps(torch, bub, case, (3,), torch_buffer=True, **kw)
    starved = len(n) == 3 and mixed and not split
    assert more == (7 if split else 9) and passes == (more if starved else 1)
    assert torch.equal(own, buf)
