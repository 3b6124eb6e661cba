"""The allocation-free right-hand side with transfer contents: its bin table holds the contents' equilibrium values
(pressure, vapour and gas mass) as a context's does, so the result is bitwise that of bub_rhs_stage.  A call on
polytropic contents with other bins goes first, so that values left over in the static scratch would show."""
import ctypes
import dataclasses

import pytest

import workloads as W
from tests.parity import perturb_bins

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,nb", [((53,), 5), ((40, 23), 3)])
def test_noalloc_rhs_of_transfer_contents_equals_context_rhs(orc, n, nb, precision):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2511_21031_amd._binding as B
    from tests.test_zz_no_alloc import _noalloc, _structs
    rc, _, _ = _noalloc(torch, B, W.random_smooth(1, (61,), 1e-4, 7, seed=46),
                        torch.ones((1 + 3 + 14, 61), dtype=torch.float64, device="cuda"), precision)
    assert rc == 0
    case = dataclasses.replace(W.random_smooth(len(n), n, 1e-4, nb, seed=45), gas=dict(W.AIR_WITH_VAPOUR),
                               contents=dict(W.AIR_VAPOUR))
    pb = orc.problem_from_case(case)
    qh = orc.init_state(pb, case.prim)
    qh[case.ndim + 2, 5:9] = 0.0   # cells without bubbles take the bins' equilibrium values
    q = torch.from_numpy(perturb_bins(qh, case.ndim, nb, seed=3)).cuda()
    ctx = B.context_from_case(case, precision=precision)
    ref = ctx.rhs_stage(q)
    g, lq, gs, bn, op = _structs(B, case, precision)
    op.contents = B.CONTENTS_TRANSFER
    op.transfer = B._Transfer(*(float(case.contents[k]) for k, _ in B._Transfer._fields_))
    rhs = torch.full_like(q, float("nan"))
    err = torch.full((3,), 7, dtype=torch.int64, device="cuda")
    p = ctypes.c_void_p
    rc = B.lib().bub_rhs_stage_noalloc(*[ctypes.byref(x) for x in (g, lq, gs, bn, op)], p(q.data_ptr()),
                                       p(rhs.data_ptr()), p(err.data_ptr()), p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    torch.cuda.synchronize()
    assert torch.equal(rhs, ref)
    assert err.tolist()[0] == ctx.last_error()[0]
