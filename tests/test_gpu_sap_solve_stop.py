"""sap_solve from an exact solution on: the residual of one-site blocks without
links is zero after one iteration at FP64 (its division is exact there). The preconditioner is launched up to the next
look at the norms at most (after 8 iterations, two colours each), whatever the
number of iterations asked for, and changes nothing.

A history that crosses several looks, with the last norm of each at its place:
the same values as from calls that stop before and after every look.
"""
import pytest
import torch

import paper_1204_5463_amd as P
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("niter", [1, 6, 7, 8, 530])
def test_exact_solution(niter):
    ctx = P.Context(0)
    L, block = (2, 2, 2, 2), (1, 1, 1, 1)
    f = P.Field(ctx, L, block, torch.zeros((4, 2, 2, 2, 2, 3, 3), dtype=torch.complex128, device="cuda"))
    b = torch.ones((2, 2, 2, 2, 4, 3), dtype=torch.complex128, device="cuda")
    sp = P.SapParams(block=block, ncycles=1, nmr=1, storage=P.DW_PREC_F64)
    ctx.profile(True)
    ctx.profile_reset()
    x, hist = f.sap_solve(0.0, sp, b, niter)
    launches = ctx.profile_stats()["sap"]["launches"]
    assert hist == [1.0] + [0.0] * niter
    assert torch.equal(x, b / 4)
    assert launches <= 2 * min(niter, 7)
    f.close()
    ctx.close()


@pytest.mark.parametrize("block", [(2, 2, 2, 2), (9, 8, 8, 1)])
def test_history_across_looks(dwctx, block):
    L = tuple(2 * v for v in block)
    f = P.Field(dwctx, L, block, P.to_device(synth.gauge_field(L, 0.3, 4)))
    b = P.to_device(synth.gaussian_spinor(L, 5))
    sp = P.SapParams(block=block, ncycles=1, nmr=2, storage=P.DW_PREC_F32)
    long = f.sap_solve(0.4, sp, b, 34)[1]
    for niter in (0, 6, 7, 8, 14, 15, 16, 30, 31, 32):
        assert f.sap_solve(0.4, sp, b, niter)[1] == long[:niter + 1]
    f.close()
