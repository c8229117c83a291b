"""Restart cycles of the smallest and largest shapes against the oracle: the QR
factorisation carried from step to step (a Householder-factored leading block
of k columns after a deflated restart, one rotation per further column), the
least-squares solution at the cycle end and the deflated restart itself.

Tolerances: both solvers stop at ||b - D x|| <= 1e-10 ||b||. The Hermitian part
of D is at least m0, so ||D^-1|| <= 1 / m0 = 2 and ||b|| <= (8 + m0) ||x||; the two
solutions differ by at most 2 x 2 x 1e-10 x 8.5 = 3.4e-9 relative. Iteration
counts may differ by one where a residual falls on the stopping threshold.
"""
import numpy as np
import pytest

import paper_1204_5463_amd as P
import synth
from oracle import fgmresdr as F
from oracle import sap as S
from oracle import wilson as W

pytestmark = pytest.mark.gpu

L, BLOCK, M0 = (8, 4, 4, 8), (2, 2, 2, 2), 0.5


@pytest.mark.parametrize("m,k", [(1, 0), (2, 1), (3, 2), (7, 1), (24, 23), (48, 0), (48, 23)])
def test_cycle_shapes_follow_oracle(dwctx, m, k):
    U = synth.gauge_field(L, 0.7, 11)
    b = synth.gaussian_spinor(L, 12)
    shp = b.shape
    xo, info = F.fgmresdr(lambda v: W.apply_D(U, M0, v.reshape(shp)).reshape(-1),
                          lambda v: S.sap(U, M0, L, BLOCK, 1, 1, v.reshape(shp)).reshape(-1),
                          b.reshape(-1), m, k, tol=1e-10, max_iter=400)
    f = P.Field(dwctx, L, BLOCK, P.to_device(U))
    prm = P.SolverParams(m=m, k=k, tol=1e-10, max_iter=400,
                         sap=P.SapParams(block=BLOCK, ncycles=1, nmr=1, storage=P.DW_PREC_F64))
    x, st = f.solve(M0, prm, P.to_device(b))
    x = x.cpu().numpy().reshape(-1)
    assert st[0].converged and info.converged
    assert abs(st[0].iterations - info.iterations) <= 1, (m, k, st[0].iterations, info.iterations)
    assert np.linalg.norm(x - xo) <= 3.4e-9 * np.linalg.norm(xo), (m, k)
    f.close()
