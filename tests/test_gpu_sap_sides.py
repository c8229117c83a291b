"""The FP64 preconditioner on 4^4 blocks around the numbers of right-hand sides at
which its form changes (one workgroup per CU: 8 blocks of a colour x 32 sides, and
33), with and without the clover term and the adaptive stop: every side as it comes
out on its own, and one against the oracle.

Both forms do the same FP64 arithmetic in another order. Tolerance: 5 x 2 x 2
steps, each with a rounding below 2e-14 of the largest entry (the operator's) and a
condition below 10 for these links: 4e-12; against the oracle the same.
"""
import numpy as np
import pytest
import torch

import paper_1204_5463_amd as P
import synth
from oracle import clover as Cl
from oracle import sap as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("csw", [0.0, 1.9])
@pytest.mark.parametrize("reduction", [0.0, 0.3])
def test_sides(dwctx, csw, reduction):
    L, block = (8, 8, 8, 8), (4, 4, 4, 4)
    U = synth.gauge_field(L, 0.3, 5)
    f = P.Field(dwctx, L, block, P.to_device(U))
    C = None
    if csw:
        f.set_clover(csw)
        C = Cl.clover_term(U, csw)
    x = synth.gaussian_spinors(L, 3)
    v = P.to_device(x).repeat((11,) + (1,) * 6).contiguous()
    sp = P.SapParams(block=block, ncycles=2, nmr=5, storage=P.DW_PREC_F64, mr_reduction=reduction)
    alone = torch.cat([f.sap(0.1, sp, v[r:r + 1].contiguous()) for r in range(3)])
    top = torch.max(torch.abs(alone))
    for n in (32, 33):
        z = f.sap(0.1, sp, v[:n].contiguous())
        for r in range(n):
            assert torch.max(torch.abs(z[r] - alone[r % 3])) <= 4e-12 * top, (n, r)
    ref = S.sap(U, 0.1, L, block, 2, 5, x[1], C=C, reduction=reduction)
    assert np.max(np.abs(z[1].cpu().numpy() - ref)) <= 4e-12 * np.max(np.abs(ref))
    f.close()
