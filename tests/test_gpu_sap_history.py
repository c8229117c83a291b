"""Residual history of the stand-alone SAP iteration over both ways its norms
are formed: in the operator's launch, one partial sum per block (blocks up to 512
sites), and by a pass of its own (540 and 576 sites). One block per
workgroup and a partly filled last wave are among the first kind.

Tolerance: a residual entry carries at most 2e-14 of the right-hand side's
entries; after 4 iterations at this mass the norm is above 1e-3 of the first
one, so the history agrees to 1e-10.
"""
import numpy as np
import pytest
import torch

import paper_1204_5463_amd as P
import synth
from oracle import sap as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [(1, 1, 1, 1), (4, 4, 4, 4), (5, 3, 3, 5), (8, 4, 4, 4), (6, 5, 6, 3), (9, 8, 8, 1)])
def test_history_matches_oracle(dwctx, block):
    L = tuple(2 * v for v in block)
    U = synth.gauge_field(L, 0.3, 4)
    f = P.Field(dwctx, L, block, P.to_device(U))
    b = synth.gaussian_spinor(L, 5)
    x, hist = f.sap_solve(0.2, P.SapParams(block=block, ncycles=1, nmr=3, storage=P.DW_PREC_F64), P.to_device(b), 4)
    xo, ho = S.sap_solve(U, 0.2, L, block, 1, 3, b, 4)
    assert min(ho) > 1e-3
    assert np.max(np.abs(np.array(hist) - ho) / np.array(ho)) < 1e-10
    assert np.max(np.abs(x.cpu().numpy() - xo)) < 1e-10 * np.max(np.abs(xo))
    f.close()


def test_long_history(dwctx):
    """Norms are fetched every 512 iterations: a history across that border
    begins with the short one's values, bit for bit, and stays at the floor; from
    an exactly solved system (one-site blocks without links) it is 0."""
    L, block = (4, 4, 4, 4), (2, 2, 2, 2)
    f = P.Field(dwctx, L, block, P.to_device(synth.gauge_field(L, 0.3, 4)))
    b = P.to_device(synth.gaussian_spinor(L, 5))
    sp = P.SapParams(block=block, ncycles=1, nmr=3, storage=P.DW_PREC_F64)
    short = f.sap_solve(0.4, sp, b, 20)[1]
    for niter in (511, 512, 600):
        hist = f.sap_solve(0.4, sp, b, niter)[1]
        assert len(hist) == niter + 1 and hist[:21] == short
        assert max(hist[400:]) < 1e-14
    f.close()
    L, block = (2, 2, 2, 2), (1, 1, 1, 1)
    f = P.Field(dwctx, L, block, torch.zeros((4, 2, 2, 2, 2, 3, 3), dtype=torch.complex128, device="cuda"))
    b = torch.ones((2, 2, 2, 2, 4, 3), dtype=torch.complex128, device="cuda")
    sp = P.SapParams(block=block, ncycles=1, nmr=1, storage=P.DW_PREC_F64)
    x, hist = f.sap_solve(0.0, sp, b, 530)
    assert hist == [1.0] + [0.0] * 530
    assert torch.equal(x, b / 4)
    f.close()
