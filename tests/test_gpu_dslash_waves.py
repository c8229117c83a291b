"""The FP64 operator on the internal layout around the block volumes where its
form changes (two lanes per site up to 128 sites and from 225 to 384, one lane in
between and above), with and without the clover term, against the oracle; and the
residual norms of sap_solve, whose operator launch keeps two lanes throughout.

Tolerances as for the operator's other block edges: 100 x 2^-53 of the largest
entry, 2e-14; and 1e-10 for the history of three iterations.
"""
import numpy as np
import pytest
import torch

import paper_1204_5463_amd as P
import synth
from oracle import clover as Cl
from oracle import sap as S
from oracle import wilson as W

pytestmark = pytest.mark.gpu

BLOCKS = [(2, 4, 4, 4), (43, 3, 1, 1), (8, 7, 4, 1), (5, 5, 3, 3), (8, 4, 4, 3), (11, 7, 5, 1)]


@pytest.mark.parametrize("block", BLOCKS)
@pytest.mark.parametrize("csw", [0.0, 1.9])
def test_operator(dwctx, block, csw):
    L = tuple(2 * v for v in block)
    U = synth.gauge_field(L, 0.7, 5)
    f = P.Field(dwctx, L, block, P.to_device(U))
    C = None
    if csw:
        f.set_clover(csw)
        C = Cl.clover_term(U, csw)
    x = synth.gaussian_spinors(L, 2)
    xi = f.pack(P.DW_PREC_F64, P.to_device(x))
    yi = torch.empty_like(xi)
    f.apply_ex(-0.4, P.DW_PREC_F64, xi, yi, nrhs=2)
    y = f.unpack(P.DW_PREC_F64, yi, nrhs=2).cpu().numpy()
    for r in range(2):
        ref = W.apply_D(U, -0.4, x[r])
        if csw:
            ref = ref + Cl.apply_clover(C, x[r])
        assert np.max(np.abs(y[r] - ref)) <= 2e-14 * np.max(np.abs(ref)), r
    f.close()


@pytest.mark.parametrize("block", [(43, 3, 1, 1), (11, 7, 5, 1)])
def test_norms(dwctx, block):
    L = tuple(2 * v for v in block)
    U = synth.gauge_field(L, 0.3, 4)
    f = P.Field(dwctx, L, block, P.to_device(U))
    b = synth.gaussian_spinor(L, 5)
    hist = f.sap_solve(0.2, P.SapParams(block=block, ncycles=1, nmr=3, storage=P.DW_PREC_F64), P.to_device(b), 3)[1]
    ho = S.sap_solve(U, 0.2, L, block, 1, 3, b, 3)[1]
    assert np.max(np.abs(np.array(hist) - ho) / np.array(ho)) < 1e-10
    f.close()
