"""sap_solve on blocks above 512 sites, where the residual's norm comes from a
pass of its own: its result and the history's entry are different places, as
the kernel that reads the one and writes the other declares (the launcher
refuses the same address). At FP64 and, for the scale formed from the norm, at
FP16 storage.

FP64: roundings only, 1e-10 after 3 iterations (see test_gpu_sap_history).
FP16: a correction M r is off by 8 x 2^-11 of itself (input, links and the
packed residual of three steps rounded), ||M r|| = 0.27 ||r|| here, ||D|| <= 8 + m0
and ||r_k+1|| >= 0.2 ||r_k||: 8 x 2^-11 x 0.27 x 8.2 / 0.2 = 0.044 per entry of the
history, and as much again from the steps before. A scale that is not the
norm's is off by a factor.
"""
import numpy as np
import pytest

import paper_1204_5463_amd as P
import synth
from oracle import sap as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [(6, 5, 6, 3), (9, 8, 8, 1)])
@pytest.mark.parametrize("prec", [P.DW_PREC_F64, P.DW_PREC_F16])
def test_history(dwctx, block, prec):
    L = tuple(2 * v for v in block)
    U = synth.gauge_field(L, 0.3, 4)
    f = P.Field(dwctx, L, block, P.to_device(U))
    b = 1e-3 * synth.gaussian_spinor(L, 6)
    _, hist = f.sap_solve(0.2, P.SapParams(block=block, ncycles=1, nmr=3, storage=prec), P.to_device(b), 3)
    ho = S.sap_solve(U, 0.2, L, block, 1, 3, b, 3)[1]
    err = np.max(np.abs(np.array(hist) - ho) / np.array(ho))
    assert err < (1e-10 if prec == P.DW_PREC_F64 else 0.09)
    f.close()
