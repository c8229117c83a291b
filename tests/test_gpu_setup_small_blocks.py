"""Import and clover term on blocks of one and two sites, whose lower-precision
copies are converted from the FP64 one, and of three, the next: the operator at
every storage precision against the oracle.

Tolerances as for other block shapes: FP64 2e-14 of the largest entry, below it 4u of
the result's norm (one rounding each of links, clover entries, spinors and hops).
"""
import numpy as np
import pytest
import torch

import paper_1204_5463_amd as P
import synth
from oracle import clover as Cl
from oracle import wilson as W

pytestmark = pytest.mark.gpu

U_ROUND = {P.DW_PREC_F32: 2.0 ** -24, P.DW_PREC_F16: 2.0 ** -11, P.DW_PREC_BF16: 2.0 ** -8}


@pytest.mark.parametrize("L,block", [((2, 4, 6, 4), (1, 1, 1, 1)), ((16, 8, 6, 4), (1, 1, 1, 1)),
                                     ((4, 2, 4, 8), (1, 1, 1, 2)), ((8, 2, 4, 2), (2, 1, 1, 1)),
                                     ((2, 6, 4, 4), (1, 3, 1, 1))])
@pytest.mark.parametrize("csw", [0.0, 1.3])
def test_storage_copies(dwctx, L, block, csw):
    U = synth.gauge_field(L, 0.7, 21)
    f = P.Field(dwctx, L, block, P.to_device(U))
    x = synth.gaussian_spinor(L, 22)
    ref = W.apply_D(U, -0.3, x)
    if csw:
        f.set_clover(csw)
        ref = ref + Cl.apply_clover(Cl.clover_term(U, csw), x)
    xt = P.to_device(x)
    y = f.apply(-0.3, xt).cpu().numpy()
    assert np.max(np.abs(y - ref)) <= 2e-14 * np.max(np.abs(ref))
    for prec, u in U_ROUND.items():
        xi = f.pack(prec, xt)
        yi = torch.empty_like(xi)
        f.apply_ex(-0.3, prec, xi, yi)
        yl = f.unpack(prec, yi).cpu().numpy()[0]
        assert np.linalg.norm(yl - ref) <= 4 * u * np.linalg.norm(ref), prec
    f.close()
