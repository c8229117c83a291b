"""Import of a configuration and its clover term over block shapes that wrap in
different ways (one-site blocks, two blocks per direction, ragged blocks): the
four storage copies of links and clover term come from one pass, so the
operator at every storage precision is compared with the oracle.

Tolerances: FP64 as for a site's sum of about 100 products (2e-14 of the largest
entry); below, links, clover entries and spinors carry one rounding each and
the FP32 / FP16 / BF16 operator one more per hop, 4u of the result's norm for
about uncorrelated errors (u = 2^-24, 2^-11, 2^-8).
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


@pytest.mark.parametrize("L,block", [((2, 4, 2, 6), (1, 1, 1, 3)), ((4, 4, 4, 4), (2, 2, 2, 2)),
                                     ((10, 6, 6, 10), (5, 3, 3, 5)), ((8, 8, 8, 16), (4, 4, 4, 4))])
def test_setup_all_storage_copies(dwctx, L, block):
    U = synth.gauge_field(L, 0.7, 21)
    f = P.Field(dwctx, L, block, P.to_device(U))
    f.set_clover(1.3)
    x = synth.gaussian_spinor(L, 22)
    m0 = -0.3
    ref = W.apply_D(U, m0, x) + Cl.apply_clover(Cl.clover_term(U, 1.3), x)
    xt = P.to_device(x)
    y = f.apply(m0, xt).cpu().numpy()
    assert np.max(np.abs(y - ref)) <= 2e-14 * np.max(np.abs(ref))
    for prec, u in U_ROUND.items():
        xi = f.pack(prec, xt)
        yi = torch.empty_like(xi)
        f.apply_ex(m0, prec, xi, yi)
        yl = f.unpack(prec, yi).cpu().numpy()[0]
        assert np.linalg.norm(yl - ref) <= 4 * u * np.linalg.norm(ref), prec
    f.close()
