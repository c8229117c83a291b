"""SAP on 4^4 blocks at FP64 and FP32 storage (two threads per site) against the
oracle: lattices with two and more blocks per direction, so that a block's two
neighbours are the same or different, no MR step, one and several, one and
several cycles, three right-hand sides in one launch, with and without the
clover term.

Tolerances: the oracle runs in FP64. An MR step is a contraction of the block
residual, so rounding errors of a step (u times a sum of about 100 terms) add up
over at most 2 x 2 x 6 hop sums: below 1e-12 at u = 2^-53 and 1e-4 at u = 2^-24;
uncorrelated errors stay a factor 20 below, 5e-6.
"""
import numpy as np
import pytest

import paper_1204_5463_amd as P
import synth
from oracle import clover as Cl
from oracle import sap as S

pytestmark = pytest.mark.gpu

B = (4, 4, 4, 4)


@pytest.mark.parametrize("prec,tol", [(P.DW_PREC_F64, 1e-12), (P.DW_PREC_F32, 5e-6)])
@pytest.mark.parametrize("L,ncycles,nmr,csw", [((8, 8, 8, 8), 1, 1, 0.0), ((8, 16, 8, 16), 2, 5, 0.0),
                                               ((16, 8, 16, 8), 1, 6, 1.9), ((8, 8, 8, 16), 2, 0, 0.0)])
def test_split_sap_matches_oracle(dwctx, prec, tol, L, ncycles, nmr, csw):
    U = synth.gauge_field(L, 0.7, 31)
    f = P.Field(dwctx, L, B, P.to_device(U))
    C = None
    if csw:
        f.set_clover(csw)
        C = Cl.clover_term(U, csw)
    m0 = -0.2
    v = synth.gaussian_spinors(L, 3)
    z = f.sap(m0, P.SapParams(block=B, ncycles=ncycles, nmr=nmr, storage=prec), P.to_device(v)).cpu().numpy()
    for r in (0, 2):
        ref = S.sap(U, m0, L, B, ncycles, nmr, v[r], C=C)
        n = np.linalg.norm(ref)
        assert np.linalg.norm(z[r] - ref) <= tol * n if n > 0 else not np.any(z[r])
    f.close()
