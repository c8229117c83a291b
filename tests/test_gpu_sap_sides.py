"""A right-hand side's preconditioned vector does not depend on the others in the
call: bit for bit the one of a call on its own, also where the sides together make
more workgroups than the GPU has CUs (8 blocks of a colour x 33 sides on 4^4 blocks)
and for any storage precision.
"""
import pytest
import torch

import paper_1204_5463_amd as P
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("csw", [0.0, 1.9])
@pytest.mark.parametrize("prec", [P.DW_PREC_F64, P.DW_PREC_F32, P.DW_PREC_F16, P.DW_PREC_BF16])
@pytest.mark.parametrize("block", [(4, 4, 4, 4), (2, 4, 4, 4)])
def test_sides(dwctx, csw, prec, block):
    L = (8, 8, 8, 8)
    f = P.Field(dwctx, L, block, P.to_device(synth.gauge_field(L, 0.3, 5)))
    if csw:
        f.set_clover(csw)
    v = P.to_device(synth.gaussian_spinors(L, 3)).repeat((11,) + (1,) * 6).contiguous()
    sp = P.SapParams(block=block, ncycles=2, nmr=5, storage=prec)
    alone = torch.cat([f.sap(0.1, sp, v[r:r + 1].contiguous()) for r in range(3)])
    for n in (2, 32, 33):
        z = f.sap(0.1, sp, v[:n].contiguous())
        assert torch.equal(z, alone.repeat((11,) + (1,) * 6)[:n]), n
    f.close()
