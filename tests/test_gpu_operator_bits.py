"""The FP64 operator has forms with one and with two lanes per site, on canonical
fields and on the internal layout. Without the clover term all of them add the
same hops in the same order, so a result does not depend on the entry point: the
same bits on blocks whose internal layout takes one lane (512 and 180 sites) and
two (128, 81).
"""
import pytest
import torch

import paper_1204_5463_amd as P
import synth

pytestmark = pytest.mark.gpu


def _results(ctx, L, block, U, x):
    f = P.Field(ctx, L, block, P.to_device(U))
    xt = P.to_device(x)
    y = f.apply(-0.4, xt)
    xi = f.pack(P.DW_PREC_F64, xt)
    yi = torch.empty_like(xi)
    f.apply_ex(-0.4, P.DW_PREC_F64, xi, yi, nrhs=2)
    out = [y, f.unpack(P.DW_PREC_F64, yi, nrhs=2)]
    f.close()
    return out


@pytest.mark.parametrize("block", [(8, 4, 4, 4), (6, 5, 2, 3), (2, 4, 4, 4), (3, 3, 3, 3)])
def test_entry_points(dwctx, block):
    L = tuple(2 * v for v in block)
    y, ye = _results(dwctx, L, block, synth.gauge_field(L, 0.7, 5), synth.gaussian_spinors(L, 2))
    assert torch.equal(y, ye)
