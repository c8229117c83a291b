"""dw_apply and dw_apply_noalloc on views of one buffer: the operator on
canonical fields writes y while it still reads x, so views that overlap have to
take the route through copies, and give the same result as fields apart.

Both routes do the same arithmetic per site; the bound of 2e-14 is the rounding
of a site's sum of some 72 products (100 x 2^-53 of the largest entry).
"""
import pytest
import torch

import paper_1204_5463_amd as P
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [(4, 4, 4, 4), (5, 3, 3, 5), (9, 8, 8, 1)])
@pytest.mark.parametrize("sites", [1, 84, -1, "field", "-field"])
def test_shifted_views(dwctx, block, sites):
    L = tuple(2 * v for v in block)
    f = P.Field(dwctx, L, block, P.to_device(synth.gauge_field(L, 0.7, 5)))
    x0 = P.to_device(synth.gaussian_spinors(L, 2))
    want = f.apply(-0.4, x0)
    one = f.volume * 12
    shift = {"field": one, "-field": -one}.get(sites) or 12 * sites
    for apply in (f.apply, f.apply_noalloc):
        buf = torch.zeros(3 * one, dtype=torch.complex128, device="cuda")
        at = max(0, -shift)
        x = buf[at:at + 2 * one].view(x0.shape)
        y = buf[at + shift:at + shift + 2 * one].view(x0.shape)
        x.copy_(x0)
        apply(-0.4, x, y)
        assert torch.max(torch.abs(y - want)) <= 2e-14 * torch.max(torch.abs(want))
    f.close()


def test_same_array_is_refused(dwctx):
    L, block = (8, 8, 8, 8), (4, 4, 4, 4)
    f = P.Field(dwctx, L, block, P.to_device(synth.gauge_field(L, 0.7, 5)))
    x = P.to_device(synth.gaussian_spinors(L, 1))
    for apply in (f.apply, f.apply_noalloc):
        with pytest.raises(P.DwError):
            apply(-0.4, x, x)
    f.close()
