"""The FP64 operator over block volumes around the edges of its launch forms:
one site, a group of 32 sites and one more, a ragged block, the largest block
of the two-lane form (512 sites), the one-lane form above it (540) and the
gather form (576), on several right-hand sides, with and without the clover
term, on canonical fields (dw_apply) and on the internal layout (dw_apply_ex).

Tolerance: a site's result is a sum of about 8 x 9 products of numbers of
modulus at most 1 with spinor entries (and 12 of the clover term), so its
rounding error is below 100 x 2^-53 times the largest entry: 2e-14.
"""
import numpy as np
import pytest
import torch

import paper_1204_5463_amd as P
import synth
from oracle import clover as Cl
from oracle import wilson as W

pytestmark = pytest.mark.gpu

BLOCKS = [(1, 1, 1, 1), (2, 4, 4, 1), (11, 3, 1, 1), (5, 3, 3, 5), (8, 4, 4, 4), (6, 5, 6, 3), (9, 8, 8, 1)]


@pytest.mark.parametrize("block", BLOCKS)
@pytest.mark.parametrize("csw", [0.0, 1.9])
def test_fp64_operator_block_edges(dwctx, block, csw):
    L = tuple(2 * v for v in block)
    U = synth.gauge_field(L, 0.7, 5)
    f = P.Field(dwctx, L, block, P.to_device(U))
    C = None
    if csw:
        f.set_clover(csw)
        C = Cl.clover_term(U, csw)
    x = synth.gaussian_spinors(L, 3)
    m0 = -0.4
    xt = P.to_device(x)
    y = f.apply(m0, xt).cpu().numpy()
    xi = f.pack(P.DW_PREC_F64, xt)
    yi = torch.empty_like(xi)
    f.apply_ex(m0, P.DW_PREC_F64, xi, yi, nrhs=3)
    ye = f.unpack(P.DW_PREC_F64, yi, nrhs=3).cpu().numpy()
    for r in range(3):
        ref = W.apply_D(U, m0, x[r])
        if csw:
            ref = ref + Cl.apply_clover(C, x[r])
        scale = np.max(np.abs(ref))
        assert np.max(np.abs(y[r] - ref)) <= 2e-14 * scale, (block, r)
        assert np.max(np.abs(ye[r] - ref)) <= 2e-14 * scale, (block, r)
    f.close()


@pytest.mark.parametrize("csw", [0.0, 1.9])
def test_fp64_operator_4x4x4x4_forms(dwctx, csw):
    """4^4 blocks have a form of their own; 16 blocks x 16 right-hand sides fill
    the CUs once, 17 do not. The oracle bound at the first and last right-hand
    side, and the same bits from both launches."""
    L, block, m0 = (8, 8, 8, 8), (4, 4, 4, 4), -0.4
    U = synth.gauge_field(L, 0.7, 5)
    f = P.Field(dwctx, L, block, P.to_device(U))
    C = None
    if csw:
        f.set_clover(csw)
        C = Cl.clover_term(U, csw)
    x = synth.gaussian_spinors(L, 17)
    xt = P.to_device(x)
    xi = f.pack(P.DW_PREC_F64, xt)
    out = {}
    for nr in (16, 17):
        y = f.apply(m0, xt[:nr].contiguous())
        yi = torch.empty_like(xi)
        f.apply_ex(m0, P.DW_PREC_F64, xi, yi, nrhs=nr)
        out[nr] = y.cpu(), f.unpack(P.DW_PREC_F64, yi, nrhs=nr).cpu()
    for r in (0, 15):
        ref = W.apply_D(U, m0, x[r])
        if csw:
            ref = ref + Cl.apply_clover(C, x[r])
        for y in out[16]:
            assert np.max(np.abs(y[r].numpy() - ref)) <= 2e-14 * np.max(np.abs(ref)), r
    for a, b in zip(out[16], out[17]):
        assert torch.equal(a, b[:16])
    f.close()


@pytest.mark.parametrize("csw", [0.0, 1.9])
def test_fp32_operator_4x4x4x4_forms(dwctx, csw):
    """FP32 storage: 16 blocks x 256 right-hand sides is the largest launch of the
    form for small grids, 257 the smallest of the general one: the same bits, and
    the FP64 operator to 4 x 2^-24 of the norm (roundings of inputs and hops)."""
    L, block, m0 = (8, 8, 8, 8), (4, 4, 4, 4), -0.4
    f = P.Field(dwctx, L, block, P.to_device(synth.gauge_field(L, 0.7, 5)))
    if csw:
        f.set_clover(csw)
    x = P.to_device(synth.gaussian_spinors(L, 3)).repeat((86,) + (1,) * 6)[:257].contiguous()
    xi = f.pack(P.DW_PREC_F32, x)
    out = []
    for nr in (256, 257):
        yi = torch.zeros_like(xi)
        f.apply_ex(m0, P.DW_PREC_F32, xi, yi, nrhs=nr)
        out.append(f.unpack(P.DW_PREC_F32, yi, nrhs=nr)[:256])
    assert torch.equal(out[0], out[1])
    ref = f.apply(m0, x[:3].contiguous())
    assert torch.linalg.vector_norm(out[0][:3] - ref) <= 4 * 2.0 ** -24 * torch.linalg.vector_norm(ref)
    f.close()
