"""The FP64 operator with the clover term, whose entries are read in two batches: rounding
error on canonical fields and the internal layout, over blocks of a lane group
(4^4), of one site, and of a partly filled last group.

Bound: an entry is a sum of 8 hops, 11 clover products and the diagonal. With
every operation off by half a unit of the largest partial sum S, the error's
norm stays below sqrt(60) / 2 x 2^-53 x S / |result|, and S / |result| below 4
(hops of modulus up to 8 and clover entries up to 2 against a diagonal of 3.6):
16 x 2^-53 = 1.8e-15 of the norm, against an 80-bit evaluation.
"""
import numpy as np
import pytest
import torch

import paper_1204_5463_amd as P
import synth
from oracle import clover as Cl
from oracle import wilson as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [(4, 4, 4, 4), (1, 1, 1, 1), (5, 3, 3, 5), (11, 3, 1, 1)])
def test_error_against_80_bits(dwctx, block):
    L = tuple(2 * v for v in block) if block != (1, 1, 1, 1) else (4, 4, 4, 4)
    U = synth.gauge_field(L, 0.7, 5)
    x = synth.gaussian_spinor(L, 3)
    m0, csw = -0.4, 1.9
    Ul, xl = U.astype(np.clongdouble), x.astype(np.clongdouble)
    ref = W.apply_D(Ul, np.longdouble(m0), xl)
    for mu in range(4):
        for nu in range(mu + 1, 4):
            F = Cl.field_strength(Ul, mu, nu) * np.longdouble(csw) * 0.5j
            ref = ref + np.einsum("st,...ab,...tb->...sa", Cl.sigma(mu, nu), F, xl)
    f = P.Field(dwctx, L, block, P.to_device(U))
    f.set_clover(csw)
    xt = P.to_device(x)
    y = f.apply(m0, xt)
    xi = f.pack(P.DW_PREC_F64, xt)
    yi = torch.empty_like(xi)
    f.apply_ex(m0, P.DW_PREC_F64, xi, yi, nrhs=1)
    for got in (y, f.unpack(P.DW_PREC_F64, yi, nrhs=1)[0]):
        err = np.linalg.norm((got.cpu().numpy() - ref).ravel()) / np.linalg.norm(ref.ravel())
        assert err < 16 * 2.0 ** -53, (block, float(err))
    f.close()
