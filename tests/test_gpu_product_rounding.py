"""Rounding error of the FP32 operator: a complex product is formed apart and
added to its sum (two roundings at the size of the product, one at that of the
sum), not chained into the sum by fused multiply-adds (every rounding at the size
of the sum), which costs about 1% more error.

Both forms are worked out here in NumPy for the same links and spinor, in the
kernel's order of hops; the GPU's error, over all entries against the FP64
operator on the FP32-rounded inputs, has to lie below the mean of the two.
"""
import numpy as np
import pytest
import torch

import paper_1204_5463_amd as P
import synth
from oracle import wilson as W

F = np.float32


def _r(x):
    return x.astype(F).astype(np.float64)  # one FP32 rounding of an FP64 (nearly exact) value


def _mul(U, h, chain):
    """sum_b U_ab h_sb over colours, entries rounded to FP32 as either form does."""
    re = im = np.zeros(h.shape)
    for b in range(3):
        ur, ui = U.real[..., None, :, b], U.imag[..., None, :, b]
        hr, hi = h.real[..., b, None], h.imag[..., b, None]
        if chain:
            re = _r(ur * hr + re)
            re = _r(-ui * hi + re)
            im = _r(ur * hi + im)
            im = _r(ui * hr + im)
        else:
            re = _r(re + _r(ur * hr - _r(ui * hi)))
            im = _r(im + _r(ur * hi + _r(ui * hr)))
    return re + 1j * im


def _rc(z):
    return _r(z.real) + 1j * _r(z.imag)


def _operator(U, m0, x, chain):
    acc = np.zeros_like(x)
    for mu in range(4):
        ax = W.AXIS[mu]
        for sign in (1, -1):
            y = np.roll(x, -1, axis=ax) if sign > 0 else x
            proj = W.P_MINUS[mu] if sign > 0 else W.P_PLUS[mu]
            half = _rc(np.matmul(proj, y)[..., :2, :])  # one addition per entry
            if sign > 0:
                g = _mul(U[mu], half, chain)
            else:
                g = np.roll(_mul(np.conj(np.swapaxes(U[mu], -1, -2)), half, chain), 1, axis=ax)
            # the lower components are the upper two times +-1 or +-i
            acc = _rc(acc + np.matmul(proj[:, :2], g))
    # scale * (diag * psi - half * acc), contracted to one fused multiply-add
    diag = float(F(4.0 + m0))
    return _rc(diag * x - 0.5 * acc)


def _case():
    L = (8, 8, 8, 8)
    U = synth.gauge_field(L, 0.7, 5).astype(np.complex64).astype(np.complex128)
    x = synth.gaussian_spinor(L, 11).astype(np.complex64).astype(np.complex128)
    m0 = -0.4
    ref = W.apply_D(U, m0, x)
    err = [np.linalg.norm(_operator(U, m0, x, chain) - ref) / np.linalg.norm(ref) for chain in (False, True)]
    return L, U, x, m0, ref, err


def test_forms_differ():
    err = _case()[-1]
    assert 1.005 * err[0] < err[1] < 1.05 * err[0]


@pytest.mark.gpu
@pytest.mark.parametrize("block", [(4, 4, 4, 4), (2, 4, 4, 4)])
def test_fp32_operator_error(dwctx, block):
    L, U, x, m0, ref, err = _case()
    f = P.Field(dwctx, L, block, P.to_device(U))
    xi = f.pack(P.DW_PREC_F32, P.to_device(x))
    yi = torch.empty_like(xi)
    f.apply_ex(m0, P.DW_PREC_F32, xi, yi, nrhs=1)
    y = f.unpack(P.DW_PREC_F32, yi, nrhs=1).cpu().numpy()[0]
    f.close()
    assert np.linalg.norm(y - ref) / np.linalg.norm(ref) < 0.5 * (err[0] + err[1])
