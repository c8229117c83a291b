"""Rounding of the clover term's build: its 3x3 products are formed apart and added
(two roundings at the size of the product), not chained into the sums by fused
multiply-adds (every rounding at the size of the sum).

With m0 = -4 and a spinor on the even sites, D x on the even sites is C x alone.
Both forms of the build are worked out here in NumPy (T(n) the difference of the
two staples of U_mu(n), Q' = T(n) U^+ - T(n - mu)^+ U) and applied with the rounding
of the application; the GPU's error against an 80-bit evaluation has to lie below
the mean of the two.
"""
import numpy as np
import pytest

import paper_1204_5463_amd as P
import synth
from oracle import clover as Cl
from oracle.wilson import AXIS

LD = np.longdouble
L, BLOCK, CSW = (8, 8, 8, 8), (4, 4, 4, 4), 1.9


def _r(x):
    return x.astype(np.float64).astype(LD)


def _mul(a, b, chain, acc=None, neg=False):
    """acc (+|-) a b entry by entry, rounded to FP64 as either form does."""
    re = np.zeros(a.shape, LD) if acc is None else acc.real.copy()
    im = np.zeros(a.shape, LD) if acc is None else acc.imag.copy()
    sg = -1 if neg else 1
    for k in range(3):
        ar, ai = sg * a.real[..., :, k, None], sg * a.imag[..., :, k, None]
        br, bi = b.real[..., None, k, :], b.imag[..., None, k, :]
        if chain:
            re = _r(_r(ar * br + re) - ai * bi)
            im = _r(_r(ar * bi + im) + ai * br)
        else:
            re = _r(re + _r(ar * br - _r(ai * bi)))
            im = _r(im + _r(ar * bi + _r(ai * br)))
    return re + 1j * im


def _dag(a):
    return np.conj(np.swapaxes(a, -1, -2))


def _sh(a, mu, s):
    return np.roll(a, -s, axis=AXIS[mu])


def _half_plane(U, mu, nu, chain):
    """(i csw / 2) F of one plane."""
    u, v = U[mu], U[nu]
    m = _mul(_sh(u, nu, 1), _dag(_sh(v, mu, 1)), chain, neg=True)
    t = _mul(v, m, chain)
    vb, ub = _sh(v, nu, -1), _sh(u, nu, -1)
    t = _mul(_dag(vb), _mul(ub, _sh(vb, mu, 1), chain), chain, acc=t)

    def herm(q):
        return _r((q - _dag(q)).real * (CSW / 16)) * 1j + _r((q - _dag(q)).imag * (CSW / 16)) * -1

    own = herm(_mul(t, _dag(u), chain))
    far = herm(_mul(_dag(t), u, chain, neg=True))
    f = own + _sh(far, mu, -1)
    return _r(f.real) + 1j * _r(f.imag)


def _apply(planes, x, exact):
    C = sum(np.einsum("st,...ab->...satb", Cl.sigma(mu, nu).astype(np.clongdouble), f) for (mu, nu), f in planes.items())
    if exact:
        return np.einsum("...satb,...tb->...sa", C, x)
    C = _r(C.real) + 1j * _r(C.imag)
    re = im = np.zeros(x.shape, LD)
    for t in range(4):
        for b in range(3):
            cr, ci = C.real[..., t, b], C.imag[..., t, b]
            xr, xi = x.real[..., t, b][..., None, None], x.imag[..., t, b][..., None, None]
            re = _r(re + _r(cr * xr - _r(ci * xi)))
            im = _r(im + _r(cr * xi + _r(ci * xr)))
    return re + 1j * im


def _case():
    U = synth.gauge_field(L, 0.7, 5)
    x = synth.gaussian_spinor(L, 3)
    par = sum(np.indices(x.shape[:4])) % 2
    x[par == 1] = 0
    Ul, xl = U.astype(np.clongdouble), x.astype(np.clongdouble)
    pairs = [(mu, nu) for mu in range(4) for nu in range(mu + 1, 4)]
    ref = _apply({p: Cl.field_strength(Ul, *p) * LD(CSW) * 0.5j for p in pairs}, xl, True)[par == 0]
    err = []
    for chain in (False, True):
        y = _apply({p: _half_plane(Ul, *p, chain) for p in pairs}, xl, False)[par == 0]
        err.append(float(np.linalg.norm((y - ref).ravel()) / np.linalg.norm(ref.ravel())))
    return U, x, par, ref, err


def test_forms_differ():
    err = _case()[-1]
    assert 1.01 * err[0] < err[1] < 1.5 * err[0]


@pytest.mark.gpu
def test_clover_error(dwctx):
    U, x, par, ref, err = _case()
    f = P.Field(dwctx, L, BLOCK, P.to_device(U))
    f.set_clover(CSW)
    y = f.apply(-4.0, P.to_device(x)).cpu().numpy()[par == 0]
    f.close()
    assert np.linalg.norm((y - ref).ravel()) / np.linalg.norm(ref.ravel()) < 0.5 * (err[0] + err[1])
