"""The clover term enters the stencil with one rounding: D psi with the term equals the plain D psi plus C psi, bit by
bit. C psi alone comes from sources on one parity of sites, whose hops end on the other, at 4 + m0 = 0."""
import numpy as np
import pytest

import latgen
from paper_0706_2298_amd import F32, F64, Solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,b", [((8, 8, 8, 8), (4, 4, 4, 4)), ((6, 4, 4, 10), (3, 2, 2, 5))])
@pytest.mark.parametrize("prec", [F64, F32])
def test_clover_added_once(dims, b, prec):
    print(f"[case] clover added once {dims} prec={prec}", flush=True)
    U = latgen.make_links(dims, 0.4, 7101)
    dt = np.complex128 if prec == F64 else np.complex64
    psi = latgen.random_field(dims, 7102, n=1).astype(dt).astype(np.complex128)
    par = (np.indices(dims).sum(axis=0).reshape(1, -1, 1) % 2).astype(bool)

    def dirac(f, m0, **kw):
        S = Solver(dims, dfl_block=b, sap_block=b, Ns=1, nkv=1, little_nkv=1, m0=m0, link_prec=prec, sap_prec=prec, **kw)
        try:
            S.set_gauge(U)
            return S.unpack(S.dirac(S.pack(f, prec=prec), prec=prec), prec=prec).reshape(psi.shape)
        finally:
            S.close()

    clover = sum(dirac(psi * p, -4.0, csw=1.90952) * p for p in (par, ~par))
    assert abs(clover).max() > 0.1
    want = (dirac(psi, -0.2) + clover).astype(dt)
    got = dirac(psi, -0.2, csw=1.90952).astype(dt)
    assert (got == want).all(), abs(got - want).max()
