"""Schwarz sweeps against the oracle for the kernels' less common forms: blocks whose sites do not fill the wavefronts
(60 and 288 sites), the clover term without antiperiodic time and the reverse, one and two fields (which select different
kernels), every arithmetic. Tolerances of the parity tests: FP64 1e-12, FP32 1e-4, BF16 links 3e-2."""
import numpy as np
import pytest

import latgen
import oracle
from paper_0706_2298_amd import BF16, F32, F64, Solver

pytestmark = pytest.mark.gpu

CLOVER, ANTI = dict(csw=1.90952), dict(antiperiodic=True)
RAGGED = ((6, 4, 4, 10), (3, 2, 2, 5))
LARGE = ((12, 8, 8, 6), (6, 4, 4, 3))
FOURS = ((8, 8, 8, 8), (4, 4, 4, 4))


@pytest.mark.parametrize("geom,kw", [(RAGGED, CLOVER), (RAGGED, ANTI), (RAGGED, {**CLOVER, **ANTI}),
                                     (LARGE, {}), (LARGE, CLOVER), (LARGE, ANTI), (LARGE, {**CLOVER, **ANTI}),
                                     (FOURS, CLOVER), (FOURS, ANTI)])
@pytest.mark.parametrize("prec,link_prec,nrhs,tol", [(F64, F64, 1, 1e-12), (F64, F64, 2, 1e-12), (F32, F32, 1, 1e-4),
                                                     (F32, F32, 2, 1e-4), (F32, BF16, 1, 3e-2), (F32, BF16, 2, 3e-2)])
def test_sap_variants(geom, kw, prec, link_prec, nrhs, tol):
    dims, sb = geom
    print(f"[case] sap variants {dims} {sb} {kw} prec={prec} links={link_prec} nrhs={nrhs}", flush=True)
    U = latgen.make_links(dims, 0.4, 7501)
    rho = latgen.random_field(dims, 7502, n=nrhs)
    S = Solver(dims, dfl_block=sb, sap_block=sb, Ns=1, nkv=1, little_nkv=1, m0=-0.2, ncy=3, nmr=4, nrhs_max=nrhs,
               sap_prec=prec, link_prec=link_prec, **kw)
    try:
        S.set_gauge(U)
        got = S.unpack(S.sap(S.pack(rho)))
    finally:
        S.close()
    for r in range(nrhs):
        ref = oracle.sap(U, rho[r], -0.2, dims, sb, 3, 4, **kw)
        assert np.abs(got[r] - ref).max() < tol * np.abs(ref).max(), r
