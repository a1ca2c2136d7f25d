"""FP32 Schwarz sweeps of very small and very large sources.

A sweep is linear in its source, its coefficients are ratios of FP64 sums and a
power of two scales FP32 values exactly, so the result of a scaled source is the
scaled result, bit by bit, while entries stay inside FP32's range. Squares of the
entries (2^-160, 2^160) lie outside it: the sums have to be formed in FP64.
"""
import pytest

import latgen
from paper_0706_2298_amd import BF16, F32, Solver

pytestmark = pytest.mark.gpu
CSW = 1.90952


@pytest.mark.parametrize("dims,sb,kw", [
    ((8, 8, 8, 8), (4, 4, 4, 4), dict(csw=CSW, antiperiodic=True)),
    ((8, 8, 8, 8), (4, 4, 4, 4), dict(antiperiodic=True)),
    ((6, 4, 4, 10), (3, 2, 2, 5), dict(csw=CSW)),
    ((16, 8, 8, 8), (8, 4, 4, 4), dict(csw=CSW, antiperiodic=True)),
    ((16, 8, 8, 8), (8, 4, 4, 4), {}),
    ((12, 8, 8, 6), (6, 4, 4, 3), {}),
])
@pytest.mark.parametrize("link_prec,nrhs", [(F32, 1), (F32, 2), (BF16, 2)])
def test_sap_f32_scaled_source(dims, sb, kw, link_prec, nrhs):
    print(f"[case] sap f32 scaled {dims} {sb} {kw} links={link_prec} nrhs={nrhs}", flush=True)
    S = Solver(dims, dfl_block=sb, sap_block=sb, Ns=1, nkv=1, little_nkv=1, m0=-0.2, ncy=3, nmr=4, nrhs_max=nrhs,
               sap_prec=F32, link_prec=link_prec, **kw)
    try:
        S.set_gauge(latgen.make_links(dims, 0.4, 7001))
        rho = latgen.random_field(dims, 7002, n=nrhs)
        ref = S.unpack(S.sap(S.pack(rho)))
        assert abs(ref).max() > 0.1
        for e in (-80, 80):
            got = S.unpack(S.sap(S.pack(rho * 2.0 ** e))) * 2.0 ** -e
            assert (got == ref).all(), (e, abs(got - ref).max())
    finally:
        S.close()
