"""Rounding error of the FP32 Schwarz sweeps with the clover term, one lane per site against lane pairs.

Both kinds of kernel round a value of the residue's size once per hop and once for the clover term; the sums inside the
term are smaller. Their errors against FP64 are therefore alike, whatever the number of fields (which selects the kernel)
and the block. Accumulating the term's eleven products per component onto the hop sum instead would add as many roundings
at its size: about 1.3 times the error. The bound lies between, at 1.15.
"""
import numpy as np
import pytest

import latgen
import oracle
from paper_0706_2298_amd import F32, Solver

pytestmark = pytest.mark.gpu
KW = dict(csw=1.90952, antiperiodic=True)


def error(dims, sb, n, U, rho):
    S = Solver(dims, dfl_block=sb, sap_block=sb, Ns=1, nkv=1, little_nkv=1, m0=-0.2, ncy=3, nmr=4, nrhs_max=n,
               sap_prec=F32, link_prec=F32, **KW)
    try:
        S.set_gauge(U)
        got = S.unpack(S.sap(S.pack(rho[:n])))[0]
    finally:
        S.close()
    ref = oracle.sap(U, rho[0], -0.2, dims, sb, 3, 4, **KW)
    return np.linalg.norm(got - ref) / np.linalg.norm(ref)


def test_sap_f32_clover_rounding():
    dims = (16, 8, 8, 8)
    print(f"[case] sap f32 clover rounding {dims}", flush=True)
    # links whose first two rows and sources whose entries are FP32 values: both precisions start from the same numbers
    U = latgen.make_links(dims, 0.4, 7201)
    U[..., :2, :] = U[..., :2, :].astype(np.complex64)
    U[..., 2, :] = np.cross(U[..., 0, :], U[..., 1, :]).conj()
    rho = latgen.random_field(dims, 7202, n=2).astype(np.complex64).astype(np.complex128)
    pair = error(dims, (4, 4, 4, 4), 1, U, rho)
    assert 1e-9 < pair < 1e-6
    assert error(dims, (4, 4, 4, 4), 2, U, rho) < 1.15 * pair
    assert error(dims, (8, 4, 4, 4), 1, U, rho) < 1.15 * pair
