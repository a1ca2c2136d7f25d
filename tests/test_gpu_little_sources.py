"""Batches of sources on both sides of the line between the block-pair little solver, whose launches take a few sources
each, and the batched one: up to three launches of one source (257..512 blocks), four of several (fewer blocks), two and
one for up to 16 and 8 fields."""
import numpy as np
import pytest

import latgen
from paper_0706_2298_amd import PROJ_COARSE, Solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,Ns,ns", [((32, 16, 16, 16), 17, (3, 4)), ((24, 16, 16, 16), 17, (3, 4)),
                                        ((16, 16, 16, 16), 17, (8, 9)), ((16, 16, 16, 16), 9, (4, 5)),
                                        ((32, 16, 16, 16), 8, (1, 2))])
def test_little_sources(dims, Ns, ns):
    print(f"[case] little sources {dims} Ns={Ns} {ns}", flush=True)
    S = Solver(dims, Ns=Ns, n_inviter=0, m0=-0.2, m0_setup=-0.2, nkv=2, nrhs_max=max(ns))
    try:
        S.set_gauge(latgen.make_links(dims, 0.4, 7301))
        S.setup(S.pack(latgen.make_init_fields(dims, Ns, 7302)))
        y = S.pack(latgen.random_field(dims, 7303, n=max(ns)))
        per = 12 * S.V
        for n in ns:
            got = S.unpack(S.project(PROJ_COARSE, y[:n * per].clone()))
            for r in (0, n - 1):
                one = S.unpack(S.project(PROJ_COARSE, y[r * per:(r + 1) * per].clone()))[0]
                # the projectors' parity tolerance (little solves to 1e-12)
                assert np.linalg.norm(got[r] - one) <= 1e-9 * np.linalg.norm(one), (n, r)
    finally:
        S.close()
