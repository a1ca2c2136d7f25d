"""Little solves with one block pair per workgroup: numbers of blocks on both
sides of the two reduction schemes (16 workgroups), fewer and more sums than
workgroups, Ns at the register sizes' edges, restarts, and more sources than
one launch takes.

The solver stops at ||r_e|| <= tol ||s_e||, s_e the source and r_e the residue
of the even-odd reduced system; the odd part of the full residue is zero and
its even part is D_e r_e (D the block diagonal), so ||w - A v|| <= max ||D_b||
tol ||s_e||, up to FP64 rounding: 2^-52 (9 Ns)^2 times max |A| ||v|| for the
operator and its reduced form.
"""
import numpy as np
import pytest

import latgen
from paper_0706_2298_amd import PROJ_COARSE, Solver

pytestmark = pytest.mark.gpu


def make(dims, Ns, **kw):
    S = Solver(dims, Ns=Ns, n_inviter=0, m0=-0.2, m0_setup=-0.2, nkv=2, **kw)
    S.set_gauge(latgen.make_links(dims, 0.4, 7101))
    S.setup(S.pack(latgen.make_init_fields(dims, Ns, 7102)))
    return S


def neighbours(nb):
    """(Nb, 8) block indices: +mu, -mu for mu = 0..3; and the colours."""
    idx = np.arange(int(np.prod(nb))).reshape(nb)
    n = np.stack([np.roll(idx, -s, axis=mu).ravel() for mu in range(4) for s in (1, -1)], axis=1)
    return n, (np.indices(nb).sum(axis=0) % 2).ravel()


@pytest.mark.parametrize("dims,Ns,nkv,tol", [((8, 8, 8, 8), 1, 32, 1e-12), ((8, 8, 8, 8), 24, 5, 1e-10),
                                             ((8, 8, 8, 16), 13, 32, 1e-6), ((8, 8, 16, 16), 32, 32, 1e-12),
                                             ((16, 16, 16, 16), 25, 7, 1e-9), ((32, 16, 16, 16), 8, 32, 1e-12)])
def test_little_pair_solve(dims, Ns, nkv, tol):
    print(f"[case] little pair solve {dims} Ns={Ns} nkv={nkv} tol={tol}", flush=True)
    S = make(dims, Ns, little_nkv=nkv)
    try:
        torch = S.torch
        rng = np.random.default_rng(7103)
        w = rng.standard_normal((S.Nb, Ns)) + 1j * rng.standard_normal((S.Nb, Ns))
        v, code, it = S.little_solve(torch.tensor(w.ravel(), device="cuda"), tol)
        assert code == 0 and it > 0
        v = v.cpu().numpy().reshape(S.Nb, Ns)
        A = S.little_operator()
        nb, colour = neighbours([d // 4 for d in dims])

        def hops(M, u):
            return sum(np.einsum("bkl,bl->bk", M[:, 1 + d], u[nb[:, d]]) for d in range(8))

        res = w - np.einsum("bkl,bl->bk", A[:, 0], v) - hops(A, v)
        Di = np.linalg.inv(A[:, 0])
        w1 = np.einsum("bkl,bl->bk", Di, w)
        s = (w1 - np.einsum("bkl,bl->bk", Di, hops(A, w1)))[colour == 0]
        slack = 2.0 ** -52 * (9 * Ns) ** 2 * np.abs(A).max() * np.linalg.norm(v)
        bound = np.linalg.norm(A[:, 0], ord=2, axis=(1, 2)).max() * tol * np.linalg.norm(s)
        assert np.linalg.norm(res) <= bound + slack
        # the same solve again: bit for bit
        v2, _, it2 = S.little_solve(torch.tensor(w.ravel(), device="cuda"), tol)
        assert it2 == it and np.array_equal(v2.cpu().numpy().reshape(S.Nb, Ns), v)
    finally:
        S.close()


@pytest.mark.parametrize("dims,n", [((8, 8, 8, 8), 16), ((16, 16, 16, 16), 5), ((32, 16, 16, 16), 2)])
def test_little_pair_sources(dims, n):
    # batches of sources (one launch, several launches with a remainder, one source per launch)
    # give what single sources give, to the projectors' parity tolerance
    print(f"[case] little pair sources {dims} n={n}", flush=True)
    S = make(dims, 8, nrhs_max=n)
    try:
        y = S.pack(latgen.random_field(dims, 7104, n=n))
        got = S.unpack(S.project(PROJ_COARSE, y))
        per = 12 * S.V
        for r in (0, n - 1):
            one = S.unpack(S.project(PROJ_COARSE, y[r * per:(r + 1) * per].clone()))[0]
            assert np.linalg.norm(got[r] - one) <= 1e-9 * np.linalg.norm(one)
    finally:
        S.close()
