"""Little solves with several blocks per workgroup: staged neighbour vectors in
one and in several pieces, waits on neighbours' flags and on all of them, fewer
and more partial sums than workgroups, rows that fill a workgroup or leave it
split over neighbours, with and without the even-odd reduction.

Even-odd, ||w - A v|| <= max ||D_b|| tol ||s_e|| (s_e the source of the reduced
system, D the block diagonal: the odd part of the residue is zero and the even
part D_e times the reduced one); else tol ||w||; both up to FP64 rounding,
2^-52 (9 Ns)^2 times max |A| ||v||.
"""
import numpy as np
import pytest

import latgen
from paper_0706_2298_amd import Solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,Ns,grid,eo,nkv", [
    ((8, 8, 8, 8), 40, 3, 1, 32), ((8, 8, 8, 16), 8, 2, 0, 5), ((8, 8, 8, 8), 1, 4, 0, 32),
    ((16, 16, 16, 16), 20, 1, 1, 32), ((16, 16, 16, 16), 33, 128, 1, 8), ((16, 16, 16, 16), 7, 5, 0, 32),
    ((24, 16, 16, 24), 12, 0, 1, 32)])
def test_little_general_solve(dims, Ns, grid, eo, nkv):
    print(f"[case] little general solve {dims} Ns={Ns} grid={grid} eo={eo} nkv={nkv}", flush=True)
    S = Solver(dims, Ns=Ns, n_inviter=0, m0=-0.2, m0_setup=-0.2, nkv=2, little_grid=grid, little_eo=eo,
               little_nkv=nkv)
    try:
        S.set_gauge(latgen.make_links(dims, 0.4, 7201))
        S.setup(S.pack(latgen.make_init_fields(dims, Ns, 7202)))
        torch = S.torch
        rng = np.random.default_rng(7203)
        w = rng.standard_normal((S.Nb, Ns)) + 1j * rng.standard_normal((S.Nb, Ns))
        tol = 1e-11
        v, code, it = S.little_solve(torch.tensor(w.ravel(), device="cuda"), tol)
        assert code == 0 and it > 0
        v = v.cpu().numpy().reshape(S.Nb, Ns)
        A = S.little_operator()
        shape = [d // 4 for d in dims]
        idx = np.arange(S.Nb).reshape(shape)
        nb = np.stack([np.roll(idx, -s, axis=mu).ravel() for mu in range(4) for s in (1, -1)], axis=1)

        def hops(M, u):
            return sum(np.einsum("bkl,bl->bk", M[:, 1 + d], u[nb[:, d]]) for d in range(8))

        res = w - np.einsum("bkl,bl->bk", A[:, 0], v) - hops(A, v)
        bound = tol * np.linalg.norm(w)
        if eo:
            Di = np.linalg.inv(A[:, 0])
            w1 = np.einsum("bkl,bl->bk", Di, w)
            even = np.indices(shape).sum(axis=0).ravel() % 2 == 0
            s = (w1 - np.einsum("bkl,bl->bk", Di, hops(A, w1)))[even]
            bound = np.linalg.norm(A[:, 0], ord=2, axis=(1, 2)).max() * tol * np.linalg.norm(s)
        assert np.linalg.norm(res) <= bound + 2.0 ** -52 * (9 * Ns) ** 2 * np.abs(A).max() * np.linalg.norm(v)
        v2, _, it2 = S.little_solve(torch.tensor(w.ravel(), device="cuda"), tol)
        assert it2 == it and np.array_equal(v2.cpu().numpy().reshape(S.Nb, Ns), v)
    finally:
        S.close()
