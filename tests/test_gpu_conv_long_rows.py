"""FP32 convolutions on lattices whose rows are too long for staged tiles of whole rows: a tile is a segment of one row.
One, two and three segments a row, equal and unequal.

Tolerance: an FP32 sum of n products in any order is off its exact value by at most n 2^-24 / (1 - n 2^-24) times the sum
of the products' moduli; the bias adds one rounding, the activation a relative error of at most 2^-20. The factor silu'(z)
= s (1 + z (1 - s)) has a zero near z = -1.28, where it keeps no relative accuracy: its error is at most 2^-20 (1 + |z|).
"""
import numpy as np
import pytest

import latgen
from oracle import net as onet
from paper_0706_2298_amd import Solver, binding

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24


@pytest.mark.parametrize("dims,blk", [((4, 4, 2, 50), (2, 2, 1, 5)), ((2, 2, 4, 96), (1, 1, 2, 8)),
                                      ((2, 4, 4, 160), (1, 2, 2, 8)), ((2, 4, 8, 130), (1, 2, 4, 5)),
                                      ((2, 4, 8, 258), (1, 2, 4, 3))])
@pytest.mark.parametrize("cin,cout", [(33, 65), (64, 32)])
def test_conv_row_segments(dims, blk, cin, cout):
    print(f"[case] conv row segments {dims} {cin}->{cout}", flush=True)
    S = Solver(dims, dfl_block=blk, sap_block=blk, Ns=1, nkv=1, little_nkv=1, m0=-0.2)
    try:
        torch, V = S.torch, S.V
        S.set_gauge(latgen.make_links(dims, 0.4, 6021))
        rng = np.random.default_rng(cin * 13 + cout + dims[3])
        x, g, zin = (rng.standard_normal((V, c)).astype(np.float32).astype(np.float64) for c in (cin, cout, cin))
        W = (rng.standard_normal((3, 3, 3, 3, cin, cout)) / np.sqrt(81 * cin)).astype(np.float32).astype(np.float64)
        b = rng.standard_normal(cout).astype(np.float32).astype(np.float64)

        def dev(a):
            return torch.tensor(np.ascontiguousarray(a, dtype=np.float32), device="cuda")

        def host(t, c):
            return t.cpu().numpy().astype(np.float64).reshape(c, V).T

        xd, gd, zd, Wd, bd = dev(x.T), dev(g.T), dev(zin.T), dev(W.reshape(81, cin, cout)), dev(b)
        z = torch.empty(cout * V, dtype=torch.float32, device="cuda")
        a = torch.empty_like(z)
        binding.conv4d_forward(S.ctx, xd, cin, Wd, bd, cout, z, a)
        n = 81 * cin + 2
        bound = n * EPS / (1 - n * EPS) * onet.conv4d(np.abs(x), np.abs(W), np.abs(b), dims)
        za = host(z, cout)
        assert np.all(np.abs(za - onet.conv4d(x, W, b, dims)) <= bound)
        assert np.all(np.abs(host(a, cout) - onet.silu(za)) <= 2.0 ** -20 * np.abs(onet.silu(za)) + 1e-30)
        dxr, _, _ = onet.conv4d_backward(x, W, g, dims)
        dxs, _, _ = onet.conv4d_backward(np.abs(x), np.abs(W), np.abs(g), dims)
        n = 81 * cout
        bound = n * EPS / (1 - n * EPS) * dxs
        for z_in, f, df in ((None, 1.0, 0.0), (zd, onet.silu_grad(zin), 2.0 ** -20 * (1 + np.abs(zin)))):
            dW, db, din = (torch.full_like(t, float("nan")) for t in (Wd, bd, xd))
            binding.conv4d_backward(S.ctx, xd, cin, Wd, cout, gd, dW, db, din, z_in)
            assert np.all(np.abs(host(din, cin) - dxr * f) <= bound * np.abs(f) + (np.abs(dxr) + bound) * df)
    finally:
        S.close()
