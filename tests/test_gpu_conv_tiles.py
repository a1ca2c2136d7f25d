"""FP32 convolutions of the start-field network on staged site tiles, at lattices
whose tiles start inside a row, cross planes or end short of a tile, with rows
too long for the tiles (vector kernels), and channel counts off the tile sizes.

Tolerance: an FP32 sum of n products in any order is off its exact value by at
most n 2^-24 / (1 - n 2^-24) times the sum of the products' moduli; the bias
and the final sum over partial sums add one rounding each, and the activation
factor silu' a relative error of at most 2^-20.
"""
import numpy as np
import pytest

import latgen
from oracle import net as onet
from paper_0706_2298_amd import Solver, binding

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24


@pytest.mark.parametrize("dims,blk", [((4, 4, 4, 4), (2, 2, 2, 2)), ((4, 4, 6, 10), (2, 2, 3, 5)),
                                      ((4, 2, 4, 48), (2, 1, 2, 4)), ((2, 2, 2, 256), (1, 1, 1, 32))])
@pytest.mark.parametrize("cin,cout", [(33, 65), (64, 32), (5, 40)])
def test_conv_tiles(dims, blk, cin, cout):
    print(f"[case] conv tiles {dims} {cin}->{cout}", flush=True)
    S = Solver(dims, dfl_block=blk, sap_block=blk, Ns=1, nkv=1, little_nkv=1, m0=-0.2)
    try:
        torch = S.torch
        V = S.V
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
        zr = onet.conv4d(x, W, b, dims)
        assert np.all(np.abs(host(z, cout) - zr) <= bound)
        za = host(z, cout)
        assert np.all(np.abs(host(a, cout) - onet.silu(za)) <= 2.0 ** -20 * np.abs(onet.silu(za)) + 1e-30)
        dxr, dWr, dbr = onet.conv4d_backward(x, W, g, dims)
        dxs, dWs, dbs = onet.conv4d_backward(np.abs(x), np.abs(W), np.abs(g), dims)
        for fn in (binding.conv4d_backward, binding.conv4d_backward_noalloc):
            dW, db, din = (torch.full_like(t, float("nan")) for t in (Wd, bd, xd))
            fn(S.ctx, xd, cin, Wd, cout, gd, dW, db, din, zd)
            n = 81 * cout
            f = np.abs(onet.silu_grad(zin))
            assert np.all(np.abs(host(din, cin) - dxr * onet.silu_grad(zin))
                          <= (n * EPS / (1 - n * EPS) + 2.0 ** -20) * dxs * np.maximum(f, 2.0 ** -20))
            n = V + 64  # partial sums of the sites, then their sum
            dWg = dW.cpu().numpy().astype(np.float64).reshape(dWr.shape)
            assert np.all(np.abs(dWg - dWr) <= n * EPS / (1 - n * EPS) * dWs)
            assert np.all(np.abs(db.cpu().numpy() - dbr) <= n * EPS / (1 - n * EPS) * dbs)
    finally:
        S.close()


def bf16_round(a):
    """Round to BF16 (nearest even)."""
    u = np.ascontiguousarray(a, dtype=np.float32).view(np.uint32).astype(np.uint64)
    u = ((u + 0x7FFF + ((u >> 16) & 1)) >> 16) << 16
    return u.astype(np.uint32).view(np.float32).astype(np.float64)


@pytest.mark.parametrize("dims,blk,cin,cout", [
    ((16, 8, 8, 32), (4, 4, 4, 4), 5, 576),      # tiles of 512 sites over two planes, two channel tiles
    ((4, 8, 12, 64), (2, 4, 6, 4), 33, 576),   # tiles that start inside a plane, two input chunks
    ((16, 16, 32, 32), (4, 4, 4, 4), 3, 8),      # tiles of 512 sites, one channel tile
    ((2, 4, 12, 32), (1, 2, 6, 4), 4, 33),       # tiles of 128 sites across planes
    ((2, 2, 4, 1024), (1, 1, 2, 64), 4, 33),     # rows too long for the tiles
])
def test_conv_bf16_tiles(dims, blk, cin, cout):
    # against the FP64 map of the BF16-rounded operands: the products are exact in FP32, so only the
    # FP32 sum of n = 81 cin products and the bias add round
    print(f"[case] conv bf16 tiles {dims} {cin}->{cout}", flush=True)
    S = Solver(dims, dfl_block=blk, sap_block=blk, Ns=1, nkv=1, little_nkv=1, m0=-0.2)
    try:
        torch = S.torch
        V = S.V
        rng = np.random.default_rng(cin * 17 + cout + dims[3])
        x = bf16_round(rng.standard_normal((V, cin)))
        W = bf16_round(rng.standard_normal((3, 3, 3, 3, cin, cout)) / np.sqrt(81 * cin))
        b = rng.standard_normal(cout).astype(np.float32).astype(np.float64)
        xd = torch.tensor(np.ascontiguousarray(x.T), dtype=torch.float32, device="cuda")
        Wd = torch.tensor(W.reshape(81, cin, cout), dtype=torch.float32, device="cuda")
        bd = torch.tensor(b, dtype=torch.float32, device="cuda")
        z = torch.empty(cout * V, dtype=torch.float32, device="cuda")
        binding.conv4d_forward_bf16(S.ctx, xd, cin, Wd, bd, cout, z, None)
        zg = z.cpu().numpy().astype(np.float64).reshape(cout, V).T
        n = 81 * cin + 2
        bound = n * EPS / (1 - n * EPS) * onet.conv4d(np.abs(x), np.abs(W), np.abs(b), dims)
        assert np.all(np.abs(zg - onet.conv4d(x, W, b, dims)) <= bound)
    finally:
        S.close()
