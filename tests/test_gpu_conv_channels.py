"""FP32 convolutions at the lines between the kernels: few input channels (vector kernel on many sites), and 32 or 64
output channels a workgroup. Tolerances as in test_gpu_conv_long_rows."""
import numpy as np
import pytest

import latgen
from oracle import net as onet
from paper_0706_2298_amd import Solver, binding

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24


@pytest.mark.parametrize("dims,blk,cin,cout", [
    ((16, 16, 16, 8), (4, 4, 4, 4), 4, 3), ((16, 16, 16, 8), (4, 4, 4, 4), 5, 7), ((16, 16, 12, 16), (4, 4, 6, 4), 1, 33),
    ((12, 12, 12, 12), (3, 3, 3, 3), 8, 192), ((12, 12, 12, 12), (3, 3, 3, 3), 9, 70),
    ((8, 8, 8, 6), (4, 4, 4, 3), 33, 130), ((4, 4, 4, 4), (2, 2, 2, 2), 7, 65)])
def test_conv_channels(dims, blk, cin, cout):
    print(f"[case] conv channels {dims} {cin}->{cout}", flush=True)
    S = Solver(dims, dfl_block=blk, sap_block=blk, Ns=1, nkv=1, little_nkv=1, m0=-0.2)
    try:
        torch, V = S.torch, S.V
        S.set_gauge(latgen.make_links(dims, 0.4, 7601))
        rng = np.random.default_rng(cin * 7 + cout)
        x, g = (rng.standard_normal((V, c)).astype(np.float32).astype(np.float64) for c in (cin, cout))
        W = (rng.standard_normal((3, 3, 3, 3, cin, cout)) / np.sqrt(81 * cin)).astype(np.float32).astype(np.float64)
        b = rng.standard_normal(cout).astype(np.float32).astype(np.float64)

        def dev(a):
            return torch.tensor(np.ascontiguousarray(a, dtype=np.float32), device="cuda")

        def host(t, c):
            return t.cpu().numpy().astype(np.float64).reshape(c, V).T

        xd, gd, Wd, bd = dev(x.T), dev(g.T), dev(W.reshape(81, cin, cout)), dev(b)
        z = torch.empty(cout * V, dtype=torch.float32, device="cuda")
        a = torch.empty_like(z)
        binding.conv4d_forward(S.ctx, xd, cin, Wd, bd, cout, z, a)
        n = 81 * cin + 2
        za = host(z, cout)
        bound = n * EPS / (1 - n * EPS) * onet.conv4d(np.abs(x), np.abs(W), np.abs(b), dims)
        assert np.all(np.abs(za - onet.conv4d(x, W, b, dims)) <= bound)
        assert np.all(np.abs(host(a, cout) - onet.silu(za)) <= 2.0 ** -20 * np.abs(onet.silu(za)) + 1e-30)
        # the input gradient is the map from cout to cin channels: W with its channels and the lattice reversed
        dW, db, din = torch.empty_like(Wd), torch.empty_like(bd), torch.full_like(xd, float("nan"))
        binding.conv4d_backward(S.ctx, xd, cin, Wd, cout, gd, dW, db, din, None)
        Wt = np.flip(W, axis=(0, 1, 2, 3)).swapaxes(4, 5)
        n = 81 * cout
        bound = n * EPS / (1 - n * EPS) * onet.conv4d(np.abs(g), np.abs(Wt), np.zeros(cin), dims)
        assert np.all(np.abs(host(din, cin) - onet.conv4d(g, Wt, np.zeros(cin), dims)) <= bound)
    finally:
        S.close()
