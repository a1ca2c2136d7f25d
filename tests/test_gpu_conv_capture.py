"""Convolutions captured into a graph after a call of the same or more weights has made room, with eager calls of other
channels between the replays (which must not move what the graph uses). Replays are compared with eager calls."""
import numpy as np
import pytest

from paper_0706_2298_amd import F32, Solver, binding

pytestmark = pytest.mark.gpu


def dev(torch, rng, *shape):
    return torch.tensor(rng.standard_normal(shape), dtype=torch.float32, device="cuda")


# BF16: 32 -> 576 channels take more room for weights than 96 -> 32, less for the input; gradient: 32 -> 320 channels have
# more partial sums than 32 -> 576 (9.1M and 9.0M floats)
@pytest.mark.parametrize("what,other,captured", [("bf16", (32, 576), (96, 32)), ("bf16", (96, 32), (32, 576)),
                                                 ("backward", (32, 576), (32, 320)), ("backward", (32, 320), (32, 576))])
def test_capture_between_other_channels(what, other, captured):
    import torch
    print(f"[case] conv capture {what} {captured} between {other}", flush=True)
    dims = (8, 8, 8, 32) if what == "bf16" else (16, 16, 16, 16)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        S = Solver(dims, Ns=1, nkv=1, little_nkv=1, sap_prec=F32, link_prec=F32)
        try:
            rng = np.random.default_rng(7401)
            V = S.V

            def call(cin, cout, x, W, g, out):
                if what == "bf16":
                    binding.conv4d_forward_bf16(S.ctx, x, cin, W, None, cout, out[0], None)
                else:
                    binding.conv4d_backward(S.ctx, x, cin, W, cout, g, *out, None)

            def args(cin, cout):
                out = [torch.zeros(cout * V, device="cuda")] if what == "bf16" else \
                    [torch.zeros(n, device="cuda") for n in (81 * cin * cout, cout, cin * V)]
                return cin, cout, dev(torch, rng, cin, V), dev(torch, rng, 81, cin, cout) / 30, dev(torch, rng, cout, V), out

            a = args(*other)
            cin, cout, x, W, g, out = args(*captured)
            if 81 * cin * cout > 81 * other[0] * other[1]:
                call(cin, cout, x, W, g, out)  # the weights' room, and the gradient's sums, may need the captured size
            else:
                call(*a)
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                call(cin, cout, x, W, g, out)
            got = []
            for k in range(3):
                for t in out:
                    t.fill_(float("nan"))
                graph.replay()
                torch.cuda.synchronize()
                got.append([t.clone() for t in out])
                call(*a)  # eager work between the replays
                torch.cuda.synchronize()
            want = [torch.full_like(t, float("nan")) for t in out]
            call(cin, cout, x, W, g, want)
            torch.cuda.synchronize()
            for k in range(3):
                for u, v in zip(got[k], want):
                    # the same sums in another order: 8 sqrt(n) roundings of the largest value at n = 2^16 terms
                    assert torch.isfinite(u).all()
                    assert (u - v).abs().max() <= 2048 * 2.0 ** -24 * v.abs().max()
        finally:
            S.close()
