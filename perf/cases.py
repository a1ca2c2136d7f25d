"""The work whose speed is measured: calls of the solver, of its parts and of the start-field network.

``listed()`` holds the named cases, ``draw()`` gives more of the same ranges, ``prepare()`` makes what a program
has in hand before the call, ``run()`` is one pass through the public entry points (``Solver``, ``StartFieldNet``
and the C names in ``binding``), ``work()`` counts the bytes and operations a pass cannot do without, and
``exact()`` computes the same outputs in 64 bits with plain torch.

A case is a dict of plain values. Lattices and blocks are texts such as "48x24x24x24" (x0 is time). ``improved``
is the operator of the production ensembles: clover term with csw = 1.90952 and antiperiodic time; otherwise the
plain Wilson operator, periodic. ``mixed`` is FP64 GCR with FP32 Schwarz sweeps and FP32 inner little solves;
otherwise everything is FP64. Links are random SU(3) matrices exp(i eps H) of the roughness eps, independent per
site, as everywhere in this repository.
"""
from __future__ import annotations

import math

import torch

from paper_0706_2298_amd import BF16, F32, F64, PROJ_PL, Solver, binding
from paper_0706_2298_amd.learned import CHANNELS, StartFieldNet, make_targets

CSW = 1.90952
NCY, NMR, STEPS = 5, 4, 3      # Schwarz cycles, minimal-residual steps, inverse-iteration steps (the defaults)
D_FLOPS = 1368                 # Wilson operator per site and field
LINK_BYTES = {"f64": 384, "f32": 192, "bf16": 96}


def listed():
    return [
        # one application of D on the smallest lattice in use: launch latency
        dict(name="dirac f64 8^4", kind="dirac", dims="8x8x8x8", prec="f64", nrhs=1, improved=False),
        # the operator of the production ensembles on their smaller lattice, as in every residual of an FP64 GCR
        dict(name="dirac f64 improved 48x24^3", kind="dirac", dims="48x24x24x24", prec="f64", nrhs=1, improved=True),
        # the twelve columns of a point source at once, in FP32
        dict(name="dirac f32 12x 48x24^3", kind="dirac", dims="48x24x24x24", prec="f32", nrhs=12, improved=False),
        # the preconditioner of an all-FP64 solve with the production operator and its 8 x 4^3 Schwarz blocks
        dict(name="sap f64 improved 32x16^3", kind="sap", dims="32x16x16x16", sap_block="8x4x4x4", nrhs=1,
             improved=True),
        # the deflation projector at full accuracy, as at the restarts of a deflated solve
        dict(name="project f64 32x16^3", kind="project", dims="32x16x16x16", Ns=20, nrhs=1, improved=False),
        # subspace generation with the default (FP64) parameters
        dict(name="setup f64 16^4", kind="setup", dims="16x16x16x16", Ns=20, improved=False),
        # the smallest whole solve, all FP64, subspace in hand
        dict(name="solve f64 8^4", kind="solve", dims="8x8x8x8", Ns=20, nrhs=1, mixed=False, improved=False,
             eps=0.4, m0=-0.2, with_setup=False, graphs=False),
        # one propagator column of the production operator in mixed precision, subspace in hand
        dict(name="solve improved 48x24^3", kind="solve", dims="48x24x24x24", Ns=20, nrhs=1, mixed=True,
             improved=True, eps=0.4, m0=-0.2, with_setup=False, graphs=False),
        # twelve sources in one batch with graph replay, subspace in hand
        dict(name="solve batch 12x 48x24^3", kind="solve", dims="48x24x24x24", Ns=24, nrhs=12, mixed=True,
             improved=False, eps=0.4, m0=-0.3, with_setup=False, graphs=True),
        # a gauge field of its own near the critical mass: one subspace, one solve, on the largest lattice
        dict(name="setup+solve 64x32^3", kind="solve", dims="64x32x32x32", Ns=24, nrhs=1, mixed=True,
             improved=False, eps=0.5, m0=-0.56, with_setup=True, graphs=False),
        # the gradient of one training field of the start-field network (forward, loss, backward)
        dict(name="net gradient 16^4", kind="net", dims="16x16x16x16", Ns=24, targets=24),
        # its largest layer at inference on the largest lattice, BF16 operands
        dict(name="conv bf16 64x32^3", kind="conv", dims="64x32x32x32", cin=32, cout=576, prec="bf16",
             backward=False),
    ]


# ------------------------------------------------------------------ drawn cases

def _ext(text):
    return tuple(int(v) for v in text.split("x"))


def _text(v):
    return "x".join(str(k) for k in v)


def _volume(dims):
    return math.prod(dims)


def _draw_block(rng, dims, most):
    """Block extents that divide the lattice into an even number of blocks: 4^4 or 8 x 4^3 where they fit, as in
    nearly all use, or ragged ones."""
    if all(d % 8 == 0 for d in dims) and rng.random() < 0.9:
        return (8, 4, 4, 4) if dims[0] % 16 == 0 and most >= 512 and rng.random() < 0.25 else (4, 4, 4, 4)
    while True:
        b = tuple(rng.choice([k for k in range(2, 9) if d % (2 * k) == 0]) for d in dims)
        if 48 <= _volume(b) <= most:
            return b


def _draw_dims(rng, lo, hi):
    """Lattice T x L^2 x L' with lo..hi sites, spread over the logarithm of the volume; a quarter of them with
    extents (12, 20) that 4^4 blocks do not fit."""
    target = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    space, time = [8, 16, 24, 32], [8, 16, 24, 32, 40, 48, 64]
    if rng.random() < 0.25:
        space, time = space + [12, 20, 12, 20], time + [12, 20]
    while True:
        a, b, t = rng.choice(space), rng.choice(space), rng.choice(time)
        v = t * a * a * b
        if lo <= v <= hi and target / 2 <= v <= target * 2 and v % 64 == 0:
            return (t, a, a, b)


def draw(rng):
    kind = rng.choice(["dirac"] * 4 + ["sap"] * 2 + ["project"] * 2 + ["setup"] * 2 + ["solve"] * 4 + ["net"] * 2
                      + ["conv"] * 3)
    case = dict(kind=kind)
    if kind == "dirac":
        nrhs = rng.choice([1, 1, 1, 2, 3, 5, 12])
        dims = _draw_dims(rng, 4096, 2000000 // max(1, nrhs // 2))
        case.update(dims=_text(dims), prec=rng.choice(["f64", "f32", "bf16"]), nrhs=nrhs,
                    improved=rng.random() < 0.4, block=_text(_draw_block(rng, dims, 512)))
    elif kind == "sap":
        dims = _draw_dims(rng, 4096, 300000)
        b = _text(_draw_block(rng, dims, 512))
        case.update(dims=_text(dims), nrhs=rng.choice([1, 1, 2, 3]), improved=rng.random() < 0.5, block=b,
                    sap_block=b)
    elif kind == "project":
        dims = _draw_dims(rng, 4096, 300000)
        case.update(dims=_text(dims), Ns=rng.choice([8, 13, 20, 24]), nrhs=rng.choice([1, 1, 2, 5]),
                    improved=rng.random() < 0.4, block=_text(_draw_block(rng, dims, 512)))
    elif kind == "setup":
        dims = _draw_dims(rng, 4096, 140000)
        b = _text(_draw_block(rng, dims, 512))
        case.update(dims=_text(dims), Ns=rng.choice([8, 13, 20, 24]), improved=rng.random() < 0.5, block=b,
                    sap_block=b)
    elif kind == "solve":
        nrhs = rng.choice([1, 1, 1, 2, 3, 6])
        dims = _draw_dims(rng, 4096, 600000 // nrhs)
        improved = rng.random() < 0.4
        b = _text(_draw_block(rng, dims, 320))
        case.update(dims=_text(dims), Ns=rng.choice([12, 20, 24]), nrhs=nrhs, mixed=rng.random() < 0.7,
                    improved=improved, eps=0.4, m0=-0.2 if improved else rng.choice([-0.2, -0.25, -0.3]),
                    with_setup=rng.random() < 0.3, graphs=nrhs > 1 and rng.random() < 0.5, block=b, sap_block=b)
    elif kind == "net":
        dims = rng.choice([(8, 8, 8, 8), (16, 8, 8, 16), (8, 8, 16, 24), (16, 16, 16, 8), (8, 8, 8, 32),
                           (16, 16, 16, 16)])
        case.update(dims=_text(dims), Ns=rng.choice([8, 12, 20, 24]), targets=rng.choice([8, 16, 24]))
    else:
        prec = rng.choice(["f32", "bf16"])
        dims = (rng.choice([4, 8, 16, 32]), rng.choice([8, 16, 24]), rng.choice([8, 16, 24, 32]),
                rng.choice([32, 64] if prec == "bf16" else [8, 16, 24, 32]))
        case.update(dims=_text(dims), cin=rng.choice([32, 32, 37, 96]), cout=rng.choice([32, 32, 48, 288, 576]),
                    prec=prec, backward=prec == "f32" and _volume(dims) <= 70000 and rng.random() < 0.6)
    return case


# ------------------------------------------------------------------ inputs

def _gen(seed, what):
    return torch.Generator(device="cuda").manual_seed(1000003 * what + int(seed))


def _mul3(a, b):
    """Product of two stacks of 3 x 3 matrices."""
    r = a[..., :, 0:1] * b[..., 0:1, :]
    for k in (1, 2):
        r += a[..., :, k:k + 1] * b[..., k:k + 1, :]
    return r


def _gauge(dims, eps, seed):
    """U = exp(i eps H), H = sum_a h_a lambda_a / 2 with standard normal h_a: (V, 4, 3, 3) complex128."""
    h = torch.randn(_volume(dims), 4, 8, generator=_gen(seed, 1), dtype=torch.float64, device="cuda") * (eps / 2)
    A = torch.zeros(h.shape[:2] + (3, 3), dtype=torch.complex128, device="cuda")
    for k, (i, j) in enumerate([(0, 1), (0, 2), (1, 2)]):
        re, im = h[..., (0, 3, 5)[k]], h[..., (1, 4, 6)[k]]
        A[..., i, j] = torch.complex(im, re)       # i (re - i im)
        A[..., j, i] = torch.complex(-im, re)
    d3, d8 = h[..., 2], h[..., 7] / math.sqrt(3)
    for k, d in enumerate([d3 + d8, d8 - d3, -2 * d8]):
        A[..., k, k] = 1j * d
    del h
    A /= 16
    eye = torch.eye(3, dtype=torch.complex128, device="cuda")
    U = A / 12 + eye
    for k in range(11, 0, -1):  # Taylor series of exp(A / 16), then four squarings
        U = _mul3(A, U)
        U /= k
        U += eye
    for _ in range(4):
        U = _mul3(U, U)
    return U


def _fields(dims, n, seed, what):
    """n Gaussian quark fields, canonical (n, V, 12) complex128, real and imaginary parts of unit variance."""
    return torch.randn(n, _volume(dims), 12, generator=_gen(seed, what), dtype=torch.complex128,
                       device="cuda") * math.sqrt(2.0)


def _planes(n, c, seed, what, scale=1.0):
    return torch.randn(c, n, generator=_gen(seed, what), dtype=torch.float32, device="cuda") * scale


def _weights(channels, seed):
    """Initial weights of 3^4 convolutions, variance 1 / (81 Cin), and small biases."""
    out = []
    for k, (ci, co) in enumerate(zip(channels[:-1], channels[1:])):
        out.append((_planes(co, 81 * ci, seed, 20 + k, 1.0 / math.sqrt(81 * ci)).reshape(81, ci, co),
                    _planes(co, 1, seed, 40 + k, 0.01).reshape(co)))
    return out


def _blocks(case):
    b = _ext(case.get("block", "4x4x4x4"))
    return b, _ext(case["sap_block"]) if "sap_block" in case else b


def _mass(case):
    return case.get("m0", -0.2 if case.get("improved") else -0.3)


def _eps(case):
    return case.get("eps", 0.5 if case["kind"] == "net" else 0.4)


def _channels(case):
    return CHANNELS[:-1] + (24 * case["Ns"],)


def _solver(case, **kw):
    dims = _ext(case["dims"])
    b, sb = _blocks(case)
    m0 = _mass(case)
    p = dict(dfl_block=b, sap_block=sb, m0=m0, m0_setup=m0, ncy=NCY, nmr=NMR, n_inviter=STEPS,
             nrhs_max=case.get("nrhs", 1), Ns=case.get("Ns", 1))
    if case.get("improved"):
        p.update(csw=CSW, antiperiodic=1)
    p.update(kw)
    return Solver(dims, **p)


def prepare(case, seed):
    dims, kind = _ext(case["dims"]), case["kind"]
    st = dict(case)
    if kind == "conv":
        ci, co, V = case["cin"], case["cout"], _volume(dims)
        b = tuple(4 if d % 8 == 0 else 2 for d in dims)
        st["S"] = _solver(dict(case, block=_text(b)), Ns=1, nkv=1, little_nkv=1, sap_prec=F32, link_prec=F32)
        st["x"] = _planes(V, ci, seed, 5)
        st["W"], st["b"] = _weights((ci, co), seed)[0]
        if case["backward"]:
            st["g"], st["z_in"] = _planes(V, co, seed, 6), _planes(V, ci, seed, 7)
        return st
    if kind == "dirac":
        lp = dict(f64=F64, f32=F32, bf16=BF16)[case["prec"]]
        S = _solver(case, nkv=1, little_nkv=1, link_prec=lp, sap_prec=F64 if lp == F64 else F32)
        S.set_gauge(_gauge(dims, _eps(case), seed))
        st.update(S=S, psi=S.pack(_fields(dims, case["nrhs"], seed, 2), prec=F64 if lp == F64 else F32))
    elif kind == "sap":
        S = _solver(case, nkv=1, little_nkv=1)
        S.set_gauge(_gauge(dims, _eps(case), seed))
        st.update(S=S, rho=S.pack(_fields(dims, case["nrhs"], seed, 2)))
    elif kind in ("project", "setup", "solve"):
        mixed = case.get("mixed", False)
        S = _solver(case, **(dict(sap_prec=F32, link_prec=F32, little_prec=F32) if mixed else {}))
        S.set_gauge(_gauge(dims, _eps(case), seed))
        init = S.pack(_fields(dims, case["Ns"], seed, 3))
        if kind == "setup" or case.get("with_setup"):
            st["init"] = init
        else:
            S.setup(init)
        if case.get("graphs"):
            S.use_graphs(True)
        st["S"] = S
        if kind != "setup":
            st["eta"] = S.pack(_fields(dims, case["nrhs"], seed, 2))
    else:
        m0 = -0.56  # near the critical mass of the training fields, as the networks are trained
        S = _solver(dict(case, m0=m0), Ns=max(case["Ns"], case["targets"]), nkv=1, little_nkv=1)
        S.set_gauge(_gauge(dims, _eps(case), seed))
        st.update(S=S, targets_f=make_targets(S, S.pack(_fields(dims, case["targets"], seed, 3)), STEPS))
        ch = _channels(case)
        w = [(W.cpu().numpy().reshape(3, 3, 3, 3, *W.shape[1:]), b.cpu().numpy()) for W, b in _weights(ch, seed)]
        st.update(net=StartFieldNet(S, w, ch), noise=_planes(24, _volume(dims), seed, 4))
    return st


# ------------------------------------------------------------------ one pass

def run(st):
    kind, S = st["kind"], st["S"]
    if kind == "dirac":
        return S.dirac(st["psi"], prec=F64 if st["prec"] == "f64" else F32)
    if kind == "sap":
        return S.sap(st["rho"])
    if kind == "project":
        return S.project(PROJ_PL, st["eta"])
    if kind == "setup":
        S.setup(st["init"])
        A = torch.empty(S.Nb * 9 * S.Ns * S.Ns, dtype=torch.complex128, device="cuda")
        binding.dfl_get_little(S.ctx, A)
        return {"basis": S.basis(), "little": A}
    if kind == "solve":
        if st["with_setup"]:
            S.setup(st["init"])
        return S.solve(st["eta"])[0]
    if kind == "net":
        fields = st["net"].forward(st["noise"])
        loss, grad = st["net"].loss(fields, st["targets_f"], st["targets"])
        return {"loss": loss, "grads": st["net"].backward(grad)}
    ci, co = st["cin"], st["cout"]
    z = torch.empty(co, S.V, dtype=torch.float32, device="cuda")
    if st["prec"] == "bf16":
        binding.conv4d_forward_bf16(S.ctx, st["x"], ci, st["W"], st["b"], co, z)
        return {"z": z}
    act = torch.empty_like(z)
    binding.conv4d_forward(S.ctx, st["x"], ci, st["W"], st["b"], co, z, act)
    out = {"z": z, "act": act}
    if st["backward"]:
        out.update(dW=torch.empty_like(st["W"]), db=torch.empty_like(st["b"]), din=torch.empty_like(st["x"]))
        binding.conv4d_backward(S.ctx, st["x"], ci, st["W"], co, st["g"], out["dW"], out["db"], out["din"],
                                st["z_in"])
    return out


# ------------------------------------------------------------------ work

def _sap_flops(V, n):
    """ncy cycles over all sites: the residue, nmr steps of the block operator with their vector updates."""
    return n * V * NCY * (D_FLOPS + 24 + NMR * (D_FLOPS + 336) + 24)


def work(case):
    dims, kind = _ext(case["dims"]), case["kind"]
    V, n, Ns = _volume(dims), case.get("nrhs", 1), case.get("Ns", 1)
    f64 = 192 * V  # one FP64 quark field; an FP32 one has half
    op = D_FLOPS + (552 if case.get("improved") else 0)
    if kind == "conv":
        ci, co = case["cin"], case["cout"]
        io, taps = 4 * V * (ci + co), 4 * 81 * ci * co
        f = 2.0 * 81 * ci * co * V
        if case["prec"] == "bf16":
            return dict(bytes=io + taps, flops=f)
        back = dict(bytes=4 * V * (3 * ci + co) + 2 * taps, flops=2 * f)
        return dict(bytes=io + 4 * V * co + taps + (back["bytes"] if case["backward"] else 0),
                    flops=f + (back["flops"] if case["backward"] else 0))
    if kind == "net":
        ch = _channels(case)
        f = sum(2.0 * 81 * a * b * V for a, b in zip(ch[:-1], ch[1:]))
        first = 2.0 * 81 * ch[0] * ch[1] * V  # no gradient with respect to the features
        K = case["targets"]
        return dict(bytes=4 * V * (96 + 2 * sum(ch[1:])) * 2 + f64 * (2 * Ns + K),
                    flops=3 * f - first + 8 * 12 * V * (Ns * (Ns + 1) / 2 + 3 * Ns * K))
    links = V * LINK_BYTES[case.get("prec", "f64")]
    if case.get("improved"):
        links += V * (576 if case.get("prec", "f64") == "f64" else 288)
    if kind == "dirac":
        return dict(bytes=links + 2 * n * (f64 if case["prec"] == "f64" else f64 // 2), flops=op * V * n)
    if kind == "sap":
        return dict(bytes=links + 2 * n * f64, flops=_sap_flops(V, n))
    if kind == "project":
        return dict(bytes=links + (2 * n + Ns) * f64, flops=n * V * (op + 2 * 96 * Ns))
    setup = dict(bytes=links + 2 * Ns * f64,
                 flops=STEPS * _sap_flops(V, Ns) + 96.0 * V * Ns * Ns * 2 + op * V * Ns)
    if kind == "setup":
        return setup
    # a solve: a dozen outer steps, each with one preconditioner, two operators and a projector; the links, the
    # basis, the source and the solution are read or written once
    solve = dict(bytes=links + (Ns + 2 * n) * f64, flops=12 * n * (_sap_flops(V, 1) + V * (2 * op + 2 * 96 * Ns)))
    if case["with_setup"]:
        return {k: setup[k] + solve[k] for k in setup}
    return solve


# ------------------------------------------------------------------ the same in 64 bits

# rows of gamma_mu: (gamma_mu chi)_s = factor[s] chi_{spin[s]}
_GAMMA = [((2, 3, 0, 1), (-1, -1, -1, -1)), ((3, 2, 1, 0), (-1j, -1j, 1j, 1j)),
          ((3, 2, 1, 0), (-1, 1, 1, -1)), ((2, 3, 0, 1), (-1j, 1j, 1j, -1j))]


class _Reference:
    """The operator and the deflation of one gauge field; fields are (n, L0, L1, L2, L3, 4, 3) complex128."""

    def __init__(self, case, seed):
        self.dims = _ext(case["dims"])
        self.b, self.sb = _blocks(case)
        self.m0 = _mass(case)
        self.anti = bool(case.get("improved"))
        U = _gauge(self.dims, _eps(case), seed).reshape(*self.dims, 4, 3, 3)
        self.U = [U[..., mu, :, :].contiguous() for mu in range(4)]
        self.C = self._clover() if self.anti else None

    def fields(self, n, seed, what, dtype=None):
        f = _fields(self.dims, n, seed, what)
        if dtype is not None:
            f = f.to(dtype).to(torch.complex128)
        return f.reshape(n, *self.dims, 4, 3)

    def _clover(self):
        dag = lambda m: m.mH  # noqa: E731
        sh = lambda m, mu, s: torch.roll(m, -s, dims=mu)  # noqa: E731  value at x + s mu
        g = torch.zeros(4, 4, 4, dtype=torch.complex128, device="cuda")
        for mu, (spin, fac) in enumerate(_GAMMA):
            for s in range(4):
                g[mu, s, spin[s]] = fac[s]
        C = torch.zeros(*self.dims, 4, 3, 4, 3, dtype=torch.complex128, device="cuda")
        for mu in range(4):
            for nu in range(mu + 1, 4):
                a, b = self.U[mu], self.U[nu]
                am, bm = sh(a, mu, -1), sh(b, nu, -1)
                Q = _mul3(_mul3(a, sh(b, mu, 1)), _mul3(dag(sh(a, nu, 1)), dag(b)))
                Q += _mul3(_mul3(b, dag(sh(am, nu, 1))), _mul3(dag(sh(b, mu, -1)), am))
                Q += _mul3(_mul3(dag(am), dag(sh(bm, mu, -1))), _mul3(sh(am, nu, -1), bm))
                Q += _mul3(_mul3(dag(bm), sh(a, nu, -1)), _mul3(sh(bm, mu, 1), dag(a)))
                F = (Q - dag(Q)) / 8
                sigma = 0.5j * (g[mu] @ g[nu] - g[nu] @ g[mu]) * (0.5j * CSW)
                for s in range(4):
                    for t in range(4):
                        if sigma[s, t] != 0:
                            C[..., s, :, t, :] += sigma[s, t] * F
        return C.reshape(*self.dims, 12, 12)

    def hop(self, f, mu, step):
        """(1 -+ gamma_mu) U psi(x +- mu), without the factor -1/2."""
        u = self.U[mu] if step > 0 else self.U[mu].mH
        if step > 0:
            f = torch.roll(f, -1, dims=1 + mu)
        v = u[..., None, :, 0] * f[..., :, None, 0]
        for k in (1, 2):
            v += u[..., None, :, k] * f[..., :, None, k]
        if step < 0:
            v = torch.roll(v, 1, dims=1 + mu)
        if mu == 0 and self.anti:
            v[:, -1 if step > 0 else 0] *= -1
        spin, fac = _GAMMA[mu]
        fac = torch.tensor(fac, dtype=torch.complex128, device="cuda")[:, None]
        return v - step * fac * v[..., spin, :]

    def inside(self, mu, step, b):
        """1 where the hop stays in its block of extents b."""
        x = torch.arange(self.dims[mu], device="cuda") % b[mu]
        m = (x < b[mu] - 1) if step > 0 else (x > 0)
        return m.double().reshape([1] + [-1 if k == mu else 1 for k in range(4)] + [1, 1])

    def D(self, f, block=None):
        """D f, or the operator restricted to the blocks of extents `block`."""
        out = (4 + self.m0) * f
        if self.C is not None:
            out += (self.C * f.reshape(*f.shape[:-2], 1, 12)).sum(-1).reshape(f.shape)
        for mu in range(4):
            for step in (1, -1):
                h = self.hop(f, mu, step)
                out -= 0.5 * (h if block is None else h * self.inside(mu, step, block))
        return out

    def blocked(self, f, b):
        """(n, L0 .. L3, ...) as (n, n0, b0, n1, b1, n2, b2, n3, b3, ...)."""
        s = [f.shape[0]]
        for d, k in zip(self.dims, b):
            s += [d // k, k]
        return f.reshape(*s, *f.shape[5:])

    def sap(self, rho):
        psi = torch.zeros_like(rho)
        grid = [torch.arange(d, device="cuda") // k for d, k in zip(self.dims, self.sb)]
        par = sum(torch.meshgrid(*grid, indexing="ij")) % 2
        dot = lambda x, y: self.blocked((x.conj() * y).sum((-2, -1)), self.sb).sum(  # noqa: E731
            (2, 4, 6, 8), keepdim=True)
        for _ in range(NCY):
            for colour in (0, 1):
                r = (rho - self.D(psi)) * (par == colour)[None, ..., None, None]
                x = torch.zeros_like(r)
                for _ in range(NMR):
                    q = self.D(r, self.sb)
                    qq = dot(q, q)
                    a = torch.where(qq.real > 0, dot(q, r) / torch.where(qq.real > 0, qq, torch.ones_like(qq)),
                                    torch.zeros_like(qq))
                    a = a.expand(self.blocked(r[..., 0, 0], self.sb).shape).reshape(r.shape[:-2])[..., None, None]
                    x += a * r
                    r = r - a * q
                psi = psi + x
        return psi

    def norm(self, f):
        return f.reshape(f.shape[0], -1).norm(dim=1).reshape(-1, 1, 1, 1, 1, 1, 1)

    def inverse_iteration(self, f):
        f = f / self.norm(f)
        for _ in range(STEPS):
            f = self.sap(f)
            f = f / self.norm(f)
        return f

    # deflation: the basis as (blocks, entries of a block, Ns)
    def to_blocks(self, f):
        g = self.blocked(f, self.b).permute(1, 3, 5, 7, 2, 4, 6, 8, 9, 10, 0)
        return g.reshape(_volume(self.dims) // _volume(self.b), 12 * _volume(self.b), f.shape[0])

    def from_blocks(self, g):
        nb = [d // k for d, k in zip(self.dims, self.b)]
        n = g.shape[-1]
        g = g.reshape(*nb, *self.b, 4, 3, n).permute(10, 0, 4, 1, 5, 2, 6, 3, 7, 8, 9)
        return g.reshape(n, *self.dims, 4, 3)

    def subspace(self, init):
        P = self.to_blocks(self.inverse_iteration(init))
        for _ in range(3):  # Cholesky QR: the same basis as Gram-Schmidt in the order of the fields
            L = torch.linalg.cholesky(torch.bmm(P.mH.contiguous(), P))
            P = torch.linalg.solve_triangular(L, P.mH.contiguous(), upper=False).mH.contiguous()
        self.P, self.PH = P, P.mH.contiguous()

    def little(self):
        """(blocks, 9, Ns, Ns): the block itself, then the terms from block + mu and block - mu."""
        f = self.from_blocks(self.P)
        out = [torch.bmm(self.PH, self.to_blocks(self.D(f, self.b)))]
        for mu in range(4):
            for step in (1, -1):
                h = self.hop(f, mu, step) * (1 - self.inside(mu, step, self.b)) * -0.5
                out.append(torch.bmm(self.PH, self.to_blocks(h)))
        return torch.stack(out, dim=1)

    def coarse(self, y):
        """Phi A^-1 Phi^+ y."""
        up = lambda v: self.from_blocks(torch.bmm(self.P, v))      # noqa: E731
        down = lambda f: torch.bmm(self.PH, self.to_blocks(f))    # noqa: E731
        flat = lambda v: v.permute(2, 0, 1).reshape(v.shape[2], -1)  # noqa: E731
        w = down(y)
        shape = (w.shape[0], w.shape[1])
        back = lambda v: v.reshape(-1, *shape).permute(1, 2, 0).contiguous()  # noqa: E731
        return up(back(_solve(lambda v: flat(down(self.D(up(back(v))))), flat(w), 1e-14)))

    def inverse(self, eta):
        flat = lambda f: f.reshape(f.shape[0], -1)  # noqa: E731
        return _solve(lambda v: flat(self.D(v.reshape(eta.shape))), flat(eta), 1e-14).reshape(eta.shape)

    def native(self, f):
        """In the library's order: sites by blocks, 64-site tiles of 12 planes."""
        n, v = f.shape[0], _volume(self.dims)
        g = self.blocked(f, self.b).permute(0, 1, 3, 5, 7, 2, 4, 6, 8, 9, 10)
        return g.reshape(n, v // 64, 64, 12).permute(0, 1, 3, 2).reshape(-1)


def _solve(op, b, tol):
    """op(x) = b for every row by BiCGstab, restarted from the true residue until it is below tol."""
    dot = lambda u, v: (u.conj() * v).sum(1, keepdim=True)  # noqa: E731
    div = lambda u, v: torch.where(v != 0, u / torch.where(v != 0, v, torch.ones_like(v)),  # noqa: E731
                                   torch.zeros_like(u))
    x, bn = torch.zeros_like(b), b.norm(dim=1).clamp_min(1e-300)
    last = math.inf
    for _ in range(8):
        r = b - op(x)
        now = float((r.norm(dim=1) / bn).max())
        if now < tol or now > 0.5 * last:
            break
        last = now
        r0, p, rho = r.clone(), r.clone(), dot(r, r)
        for it in range(3000):
            v = op(p)
            a = div(rho, dot(r0, v))
            s = r - a * v
            t = op(s)
            w = div(dot(t, s), dot(t, t))
            x = x + a * p + w * s
            r = s - w * t
            if it % 8 == 7 and float((r.norm(dim=1) / bn).max()) < max(tol, 1e-6 * now):
                break
            new = dot(r0, r)
            p = r + div(new, rho) * div(a, w) * (p - w * v)
            rho = new
    return x


def _conv(x, W, b, dims):
    """Periodic 3^4 convolution of planes (Cin, V) in 64 bits."""
    x = x.reshape(-1, *dims)
    z = torch.zeros(W.shape[2], _volume(dims), dtype=torch.float64, device="cuda")
    if b is not None:
        z = z + b[:, None]
    inplace = not (x.requires_grad or W.requires_grad)
    for t in range(81):
        o = [t // 27 - 1, t // 9 % 3 - 1, t // 3 % 3 - 1, t % 3 - 1]
        xt = torch.roll(x, [-k for k in o], dims=(1, 2, 3, 4)).reshape(x.shape[0], -1)
        z = z.addmm_(W[t].t(), xt) if inplace else torch.addmm(z, W[t].t(), xt)
    return z


def _silu_grad(z):
    s = torch.sigmoid(z)
    return s * (1 + z * (1 - s))


def _exact_conv(case, seed):
    dims, ci, co, V = _ext(case["dims"]), case["cin"], case["cout"], _volume(_ext(case["dims"]))
    x = _planes(V, ci, seed, 5).double()
    W, b = (t.double() for t in _weights((ci, co), seed)[0])
    z = _conv(x, W, b, dims)
    if case["prec"] == "bf16":
        return {"z": z}
    out = {"z": z, "act": torch.nn.functional.silu(z)}
    if case["backward"]:
        g, z_in = _planes(V, co, seed, 6).double(), _planes(V, ci, seed, 7).double()
        out["db"] = g.sum(1)
        # the input gradient is the convolution of g with the reflected, transposed taps
        out["din"] = _conv(g, W.flip(0).transpose(1, 2).contiguous(), None, dims) * _silu_grad(z_in)
        x4, dW = x.reshape(-1, *dims), []
        for t in range(81):
            o = [t // 27 - 1, t // 9 % 3 - 1, t // 3 % 3 - 1, t % 3 - 1]
            dW.append(torch.roll(x4, [-k for k in o], dims=(1, 2, 3, 4)).reshape(ci, -1) @ g.t())
        out["dW"] = torch.stack(dW)
    return out


def _exact_net(case, seed):
    R = _Reference(dict(case, m0=-0.56), seed)
    dims, V, Ns, K = R.dims, _volume(R.dims), case["Ns"], case["targets"]
    T = R.to_blocks(R.inverse_iteration(R.fields(K, seed, 3)))
    links = torch.stack(R.U, dim=4).reshape(V, 36)
    x = torch.cat([torch.view_as_real(links).reshape(V, 72).float().double().t(),
                   _planes(24, V, seed, 4).double().t()]).contiguous()
    params = [tuple(t.double().requires_grad_() for t in wb) for wb in _weights(_channels(case), seed)]
    for k, (W, b) in enumerate(params):
        x = _conv(x, W, b, dims)
        if k < len(params) - 1:
            x = torch.nn.functional.silu(x)
    f = torch.view_as_complex(x.reshape(Ns, 12, 2, V).permute(0, 3, 1, 2).contiguous())
    P = R.to_blocks(f.reshape(Ns, *dims, 4, 3))
    PH = P.mH.contiguous()
    proj = torch.bmm(P, torch.linalg.solve(torch.bmm(PH, P), torch.bmm(PH, T)))
    loss = ((T - proj).abs().square().sum((0, 1)) / T.abs().square().sum((0, 1))).mean()
    loss.backward()
    return {"loss": float(loss), "grads": [(W.grad, b.grad) for W, b in params]}


def exact(case, seed):
    """What run() returns for these inputs, in 64 bits; None for the largest solves (minutes in plain torch)."""
    kind = case["kind"]
    if kind == "conv":
        return _exact_conv(case, seed)
    if kind == "net":
        return _exact_net(case, seed)
    n = case.get("nrhs", 1)
    if kind == "solve" and _volume(_ext(case["dims"])) * n > 300000:
        return None
    R = _Reference(case, seed)
    if kind == "dirac":
        f = R.fields(n, seed, 2, None if case["prec"] == "f64" else torch.complex64)
        return torch.cat([R.native(R.D(f[k:k + 1])) for k in range(n)])
    if kind == "sap":
        return R.native(R.sap(R.fields(n, seed, 2)))
    if kind == "solve":
        return R.native(R.inverse(R.fields(n, seed, 2)))
    R.subspace(R.fields(case["Ns"], seed, 3))
    if kind == "setup":
        return {"basis": R.native(R.from_blocks(R.P)), "little": R.little().reshape(-1)}
    eta = R.fields(n, seed, 2)
    return R.native(eta - R.D(R.coarse(eta)))
