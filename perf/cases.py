"""Performance cases of the improved-staggered solver: the work its users call it for, through
the Python binding's entry points, from one 8^4 hopping term to the nine-shift solve on
32^3 x 48.

Each case is a dict of plain values.  `kind` names the path, x, y, z, t the lattice extents; the
fields and sources are synthetic (drawn from the seed on the GPU), with the recipe of the
`ksinputs` package: SU(3) thin links near the identity, a noisy fat link, the three-link Naik
product, staggered phases and the antiperiodic time boundary folded in.

Results come back in the precision the path works in: an FP32 field or network as complex64, a
binary16 field or the matrix-core network (binary16 activations) as float16 (re, im) pairs, and
everything that is FP64 or refined to an FP64 residual as complex128.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1611_00728_amd as ks

PREC = {"f64": ks.F64, "f32": ks.F32, "f16": ks.F16}
TOL = 1e-12                     # true relative residual of every solve
LEVEL1 = (1.0 / 8, 1.0 / 16, 1.0 / 64, 1.0 / 384, 0.0)
LEVEL2 = (1.0, 1.0 / 16, 1.0 / 64, 1.0 / 384, -1.0 / 8)
NAIK = -1.0 / 24
NET_CHANNELS = (1, 8, 8)


def listed():
    return [
        # one hopping term on the smallest lattice in use: launch and latency
        dict(name="dslash_f64_8x8x8x8", kind="dslash", x=8, y=8, z=8, t=8, prec="f64",
             recon=18, parity=1),
        # the paper's 20^3 x 64 lattice at the lowest storage precision
        dict(name="dslash_f16_20x20x20x64", kind="dslash", x=20, y=20, z=20, t=64, prec="f16",
             recon=18, parity=1),
        # the FP64 normal operator on the benchmark lattice: a user's own Krylov or eigen-solver
        dict(name="apply_A_32x32x32x32", kind="apply_A", x=32, y=32, z=32, t=32, mass=0.01),
        # the smallest whole solve: some 200 dependent steps of short kernels
        dict(name="cg_f64_8x8x8x8", kind="cg", x=8, y=8, z=8, t=8, prec="f64", recon=18,
             mass=0.1),
        # an ordinary mixed-precision solve with compressed Naik links, on extents that divide no
        # tile evenly
        dict(name="cg_f32_14x18x16x20", kind="cg", x=14, y=18, z=16, t=20, prec="f32", recon=12,
             mass=0.01),
        # production: nine masses in one Krylov space
        dict(name="multishift_f32_32x32x32x48", kind="multishift", x=32, y=32, z=32, t=48,
             prec="f32", recon=18, shifts=9),
        # many small lattices of three sizes with four sources each
        dict(name="batch_f32_8_12_16", kind="batch", n8=6, n12=6, n16=4, nrhs=4, prec="f32"),
        # links for the solver from thin links, as every molecular-dynamics step needs them
        dict(name="hisq_32x32x32x32", kind="hisq", x=32, y=32, z=32, t=32),
        # the fermion force from nine shifted solutions, the step after the multi-mass solve
        dict(name="force_9_32x32x32x48", kind="force", x=32, y=32, z=32, t=48, terms=9),
        # the preconditioner on the matrix cores, as the flexible CG applies it each step
        dict(name="net_mfma_32x32x32x32", kind="net", x=32, y=32, z=32, t=32, mfma=True),
        # the same in FP32, the entry points' default, on a smaller lattice
        dict(name="net_f32_16x16x16x32", kind="net", x=16, y=16, z=16, t=32, mfma=False),
        # one minibatch of the preconditioner's training: forward, loss, backward on 16^4 blocks
        dict(name="loss_grad_8_16x16x16x16", kind="loss_grad", x=16, y=16, z=16, t=16, pairs=8),
    ]


def _dims(case):
    return case["x"], case["y"], case["z"], case["t"]


def _volume(case):
    return case["x"] * case["y"] * case["z"] * case["t"]


def _draw_dims(rng, lo, hi):
    """Even extents >= 4 with a volume spread over [lo, hi] on a logarithmic scale."""
    while True:
        v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        side = v ** 0.25
        d = [max(4, 2 * round(0.5 * side * math.exp(rng.uniform(-0.3, 0.3)))) for _ in range(3)]
        d.append(max(4, 2 * round(0.5 * v / (d[0] * d[1] * d[2]))))
        if lo <= d[0] * d[1] * d[2] * d[3] <= hi and d[3] <= 96:
            return dict(x=d[0], y=d[1], z=d[2], t=d[3])


def draw(rng):
    kind = rng.choice(["dslash", "dslash", "apply_A", "cg", "cg", "multishift", "batch", "hisq",
                       "force", "net", "net", "loss_grad"])
    prec = rng.choice(["f64", "f32", "f16"])
    recon = rng.choice([18, 12])
    mass = round(math.exp(rng.uniform(math.log(0.01), math.log(0.2))), 4)
    if kind == "dslash":
        return dict(kind=kind, **_draw_dims(rng, 8**4, 32**4), prec=prec, recon=recon,
                    parity=rng.choice([0, 1]))
    if kind == "apply_A":
        return dict(kind=kind, **_draw_dims(rng, 8**4, 32**4), mass=mass)
    if kind == "cg":
        return dict(kind=kind, **_draw_dims(rng, 8**4, 24**4), prec=prec, recon=recon, mass=mass)
    if kind == "multishift":
        return dict(kind=kind, **_draw_dims(rng, 8**4, 32**4), prec=rng.choice(["f64", "f32"]),
                    recon=recon, shifts=rng.randint(2, 12))
    if kind == "batch":
        return dict(kind=kind, n8=rng.randint(1, 6), n12=rng.randint(0, 6), n16=rng.randint(0, 4),
                    nrhs=rng.choice([1, 2, 4]), prec=prec)
    if kind == "hisq":
        return dict(kind=kind, **_draw_dims(rng, 8**4, 32**4))
    if kind == "force":
        return dict(kind=kind, **_draw_dims(rng, 8**4, 32**4), terms=rng.randint(1, 12))
    if kind == "net":
        return dict(kind=kind, **_draw_dims(rng, 8**4, 32**4), mfma=rng.choice([True, False]))
    return dict(kind=kind, **_draw_dims(rng, 8**4, 16**4), pairs=rng.randint(1, 8))


# ------------------------------------------------------------------ synthetic inputs

def _generator(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1009 + stream)
    return g


def _gauss(shape, gen):
    """i.i.d. CN(0, 1) complex128."""
    z = torch.randn(tuple(shape) + (2,), generator=gen, device="cuda", dtype=torch.float64)
    return torch.view_as_complex(z * math.sqrt(0.5))


def _mul(a, b):
    return sum(a[..., :, k, None] * b[..., None, k, :] for k in range(3))


def _dagger(a):
    return a.conj().transpose(-1, -2)


def _su3(n, scale, gen):
    """exp(i scale H) of random traceless Hermitian H, reunitarised (det 1)."""
    G = _gauss((n, 3, 3), gen)
    H = 0.5 * (G + _dagger(G))
    tr = (H[:, 0, 0] + H[:, 1, 1] + H[:, 2, 2]) / 3.0
    eye = torch.eye(3, dtype=torch.complex128, device="cuda")
    X = (0.25j * scale) * (H - tr[:, None, None] * eye)
    U = eye + X / 14
    for k in range(13, 0, -1):
        U = eye + _mul(X, U) / k
    U = _mul(U, U)
    U = _mul(U, U)
    r0 = U[:, 0] / torch.linalg.vector_norm(U[:, 0], dim=-1, keepdim=True)
    r1 = U[:, 1] - (r0.conj() * U[:, 1]).sum(-1, keepdim=True) * r0
    r1 = r1 / torch.linalg.vector_norm(r1, dim=-1, keepdim=True)
    r2 = torch.stack([r0[:, (a + 1) % 3] * r1[:, (a + 2) % 3] -
                      r0[:, (a + 2) % 3] * r1[:, (a + 1) % 3] for a in range(3)], dim=-1).conj()
    return torch.stack([r0, r1, r2], dim=-2)


def _shift(a, dims, mu, k):
    """a(x + k mu) for a per-site array a[V, ...], periodic."""
    nx, ny, nz, nt = dims
    v = a.reshape((nt, nz, ny, nx) + a.shape[1:])
    return torch.roll(v, -k, dims=3 - mu).reshape(a.shape)


def _coords(dims):
    i = torch.arange(dims[0] * dims[1] * dims[2] * dims[3], device="cuda")
    return (i % dims[0], (i // dims[0]) % dims[1], (i // (dims[0] * dims[1])) % dims[2],
            i // (dims[0] * dims[1] * dims[2]))


def _fold(fat, naik, dims):
    """Staggered phases and the antiperiodic time sign multiplied into the links, in place."""
    x, y, z, t = _coords(dims)
    for mu, e in enumerate((0 * x, x, x + y, x + y + z)):
        eta = 1.0 - 2.0 * (e & 1)
        wrap = (lambda h: 1.0 - 2.0 * (t + h >= dims[3])) if mu == 3 else (lambda h: 1.0)
        fat[mu] *= (eta * wrap(1))[:, None, None]
        naik[mu] *= (eta * wrap(3))[:, None, None]


def _thin(dims, seed, scale=0.5):
    vol = dims[0] * dims[1] * dims[2] * dims[3]
    gen = _generator(seed, 1)
    U = torch.empty((4, vol, 3, 3), dtype=torch.complex128, device="cuda")
    for mu in range(4):
        U[mu] = _su3(vol, scale, gen)
    return U


def _links(dims, seed, scale=0.5):
    """Fat and Naik links with phases and boundary folded in, complex128 [4][V][3][3]."""
    U = _thin(dims, seed, scale)
    gen = _generator(seed, 2)
    naik = torch.empty_like(U)
    for mu in range(4):
        naik[mu] = NAIK * _mul(_mul(U[mu], _shift(U[mu], dims, mu, 1)),
                               _shift(U[mu], dims, mu, 2))
    for mu in range(4):
        U[mu] *= 0.9
        U[mu] += 0.05 * _gauss(U[mu].shape, gen)
    _fold(U, naik, dims)
    return U, naik


def _source(vh, seed, stream=3):
    return _gauss((vh, 3), _generator(seed, stream))


def _net_weights(seed):
    """Initial weights of the preconditioner, as a training run starts from them."""
    rng = np.random.default_rng(int(seed))
    ws = []
    for cin, cout in zip(NET_CHANNELS[:-1], NET_CHANNELS[1:]):
        g = rng.standard_normal((cout, cin, 9, 2)) * np.sqrt(0.5 / (9 * cin))
        w = g[..., 0] + 1j * g[..., 1]
        for c in range(min(cin, cout)):
            w[c, c, 0] += 1.0
        ws.append(w)
    return ws


def _sigmas(case):
    m = np.geomspace(0.002, 0.5, case["shifts"])
    return [float(4 * v * v) for v in m]


def _batch_dims(case):
    return [(8,) * 4] * case["n8"] + [(12,) * 4] * case["n12"] + [(16,) * 4] * case["n16"]


def _batch_masses(case, seed):
    return [float(v) for v in
            np.random.default_rng(int(seed)).uniform(0.01, 0.2, len(_batch_dims(case)))]


def _residues(case, seed):
    return [float(v) for v in np.random.default_rng(int(seed)).uniform(0.1, 1.0, case["terms"])]


def _pairs(case, seed, hops):
    """Training pairs (sigma_j, b_j, x_j) of one lattice with A_j x_j = b_j: b_j is formed from a
    drawn x_j."""
    out = []
    for j in range(case["pairs"]):
        x = _source(_volume(case) // 2, seed, 10 + j)
        sigma = 4.0 * (0.01 * (1 + j)) ** 2
        out.append((sigma, hops.A(sigma, x[..., None])[..., 0], x))
    return out


# ------------------------------------------------------------------ prepare and run

def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        dims = _batch_dims(case)
        links = [_links(d, seed * 64 + l, 0.4) for l, d in enumerate(dims)]
        B = ks.Batch(dims, [f.cpu().numpy() for f, _ in links], [n.cpu().numpy() for _, n in links],
                     case["nrhs"], PREC[case["prec"]])
        vhs = [d[0] * d[1] * d[2] * d[3] // 2 for d in dims for _ in range(case["nrhs"])]
        bs = [_source(vh, seed, 10 + p) for p, vh in enumerate(vhs)]
        x = torch.zeros((sum(vhs), 3), dtype=torch.complex128, device="cuda")
        params = ks.default_params(tol=TOL, delta=0.03 if case["prec"] == "f16" else 0.01)
        return dict(case=case, B=B, bs=bs, x=x, xs=list(x.split(vhs)), params=params,
                    masses=_batch_masses(case, seed))
    dims, vol = _dims(case), _volume(case)
    vh = vol // 2
    if kind == "hisq":
        U = _thin(dims, seed)
        return dict(case=case, dims=dims, thin=U, fat=torch.empty_like(U),
                    naik=torch.empty_like(U))
    fat, naik = _links(dims, seed)
    G = ks.Gauge(dims, fat, naik)
    s = dict(case=case, G=G, b=_source(vh, seed))
    if kind == "dslash":
        prec = PREC[case["prec"]]
        G.prepare(prec, case["recon"])
        s["inp"] = ks.Field(G, 1 - case["parity"], prec).load(s["b"])
        s["out"] = ks.Field(G, case["parity"], prec)
        s["y"] = torch.empty_like(s["b"])
    elif kind == "apply_A":
        s["y"] = torch.empty_like(s["b"])
    elif kind in ("cg", "multishift"):
        prec = PREC[case["prec"]]
        G.prepare(prec, case["recon"])
        s["params"] = ks.default_params(tol=TOL, inner=prec, recon=case["recon"])
        if kind == "cg":
            s["x"] = torch.zeros_like(s["b"])
        else:
            s["sigmas"] = _sigmas(case)
            s["xs"] = [torch.zeros_like(s["b"]) for _ in s["sigmas"]]
    elif kind == "force":
        s["residues"] = _residues(case, seed)
        s["xs"] = [_source(vh, seed, 10 + i) for i in range(case["terms"])]
        s["ff"], s["fn"] = torch.empty_like(fat), torch.empty_like(naik)
    elif kind == "net":
        s["net"] = ks.Net(np.concatenate([w.ravel() for w in _net_weights(seed)]))
        s["inp"] = ks.Field(G, ks.EVEN, ks.F32).load(s["b"])
        s["out"] = ks.Field(G, ks.EVEN, ks.F32)
        s["y"] = torch.empty_like(s["b"])
    else:
        pairs = _pairs(case, seed, _Hops((fat, naik), dims))
        s["net"] = ks.Net(np.concatenate([w.ravel() for w in _net_weights(seed)]))
        s["gauges"] = [G] * len(pairs)
        s["sigmas"], s["bs"], s["xs"] = (list(v) for v in zip(*pairs))
    return s


def _values(y, prec):
    """A field's values in its own precision."""
    if prec == "f64":
        return y
    if prec == "f32":
        return y.to(torch.complex64)
    return torch.view_as_real(y).to(torch.float16)


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "dslash":
        ks.dslash_eo(s["G"], s["out"], s["inp"], case["recon"])
        return _values(s["out"].store(s["y"]), case["prec"])
    if kind == "apply_A":
        return ks.apply_A(s["G"], 4 * case["mass"] ** 2, s["b"], s["y"])
    if kind == "cg":
        s["x"].zero_()
        ks.cg_solve(s["G"], case["mass"], s["b"], s["x"], s["params"])
        return s["x"]
    if kind == "multishift":
        ks.multishift_cg_solve(s["G"], s["sigmas"], s["b"], s["xs"], TOL, s["params"])
        return s["xs"]
    if kind == "batch":
        s["x"].zero_()
        s["B"].solve(s["masses"], s["bs"], s["xs"], s["params"])
        return s["x"]
    if kind == "hisq":
        ks.hisq_links(s["dims"], s["thin"], s["fat"], s["naik"])
        return s["fat"], s["naik"]
    if kind == "force":
        ks.force(s["G"], s["residues"], s["xs"], s["ff"], s["fn"])
        return s["ff"], s["fn"]
    if kind == "net":
        s["net"].apply_field(s["inp"], s["out"], mfma=case["mfma"])
        return _values(s["out"].store(s["y"]), "f16" if case["mfma"] else "f32")
    loss, grad = s["net"].loss_grad(s["gauges"], s["sigmas"], s["bs"], s["xs"])
    return loss, grad.astype(np.complex64)       # FP32 forward and backward


# ------------------------------------------------------------------ the least work

def _real_bytes(prec):
    return {"f64": 8, "f32": 4, "f16": 2}[prec]


def _vector_bytes(prec):
    return {"f64": 48, "f32": 24, "f16": 16}[prec]


def _link_bytes(prec, recon=18):
    """The 16 matrices of an output site."""
    return 8 * (18 + recon) * _real_bytes(prec)


def _steps(mass, nt):
    """CG steps to TOL: the Chebyshev rate for the spectrum these fields have (largest eigenvalue
    18.7, smallest 4 m^2 + (pi / Nt)^2 / 2)."""
    kappa = 18.7 / (4 * mass * mass + 0.5 * (math.pi / nt) ** 2)
    return 0.41 * math.sqrt(kappa) * math.log(2 / TOL)


DSLASH_FLOPS = 1146.0            # per output site


def work(case):
    kind = case["kind"]
    if kind == "batch":
        b = f = 0.0
        # a lattice's links serve its right-hand sides; p, r, q, x per right-hand side
        for d in _batch_dims(case):
            vh = d[0] * d[1] * d[2] * d[3] / 2
            n = _steps(0.03, d[3])
            p, r = case["prec"], case["nrhs"]
            b += n * vh * (2 * _link_bytes(p) + r * (12 * _vector_bytes(p)))
            f += n * vh * r * (2 * DSLASH_FLOPS + 72)
        return {"bytes": b, "flops": f}
    vol = _volume(case)
    vh = vol / 2
    if kind == "dslash":
        p = case["prec"]
        return {"bytes": vh * (_link_bytes(p, case["recon"]) + 2 * _vector_bytes(p)),
                "flops": vh * DSLASH_FLOPS}
    if kind == "apply_A":
        return {"bytes": vh * (2 * _link_bytes("f64") + 96), "flops": vh * (2 * DSLASH_FLOPS + 12)}
    if kind in ("cg", "multishift"):
        # per step: both hopping terms' links, and p, q, t, r, x moved between them
        p = case["prec"]
        n = _steps(case["mass"] if kind == "cg" else 0.002, case["t"])
        b = 2 * _link_bytes(p, case["recon"]) + 12 * _vector_bytes(p)
        f = 2 * DSLASH_FLOPS + 72
        if kind == "multishift":
            b += (case["shifts"] - 1) * 4 * _vector_bytes(p) / 2   # heavy shifts freeze early
            f += (case["shifts"] - 1) * 24
        return {"bytes": n * vh * b, "flops": n * vh * f}
    if kind == "hisq":
        # thin links in, fat and Naik links out; 3x3 products: per level and direction 6 three-,
        # 12 five- and 6 seven-link staples of 2 products, then the Naik link
        return {"bytes": 3.0 * 576 * vol, "flops": vol * 198.0 * (2 * 4 * 24 * 2 + 8)}
    if kind == "force":
        return {"bytes": vh * (_link_bytes("f64") + 48.0 * case["terms"]) + 1152.0 * vol,
                "flops": case["terms"] * (vh * DSLASH_FLOPS + vol * 8 * 72.0)}
    # network, per site of the full lattice: four layers of channel mixing (9 paths) and
    # transports (8 hops), the links read once
    layers = [(1, 8), (8, 8), (8, 8), (8, 1)]
    f = vol * sum(3 * 9 * ci * co * 8.0 + 8 * ci * 66.0 for ci, co in layers)
    if kind == "net":
        return {"bytes": vol * (8 * 18 * (2 if case["mfma"] else 4)) + vh * 48, "flops": f}
    # training: forward, input gradients and weight gradients; A in FP64
    links = vol * 8 * 18 * 4 + vh * 2 * _link_bytes("f64")
    return {"bytes": links + case["pairs"] * vh * 96.0,
            "flops": case["pairs"] * (3 * f + vh * 2 * DSLASH_FLOPS)}


# ------------------------------------------------------------------ the same in 64 bits

def _embed(cb, parity, dims):
    x, y, z, t = _coords(dims)
    full = torch.zeros((x.numel(),) + cb.shape[1:], dtype=cb.dtype, device=cb.device)
    full[((x + y + z + t) & 1) == parity] = cb
    return full


def _restrict(full, parity, dims):
    x, y, z, t = _coords(dims)
    return full[((x + y + z + t) & 1) == parity]


def _mv(m, v):
    """3x3 matrices times vectors v[..., 3, R]."""
    return sum(m[..., :, k, None] * v[..., None, k, :] for k in range(3))


class _Hops:
    """The hopping terms of a lattice: per output parity the 16 matrices of every site and the
    rows of the other parity they multiply."""

    def __init__(self, links, dims):
        vol = links[0].shape[1]
        sites = torch.arange(vol, device="cuda")
        self.terms = {}
        for p in (0, 1):
            self.terms[p] = []
            for L, hops in zip(links, (1, 3)):
                for mu in range(4):
                    back = _shift(L[mu], dims, mu, -hops)
                    for m, k in ((L[mu], hops), (-_dagger(back), -hops)):
                        row = _shift(sites, dims, mu, k) >> 1
                        self.terms[p].append((_restrict(m, p, dims).contiguous(),
                                              _restrict(row, p, dims)))

    def __call__(self, parity, v):
        return sum(_mv(m, v[row]) for m, row in self.terms[parity])

    def A(self, sigma, v):
        return sigma * v - self(0, self(1, v))


def _dslash(links, dims, parity, v):
    return _Hops(links, dims)(parity, v[..., None])[..., 0]


def _apply_A(links, dims, sigma, v):
    return _Hops(links, dims).A(sigma, v[..., None])[..., 0]


def _cg(hops, sigma, b, tol=1e-14, most=4000):
    """CG on every column of b[Vh, 3, R], sigma per column."""
    x, r = torch.zeros_like(b), b.clone()
    p = r.clone()
    dot = lambda u, v: (u.real * v.real + u.imag * v.imag).sum((0, 1))  # noqa: E731
    rho = dot(r, r)
    stop = tol * tol * rho
    for k in range(most):
        q = hops.A(sigma, p)
        a = torch.where(rho > stop, rho / dot(p, q), torch.zeros_like(rho))
        x += a * p
        r -= a * q
        new = torch.where(rho > stop, dot(r, r), rho)
        p = torch.where(rho > stop, r + (new / rho) * p, p)
        rho = new
        if k % 25 == 24 and bool((rho <= stop).all()):
            break
    return x


def _net_layers(ws):
    """The four applied layers: the free two, then their adjoints."""
    back = [0, 5, 6, 7, 8, 1, 2, 3, 4]
    return list(ws) + [w.conj().transpose(0, 1)[:, :, back] for w in reversed(ws)]


def _net(ws, fat, dims, b):
    phi = _embed(b, 0, dims)[None]
    hop = lambda p, v: (_mv(fat[p - 1], _shift(v, dims, p - 1, 1)[..., None])[..., 0] if p < 5  # noqa: E731
                        else _shift(_mv(_dagger(fat[p - 5]), v[..., None])[..., 0], dims, p - 5, -1))
    for w in _net_layers(ws):
        paths = [torch.stack([hop(p, v) if p else v for v in phi]) for p in range(9)]
        phi = torch.stack([sum(w[c, d, p] * paths[p][d] for p in range(9)
                               for d in range(w.shape[1])) for c in range(w.shape[0])])
    return _restrict(phi[0], 0, dims)


def _weights64(seed):
    return [torch.from_numpy(w).cuda() for w in _net_weights(seed)]


def _staple(U, dims, mu, nu, s, M):
    L = U[nu] if s > 0 else _dagger(_shift(U[nu], dims, nu, -1))
    return _mul(_mul(L, _shift(M, dims, nu, s)), _dagger(_shift(L, dims, mu, 1)))


def _smear(U, dims, coeffs):
    c1, c3, c5, c7, cl = coeffs
    out = torch.empty_like(U)
    for mu in range(4):
        dirs = [(nu, s) for nu in range(4) if nu != mu for s in (1, -1)]
        s1 = {d: _staple(U, dims, mu, *d, U[mu]) for d in dirs}
        f = c1 * U[mu]
        for a in dirs:
            inner = c3 * U[mu] + cl * s1[a]
            for b in dirs:
                if b[0] != a[0]:
                    m = c5 * U[mu] + c7 * sum(s1[c] for c in dirs if c[0] not in (a[0], b[0]))
                    inner = inner + _staple(U, dims, mu, *b, m)
            f = f + _staple(U, dims, mu, *a, inner)
        out[mu] = f
    return out


def _polar(V):
    """The unitary factor of V by Newton's iteration X <- (X + X^-dagger) / 2."""
    X = V
    for _ in range(14):
        cof = torch.stack([torch.stack([
            X[..., (a + 1) % 3, (b + 1) % 3] * X[..., (a + 2) % 3, (b + 2) % 3] -
            X[..., (a + 1) % 3, (b + 2) % 3] * X[..., (a + 2) % 3, (b + 1) % 3]
            for b in range(3)], -1) for a in range(3)], -2)
        det = sum(X[..., 0, b] * cof[..., 0, b] for b in range(3))
        X = 0.5 * (X + (cof / det[..., None, None]).conj())
    return X


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        # lattice after lattice; the right-hand sides of one together
        out, pair = [], 0
        for l, (d, m) in enumerate(zip(_batch_dims(case), _batch_masses(case, seed))):
            hops = _Hops(_links(d, seed * 64 + l, 0.4), d)
            vh = d[0] * d[1] * d[2] * d[3] // 2
            b = torch.stack([_source(vh, seed, 10 + pair + r) for r in range(case["nrhs"])], -1)
            pair += case["nrhs"]
            x = _cg(hops, torch.full((case["nrhs"],), 4 * m * m, device="cuda",
                                     dtype=torch.float64), b)
            out += [x[..., r] for r in range(case["nrhs"])]
        return torch.cat(out)
    dims, vol = _dims(case), _volume(case)
    vh = vol // 2
    if kind == "hisq":
        W = _polar(_smear(_thin(dims, seed), dims, LEVEL1))
        fat = _smear(W, dims, LEVEL2)
        naik = torch.stack([NAIK * _mul(_mul(W[mu], _shift(W[mu], dims, mu, 1)),
                                        _shift(W[mu], dims, mu, 2)) for mu in range(4)])
        _fold(fat, naik, dims)
        return fat, naik
    if kind in ("cg", "multishift") and vol > 20**4:
        return None                       # hundreds of steps of a large lattice
    links = _links(dims, seed)
    b = _source(vh, seed)
    if kind == "dslash":
        y = _dslash(links, dims, case["parity"], b)
        return torch.view_as_real(y) if case["prec"] == "f16" else y
    if kind == "apply_A":
        return _apply_A(links, dims, 4 * case["mass"] ** 2, b)
    if kind == "cg":
        sigma = torch.full((1,), 4 * case["mass"] ** 2, device="cuda", dtype=torch.float64)
        return _cg(_Hops(links, dims), sigma, b[..., None])[..., 0]
    if kind == "multishift":
        sigma = torch.tensor(_sigmas(case), device="cuda", dtype=torch.float64)
        x = _cg(_Hops(links, dims), sigma, b[..., None].repeat(1, 1, case["shifts"]))
        return [x[..., i] for i in range(case["shifts"])]
    if kind == "force":
        x, y, z, t = _coords(dims)
        eps = (1 - 2 * ((x + y + z + t) & 1)).to(torch.float64)
        hops = _Hops(links, dims)
        ff, fn = torch.zeros_like(links[0]), torch.zeros_like(links[1])
        for i, r in enumerate(_residues(case, seed)):
            even = _source(vh, seed, 10 + i)
            psi = _embed(even, 0, dims) + _embed(hops(1, even[..., None])[..., 0], 1, dims)
            for mu in range(4):
                for f, k in ((ff, 1), (fn, 3)):
                    f[mu] += (r * eps)[:, None, None] * (
                        _shift(psi, dims, mu, k)[:, :, None] * psi.conj()[:, None, :])
        return ff, fn
    if kind == "net":
        y = _net(_weights64(seed), links[0], dims, b)
        return torch.view_as_real(y) if case["mfma"] else y
    ws = [w.requires_grad_() for w in _weights64(seed)]
    hops = _Hops(links, dims)
    pairs = _pairs(case, seed, hops)
    total = 0.0
    for sigma, bj, xj in pairs:
        with torch.enable_grad():
            d = _net(ws, links[0], dims, bj) - xj
            ad = hops.A(sigma, d[..., None])[..., 0]
            xax = float((xj.conj() * bj).sum().real)
            loss = (d.conj() * ad).sum().real / (xax * len(pairs))
            loss.backward()
        total += float(loss.detach())
    return total, torch.cat([w.grad.reshape(-1) for w in ws])
