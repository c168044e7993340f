"""The work that programs have this library do, as timed cases.

Lattices are those of this repository's benchmarks (4^4, 8^3x16, 16^3x32,
24^3x48, 32^3x64) and ragged ones; links are random SU(3) matrices near 1
(eps = 0.3, as synth.random_gauge draws them), sources are Gaussian or point
sources, kappa, 2 kappa mu and the doublet's masses are the benchmarks'.

listed() gives the cases, draw() more of the same ranges; prepare() makes a
case's inputs and the lattice handle a program keeps, run() is one pass
through the public calls, work() the bytes and operations a pass cannot do
without, and exact() the same outputs in complex128 torch operations.

A case is a dict: "op" (the call, see run()), "dims" extents T, LZ, LY, LX,
"prec" (storage of an applied operator, or of a solve's inner iteration),
"nrhs" right-hand sides, "theta" 1 for antiperiodic fermions in time only, 2
for phases in every direction, "mu" 2 kappa mu.
"""
import math

import torch

from paper_0905_3331_amd import tmq

KAPPA, KAPPA_FULL = 0.1632, 0.16
ND = (0.17, 0.1105, 0.0935)  # kappa, 2 kappa mubar, 2 kappa epsbar of the doublet runs
TOL = 1e-10
THETA = {1: (1.0, 0.0, 0.0, 0.0), 2: (1.0, 0.25, -0.5, 0.125)}
# iterations a solve of these operators takes to TOL (they hardly depend on the lattice)
ITERS = {"solve": 35, "batch": 35, "md": 35, "prop": 35, "nd": 40, "full": 107}


def _case(op, T, LZ, LY, LX, prec, nrhs=1, theta=1, mu=0.004, name=None):
    c = {"op": op, "T": T, "LZ": LZ, "LY": LY, "LX": LX, "prec": prec, "nrhs": nrhs, "theta": theta, "mu": mu}
    return dict(c, name=name) if name else c


def listed():
    return [
        # one application of Qhat on the smallest lattice of the serving mix: launches and latency
        _case("qhat", 16, 8, 8, 8, "fp64", name="qhat64_8c16"),
        # an application on extents that no tile divides (x rows of 9 sites per parity), FP32
        _case("qhat", 20, 10, 14, 18, "fp32", name="qhat32_ragged"),
        # the headline's 16-bit operator, on the lattice of the paper-size runs
        _case("qhat", 48, 24, 24, 24, "fp16", name="qhat16_24c48"),
        # the full-lattice operator on the largest lattice
        _case("qfull", 64, 32, 32, 32, "fp64", name="qfull64_32c64"),
        # the smallest solve: plain FP64 CG on the full lattice
        _case("full", 4, 4, 4, 4, "fp64", mu=0.01, name="full64_4c4"),
        # one served request's solve on a small lattice, FP32 inner iteration
        _case("solve", 16, 8, 8, 8, "fp32", mu=0.011, name="solve32_8c16"),
        # the reference solver: FP64 CG
        _case("solve", 48, 24, 24, 24, "fp64", name="solve64_24c48"),
        # the headline solve: FP16 inner iteration, FP64 reliable updates
        _case("solve", 64, 32, 32, 32, "fp16", name="solve16_32c64"),
        # many inversions per gauge field: 12 spin-colour point sources x 2 masses in one batch, FP32 inner
        _case("batch", 48, 24, 24, 24, "fp32", nrhs=24, name="batch32_24c48"),
        # the strange-charm doublet, FP16 inner iteration
        _case("nd", 48, 24, 24, 24, "fp16", name="nd16_24c48"),
        # a propagator: M psi = phi for the 12 spin-colour sources of a site
        _case("prop", 32, 16, 16, 16, "fp16", nrhs=12, name="prop16_16c32"),
        # a molecular-dynamics step's solver part: new links, then the force solves
        _case("md", 48, 24, 24, 24, "fp16", name="md16_24c48"),
    ]


def _dims(rng, lo, hi):
    """Even extents with a volume spread over [lo, hi] on a logarithmic scale."""
    while True:
        want = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        side = want ** 0.25
        d = [max(4, 2 * round(side * math.exp(rng.uniform(-0.4, 0.4)) / 2)) for _ in range(4)]
        d[0] = max(4, 2 * round(want / (d[1] * d[2] * d[3]) / 2))
        if d[0] <= 128 and lo <= d[0] * d[1] * d[2] * d[3] <= hi:
            return d


def draw(rng):
    op = rng.choice(["qhat", "qhat", "qhat", "qfull", "full", "solve", "solve", "solve", "batch", "nd", "prop", "md"])
    theta = 2 if rng.random() < 0.2 else 1
    mu = round(rng.uniform(0.002, 0.02), 4)
    prec, nrhs, lo, hi = "fp64", 1, 8192, 1 << 21
    if op == "qhat":
        prec = rng.choice(["fp64", "fp32", "fp16", "bf16"])
    elif op == "full":
        lo, hi = 256, 1024
    elif op in ("solve", "md"):
        prec = rng.choice(["fp64", "fp32", "fp16"])
    elif op == "batch":
        prec, nrhs = rng.choice(["fp32", "fp16"]), rng.randint(2, 24)
        hi = 663552
    elif op == "nd":
        prec, hi = rng.choice(["fp64", "fp32", "fp16"]), 663552
    elif op == "prop":
        prec, nrhs, hi = rng.choice(["fp32", "fp16"]), 12, 131072
    return _case(op, *_dims(rng, lo, hi), prec, nrhs, theta, mu)


# ------------------------------------------------------------------- inputs


def _dim4(case):
    return case["T"], case["LZ"], case["LY"], case["LX"]


def _gauss(gen, *shape):
    return torch.view_as_complex(torch.randn(*shape, 2, generator=gen, dtype=torch.float64, device="cuda")) / math.sqrt(2)


def _links(gen, dims, eps=0.3):
    """Random SU(3) links (T, LZ, LY, LX, 4, 3, 3): the rows of 1 + i eps H, orthonormalised."""
    h = eps / 2 * torch.randn(8, *dims, 4, generator=gen, dtype=torch.float64, device="cuda")
    z = torch.complex
    d8 = h[7] / math.sqrt(3)
    one = torch.ones_like(h[0])
    r0 = torch.stack([z(one, h[2] + d8), z(h[1], h[0]), z(h[4], h[3])], dim=-1)
    r1 = torch.stack([z(-h[1], h[0]), z(one, d8 - h[2]), z(h[6], h[5])], dim=-1)
    r0 = r0 / torch.linalg.vector_norm(r0, dim=-1, keepdim=True)
    r1 = r1 - (r0.conj() * r1).sum(-1, keepdim=True) * r0
    r1 = r1 / torch.linalg.vector_norm(r1, dim=-1, keepdim=True)
    r2 = torch.stack([r0[..., 1] * r1[..., 2] - r0[..., 2] * r1[..., 1], r0[..., 2] * r1[..., 0] - r0[..., 0] * r1[..., 2],
                      r0[..., 0] * r1[..., 1] - r0[..., 1] * r1[..., 0]], dim=-1).conj()
    return torch.stack([r0, r1, r2], dim=-2).contiguous()


def _inputs(case, seed):
    """Links, sources and 2 kappa mu per right-hand side."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dims, op, n = _dim4(case), case["op"], case["nrhs"]
    V = math.prod(dims)
    U = _links(gen, dims)
    if op in ("batch", "prop"):  # the spin-colour point sources of one site, for one or more masses
        sites = V // 2 if op == "batch" else V
        at = int(torch.randint(sites, (1,), generator=gen, device="cuda"))
        b = []
        for k in range(n):
            v = torch.zeros(sites, 4, 3, dtype=torch.complex128, device="cuda")
            v[at, k % 12 // 3, k % 3] = 1.0
            b.append(v)
    elif op == "nd":
        b = [_gauss(gen, 2, V // 2, 4, 3)]
    else:
        b = [_gauss(gen, V if op in ("qfull", "full") else V // 2, 4, 3)]
    mus = [case["mu"] * 2 ** (k // 12) if op == "batch" else case["mu"] for k in range(n)]
    return U, b, mus


def _kappa(case):
    return KAPPA_FULL if case["op"] == "full" else ND[0] if case["op"] == "nd" else KAPPA


def prepare(case, seed):
    U, b, mus = _inputs(case, seed)
    lat = tmq.Lattice(_dim4(case))
    lat.load_gauge(U)
    th = THETA[case["theta"]]
    if case["op"] == "nd":
        ps = [tmq.nd_params(*ND, th)]
    else:
        ps = [tmq.params(_kappa(case), m, th) for m in mus]
    prec = case["prec"]
    opts = tmq.solver_opts(tol=TOL, sloppy=prec, sloppy_link="fp32" if prec == "fp32" else "fp16")
    s = {"op": case["op"], "lat": lat, "ps": ps, "b": b, "opts": opts, "prec": prec}
    if case["op"] == "md":
        s["U"] = U
    return s


def run(s):
    op, lat, ps, b, opts = s["op"], s["lat"], s["ps"], s["b"], s["opts"]
    if op == "qhat":
        return lat.apply_Qhat(ps[0], +1, b[0], prec=s["prec"])
    if op == "qfull":
        return lat.apply_Q_full(ps[0], +1, b[0])
    if op == "full":
        return lat.solve_full(ps[0], b[0], opts)[0]
    if op == "solve":
        return lat.solve(ps[0], b[0], opts)[0]
    if op == "batch":
        return lat.solve_batch(ps, b, opts)[0]
    if op == "nd":
        return lat.solve_nd(ps[0], b[0], opts)[0]
    if op == "prop":
        return lat.solve_M_batch(ps[0], +1, b, opts)[0]
    lat.load_gauge(s["U"])
    return list(lat.solve_force(ps[0], b[0], opts)[:3])


# --------------------------------------------------------------------- work


def work(case):
    """Bytes of the operands in the storage that the call asks for, each once
    per half-sweep or vector update, and the 1320 flop per output site of a
    half-sweep."""
    V = math.prod(_dim4(case))
    vh, op, prec, n = V // 2, case["op"], case["prec"], case["nrhs"]
    sp = {"fp64": 192, "fp32": 96, "fp16": 52, "bf16": 52}[prec]
    lk = {"fp64": 96, "fp32": 48, "fp16": 24, "bf16": 24}[prec]
    if op == "qhat":  # the source and the result, the links of K1 and K2, the even-site field between them
        return {"bytes": vh * (2 * 192 + 2 * 8 * lk + 2 * sp), "flops": 2 * 1320.0 * vh}
    if op == "qfull":
        return {"bytes": V * (2 * 192 + 4 * lk), "flops": 1320.0 * V}
    it = ITERS[op]
    if op == "full":  # fits the caches: the links, the source and the solution once
        return {"bytes": V * (2 * 192 + 4 * 96), "flops": 2 * 1320.0 * V * it}
    fl = 2 if op == "nd" else 1
    # an iteration: four half-sweeps (links for all right-hand sides, input, own site in two of them, output in
    # three), r, p and x of the update; the true residual at the end in FP64; the source and the solution
    xs = 192 if prec == "fp64" else 96
    body = 4 * 8 * lk + n * fl * ((4 + 2 + 3) * sp + 4 * sp + 2 * xs)
    end = 4 * 8 * 96 + n * fl * 192 * 10
    b = vh * (it * body + end)
    if op == "md":  # the new links, and their copies in each storage
        b += 4 * V * (144 + 144 + 96 + 48 + 24)
    return {"bytes": b, "flops": 4 * 1320.0 * vh * n * fl * it}


# -------------------------------------------------------------------- exact


class _Op:
    """The operators in complex128 torch operations on full-lattice fields (T, LZ, LY, LX, 4, 3)."""

    AXIS = (0, 3, 2, 1)  # of t, x, y, z

    def __init__(self, U, dims, kappa, theta):
        self.U, self.dims, self.kappa = U, dims, kappa
        self.ph = [complex(math.cos(math.pi * th / dims[a]), math.sin(math.pi * th / dims[a])) for th, a in zip(theta, self.AXIS)]
        t, z, y, x = torch.meshgrid(*(torch.arange(d, device="cuda") for d in dims), indexing="ij")
        self.odd = ((t + x + y + z) % 2 == 1).reshape(-1)
        # the upper right block of gamma_mu; the lower left one is its adjoint
        self.g = torch.tensor([[[-1, 0], [0, -1]], [[0, -1j], [-1j, 0]], [[0, -1], [1, 0]], [[-1j, 0], [0, 1j]]],
                              dtype=torch.complex128, device="cuda")

    def full(self, odd=None, even=None):
        f = torch.zeros(self.odd.numel(), 4, 3, dtype=torch.complex128, device="cuda")
        if odd is not None:
            f[self.odd] = odd
        if even is not None:
            f[~self.odd] = even
        return f.reshape(*self.dims, 4, 3)

    def of(self, f, odd):
        return f.reshape(-1, 4, 3)[self.odd if odd else ~self.odd]

    @staticmethod
    def _mix(m, h):  # the 2x2 spin matrix m (one entry per row) on the two spin rows of h
        rows = []
        for i in range(2):
            j = 0 if m[i][0] != 0 else 1
            rows.append(m[i][j] * h[..., j, :])
        return torch.stack(rows, dim=-2)

    def H(self, psi):
        up, dn = torch.zeros_like(psi[..., :2, :]), torch.zeros_like(psi[..., 2:, :])
        for mu in range(4):
            a, ph = self.AXIS[mu], self.ph[mu]
            g = self.g[mu].tolist()
            gh = self.g[mu].conj().T.tolist()
            u = self.U[..., mu, :, :]
            n = torch.roll(psi, -1, a)
            h = n[..., :2, :] + self._mix(g, n[..., 2:, :])
            w = sum(u[..., None, :, c] * h[..., c, None] for c in range(3)) * ph
            up += w
            dn += self._mix(gh, w)
            h = psi[..., :2, :] - self._mix(g, psi[..., 2:, :])
            w = torch.roll(sum(u[..., None, c, :].conj() * h[..., c, None] for c in range(3)), 1, a) * ph.conjugate()
            up += w
            dn -= self._mix(gh, w)
        return torch.cat([up, dn], dim=-2)

    @staticmethod
    def tw(f, a, b):  # (a + b g5) f
        return torch.cat([(a + b) * f[..., :2, :], (a - b) * f[..., 2:, :]], dim=-2)

    def Q(self, psi, m, sign):
        return self.tw(self.tw(psi, 1, 1j * sign * m) - self.kappa * self.H(psi), 0, 1)

    def Qhat(self, o, m, sign):
        e = self.of(self.H(self.full(odd=o)), False)
        e = self.tw(e, 1, -1j * sign * m) * (self.kappa ** 2 / (1 + m * m))
        return self.tw(self.tw(o, 1, 1j * sign * m) - self.of(self.H(self.full(even=e)), True), 0, 1)

    def Qhat_nd(self, o, m, eps, sign):
        m = sign * m
        e = [self.of(self.H(self.full(odd=o[f])), False) for f in range(2)]
        c = self.kappa ** 2 / (1 + m * m - eps * eps)
        e = [c * (self.tw(e[0], 1, -1j * m) - eps * e[1]), c * (self.tw(e[1], 1, 1j * m) - eps * e[0])]
        w = [self.tw(o[0], 1, 1j * m) + eps * o[1], self.tw(o[1], 1, -1j * m) + eps * o[0]]
        return torch.stack([self.tw(w[f] - self.of(self.H(self.full(even=e[f])), True), 0, 1) for f in range(2)])


def _cg(A, b, tol=1e-14, most=1000):
    x, r = torch.zeros_like(b), b.clone()
    p, rr = r.clone(), float((r.abs() ** 2).sum())
    stop = tol * tol * rr
    for _ in range(most):
        if rr <= stop:
            break
        ap = A(p)
        al = rr / float((p.conj() * ap).sum().real)
        x += al * p
        r -= al * ap
        new = float((r.abs() ** 2).sum())
        p = r + new / rr * p
        rr = new
    return x


def exact(case, seed):
    U, b, mus = _inputs(case, seed)
    dims, op, m = _dim4(case), case["op"], mus[0]
    D = _Op(U, dims, _kappa(case), THETA[case["theta"]])
    if op == "qhat":
        return D.Qhat(b[0], m, +1)
    if op == "qfull":
        return D.Q(b[0].reshape(*dims, 4, 3), m, +1).reshape(-1, 4, 3)
    if op == "full":
        x = _cg(lambda v: D.Q(D.Q(v, m, -1), m, +1), b[0].reshape(*dims, 4, 3))
        return x.reshape(-1, 4, 3)
    if op == "nd":
        return _cg(lambda v: D.Qhat_nd(D.Qhat_nd(v, ND[1], ND[2], -1), ND[1], ND[2], +1), b[0])

    def inv(rhs, mk):
        return _cg(lambda v: D.Qhat(D.Qhat(v, mk, -1), mk, +1), rhs)

    if op in ("solve", "batch"):  # of a batch the first four right-hand sides (the others take too long)
        xs = [inv(b[k], mus[k]) if k < 4 else None for k in range(len(b))]
        return xs if op == "batch" else xs[0]
    if op == "prop":
        out = []
        for v in b:
            f = v.reshape(*dims, 4, 3)
            e, o = D.of(f, False), D.of(f, True)
            e1 = D.tw(e, 1, -1j * m) / (1 + m * m)
            o1 = o + D.kappa * D.of(D.H(D.full(even=e1)), True)
            po = D.Qhat(inv(D.tw(o1, 0, 1), m), m, -1)
            pe = D.tw(e + D.kappa * D.of(D.H(D.full(odd=po)), False), 1, -1j * m) / (1 + m * m)
            out.append(D.full(odd=po, even=pe).reshape(-1, 4, 3))
        return out
    X = inv(b[0], m)
    return [X, D.Qhat(X, m, -1), float((b[0].conj() * X).sum().real)]
