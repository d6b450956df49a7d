"""The library's work, as a user's program has it done, in cases that can be timed.

Each case is one call sequence through the binding of the C ABI on one lattice: applications of
the fermion matrix, the transfer of fields in and out of the library's layout, taking up a new
gauge configuration, the solvers, and the solve server.  listed() holds the cases, draw() makes
others of the same ranges, prepare() makes what a program holds before the call, run() is one
pass, exact() the same result in plain FP64 torch, and work() the bytes and operations that one
pass cannot do without.

Links are U = exp(0.2 i H) with H Gaussian, traceless and Hermitian; sources are complex Gaussian.
"""
import math

import torch

from paper_1711_03836_amd import bqhip as bq

DEVICE = "cuda" if torch.cuda.is_available() else "cpu"
EPS, CSW, T_BC = 0.2, 1.5, -1
PREC = {"f64": bq.BQ_F64, "f32": bq.BQ_F32, "f16": bq.BQ_F16}
KINDS = {"M": bq.BQ_OP_M, "Mdag": bq.BQ_OP_MDAG, "Mhat": bq.BQ_OP_MHAT, "MhatdagMhat": bq.BQ_OP_MHATDAG_MHAT,
         "K1": bq.BQ_OP_K1, "clover": bq.BQ_OP_CLOVER}
SOLVERS = {"cg": bq.BQ_SOLVER_CG, "bicgstab": bq.BQ_SOLVER_BICGSTAB, "block": bq.BQ_SOLVER_BLOCK_CG}
# What a tuning file written by save_tuning holds for 12 columns: (recon, R, bs, march, lds, order)
TUNED_12 = {"f64": (12, 1, 256, 0, 1, 2), "f32": (12, 1, 768, 0, 1, 1), "f16": (12, 1, 768, 0, 1, 1)}


def listed():
    return [
        # The smallest call: one application of the Schur operator on the smallest lattice of the
        # serving mix, where launches and allocations are all that it costs.
        dict(name="apply_8_f64_1", do="apply", kind="Mhat", x=8, y=8, z=8, t=8, prec="f64", nrhs=1),
        # An odd lattice, whose last 64-site tile is not full and whose planes hold no whole tiles,
        # with an odd number of columns.
        dict(name="apply_ragged_f32_3", do="apply", kind="Mdag", x=6, y=10, z=14, t=18, prec="f32", nrhs=3),
        # One FP64 column of the normal operator, as an eigensolver or a molecular-dynamics force has it applied.
        dict(name="apply_24_f64_1", do="apply", kind="MhatdagMhat", x=24, y=24, z=24, t=48, prec="f64", nrhs=1),
        # The twelve spin-colour columns of a propagator on the lattice of the benchmark, library defaults.
        dict(name="apply_32_f32_12", do="apply", kind="MhatdagMhat", x=32, y=32, z=32, t=64, prec="f32", nrhs=12),
        # A block of noise vectors in FP16 storage.
        dict(name="apply_24_f16_16", do="apply", kind="Mhat", x=24, y=24, z=24, t=48, prec="f16", nrhs=16),
        # Twelve FP64 sources into the library's layout and back (device buffers of the caller).
        dict(name="transfer_24_f64_12", do="transfer", x=24, y=24, z=24, t=48, prec="f64", nrhs=12),
        # A new configuration of a Markov chain: upload, clover term and inverse, plaquette, one use.
        dict(name="configuration_24", do="configuration", x=24, y=24, z=24, t=48, nrhs=1),
        # One Gaussian source on 16^3x32 solved with FP32 inner iterations.
        dict(name="solve_16_f32_1", do="solve", solver="cg", system="M", x=16, y=16, z=16, t=32, prec="f32", nrhs=1,
             kappa=0.125, mu=0.0, tuned=False),
        # A propagator: twelve sources, FP32 inner iterations, with the settings of a tuning file.
        dict(name="solve_24_f32_12", do="solve", solver="cg", system="M", x=24, y=24, z=24, t=48, prec="f32", nrhs=12,
             kappa=0.124, mu=0.1, tuned=True),
        # The shifted systems of a rational approximation (RHMC).
        dict(name="multishift_16_8", do="multishift", x=16, y=16, z=16, t=32, nshift=8, nrhs=1, kappa=0.124),
        # Block CG on twelve sources.
        dict(name="block_16_12", do="solve", solver="block", system="M", x=16, y=16, z=16, t=32, prec="f64", nrhs=12,
             kappa=0.124, mu=0.0, tuned=False),
        # The solve server: six requests of 1 to 4 columns with kappas of their own on one small gauge field.
        dict(name="serve_8_6", do="serve", x=8, y=8, z=8, t=8, requests=6, maxcols=4),
    ]


def _lattice(rng, vmin, vmax):
    """Even extents with a volume between vmin and vmax, spread over its logarithm."""
    while True:
        v = math.exp(rng.uniform(math.log(vmin), math.log(vmax)))
        side = (v / 2) ** 0.25
        x, y, z = (max(4, 2 * round(side * rng.uniform(0.75, 1.3) / 2)) for _ in range(3))
        t = max(4, 2 * round(v / (x * y * z) / 2))
        if vmin <= x * y * z * t <= vmax and t <= 96:
            return dict(x=x, y=y, z=z, t=t)


def draw(rng):
    do = rng.choice(["apply", "apply", "apply", "apply", "transfer", "configuration", "solve", "solve", "multishift",
                     "block", "serve"])
    if do == "apply":
        prec = rng.choice(["f64", "f32", "f16"])
        d = _lattice(rng, 4096, 2_000_000)
        v = d["x"] * d["y"] * d["z"] * d["t"]
        most = min(16, int((12e6 if prec == "f64" else 24e6) / v))
        return dict(do=do, kind=rng.choice(sorted(KINDS)), prec=prec, nrhs=rng.randint(1, max(1, most)), **d)
    if do == "transfer":
        return dict(do=do, prec=rng.choice(["f64", "f64", "f32", "f16"]), nrhs=rng.randint(1, 12),
                    **_lattice(rng, 4096, 660_000))
    if do == "configuration":
        return dict(do=do, nrhs=1, **_lattice(rng, 4096, 660_000))
    if do == "solve":
        solver = rng.choice(["cg", "cg", "bicgstab"])
        return dict(do=do, solver=solver, system="M", prec=rng.choice(["f64", "f32", "f32"]), nrhs=rng.randint(1, 12),
                    kappa=round(rng.uniform(0.118, 0.124), 4), mu=rng.choice([0.0, 0.05, 0.1]), tuned=False,
                    **_lattice(rng, 4096, 140_000))
    if do == "multishift":
        return dict(do=do, nshift=rng.randint(2, 12), nrhs=rng.randint(1, 2), kappa=round(rng.uniform(0.118, 0.124), 4),
                    **_lattice(rng, 4096, 140_000))
    if do == "block":
        return dict(do="solve", solver="block", system="M", prec="f64", nrhs=rng.randint(2, 14),
                    kappa=round(rng.uniform(0.118, 0.124), 4), mu=0.0, tuned=False, **_lattice(rng, 4096, 140_000))
    return dict(do=do, requests=rng.randint(2, 8), maxcols=rng.randint(1, 6), **_lattice(rng, 2048, 16_000))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _dims(case):
    return case["x"], case["y"], case["z"], case["t"]


def _volume(case):
    return case["x"] * case["y"] * case["z"] * case["t"]


def _rng(seed, salt):
    g = torch.Generator(device=DEVICE)
    g.manual_seed((int(seed) * 1_000_003 + salt) % (1 << 62))
    return g


def _matmul3(a, b):
    return sum(a[..., :, k, None] * b[..., None, k, :] for k in range(3))


def _links(case, seed):
    """exp(i EPS H) per link by its Taylor series at half the angle, squared: (4, V, 3, 3) complex128."""
    a = torch.randn((4, _volume(case), 3, 3, 2), dtype=torch.float64, device=DEVICE, generator=_rng(seed, 1))
    a = torch.view_as_complex(a)
    h = 0.5 * (a + a.conj().transpose(-1, -2))
    one = torch.eye(3, dtype=torch.complex128, device=DEVICE)
    h = (0.5j * EPS) * (h - (h.diagonal(dim1=-2, dim2=-1).real.sum(-1) / 3.0)[..., None, None] * one)
    u = one + h / 18.0
    for k in range(17, 0, -1):
        u = one + _matmul3(h, u) / k
    return _matmul3(u, u).contiguous()


def _source(case, seed, ncol, salt=2):
    s = torch.randn((ncol, _volume(case), 4, 3, 2), dtype=torch.float64, device=DEVICE, generator=_rng(seed, salt))
    return torch.view_as_complex(s)


def _shifts(case):
    """Poles of a rational approximation: spread over four decades."""
    n = case["nshift"]
    return [1e-4 * 10.0 ** (4.0 * k / max(1, n - 1)) for k in range(n)]


def _requests(case, seed):
    """(kappa, number of columns) of the requests of a serving case."""
    return [(0.118 + 0.006 * ((seed * 7 + 5 * k) % 13) / 13.0, 1 + (k * k + k // 2) % case["maxcols"])
            for k in range(case["requests"])]


def prepare(case, seed):
    dims, do = _dims(case), case["do"]
    s = {"case": case, "ctx": bq.Context(0)}
    ctx = s["ctx"]
    if do == "transfer":
        s["src"] = _source(case, seed, case["nrhs"])
        s["field"] = bq.Field(ctx, dims, bq.BQ_FULL, PREC[case["prec"]], case["nrhs"])
        s["out"] = torch.zeros_like(s["src"])
        return s
    if do == "configuration":
        s["links"] = _links(case, seed)
        s["in"] = bq.Field(ctx, dims, bq.BQ_FULL, bq.BQ_F64, case["nrhs"])
        s["in"].put(_source(case, seed, case["nrhs"]))
        s["to"] = bq.Field(ctx, dims, bq.BQ_FULL, bq.BQ_F64, case["nrhs"])
        s["out"] = torch.zeros((case["nrhs"], _volume(case), 4, 3), dtype=torch.complex128, device=DEVICE)
        return s
    s["gauge"] = bq.Gauge(ctx, dims, _links(case, seed), t_bc=T_BC)
    if do == "serve":
        s["server"] = bq.Server(ctx, slots=16, chunk=16)
        s["ask"] = [(kappa, _source(case, seed, n, salt=10 + k)) for k, (kappa, n) in enumerate(_requests(case, seed))]
        return s
    n = case["nrhs"]
    if do == "apply":
        s["op"] = bq.Op(s["gauge"], 0.124, CSW, 0.1)
        sub_in, sub_out = bq.OP_SUBSETS[KINDS[case["kind"]]]
        prec = PREC[case["prec"]]
    else:
        s["op"] = bq.Op(s["gauge"], case["kappa"], CSW, case.get("mu", 0.0))
        sub_in = sub_out = bq.BQ_FULL if do == "solve" else bq.BQ_ODD
        prec = bq.BQ_F64
        if case.get("tuned"):
            for p in {"f64", case["prec"]}:
                ctx.tune_set(PREC[p], n, *TUNED_12[p])
    s["in"] = bq.Field(ctx, dims, sub_in, prec, n)
    s["in"].put(_source(case, seed, n))
    outs = case["nshift"] if do == "multishift" else 1
    s["to"] = [bq.Field(ctx, dims, sub_out, prec, n) for _ in range(outs)]
    s["out"] = [torch.zeros((n, _volume(case), 4, 3), dtype=torch.complex128, device=DEVICE) for _ in range(outs)]
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(s):
    case = s["case"]
    do = case["do"]
    if do == "apply":
        s["op"].apply(KINDS[case["kind"]], s["in"], s["to"][0])
    elif do == "transfer":
        s["field"].put(s["src"])
        return s["field"].get(out=s["out"])
    elif do == "configuration":
        gauge = bq.Gauge(s["ctx"], _dims(case), s["links"], t_bc=T_BC)
        op = bq.Op(gauge, 0.124, CSW, 0.1)
        op.apply(bq.BQ_OP_CLOVER, s["in"], s["to"])
        res = {"plaquette": gauge.plaquette(), "clover": s["to"].get(out=s["out"])}
        op.close()
        gauge.close()
        return res
    elif do == "solve":
        s["op"].solve(s["in"], s["to"][0], 1e-10, system=bq.BQ_SYS_M, inner_prec=PREC[case["prec"]],
                      solver=SOLVERS[case["solver"]])
    elif do == "multishift":
        s["op"].solve_multishift(s["in"], s["to"], _shifts(case), 1e-10)
    else:
        server = s["server"]
        tickets = [server.submit(s["gauge"], b, kappa, CSW, 0.0, 1e-10, bq.BQ_F32) for kappa, b in s["ask"]]
        while sum(server.pending()):
            server.step()
        return [server.result(t)[2] for t in tickets]
    for field, out in zip(s["to"], s["out"]):
        field.get(out=out)
    return s["out"]


# ---------------------------------------------------------------------------
# what one pass cannot do without
# ---------------------------------------------------------------------------

def _stencil(sites, n, prec, spinors):
    """Bytes and operations of one stencil over `sites` outputs: 12-real links and packed clover once,
    `spinors` spinor reads or writes for each of n columns; 8 SU(3) half hops and two 6x6 blocks."""
    real = {"f64": 8, "f32": 4, "f16": 2}[prec]
    return sites * (168 * real + 24 * real * spinors * n), sites * n * (1320 + 552)


def work(case):
    v, do = _volume(case), case["do"]
    half, n, canon = v // 2, case.get("nrhs", 1), 192
    if do == "transfer":
        real = {"f64": 8, "f32": 4, "f16": 2}[case["prec"]]
        return {"bytes": n * v * (2 * canon + 2 * 24 * real), "flops": 0}
    if do == "configuration":
        # links in once, the three precisions of links and clover (T, inverse) out once, one application
        return {"bytes": 4 * v * 144 * (1 + 1 + 0.667 + 0.5 + 0.333 + 0.167) + v * 576 * (1 + 1.75 + 1.75) + v * 5 * canon,
                "flops": v * (24 * 3 * 198 + 2 * 1200)}
    if do == "apply":
        calls, sites, spinors = {"M": (2, half, 3), "Mdag": (2, half, 3), "Mhat": (2, half, 2.5),
                                 "MhatdagMhat": (4, half, 2.5), "K1": (1, half, 2), "clover": (1, v, 2)}[case["kind"]]
        b, f = _stencil(sites, n, case["prec"], spinors)
        got = v if case["kind"] in ("M", "Mdag", "clover") else half
        return {"bytes": calls * b + n * got * canon, "flops": calls * f}
    iters = 100  # about what these systems take to 1e-10
    if do == "solve":
        # four stencils and the vector updates (x, p, r) of each iteration in the inner precision
        b, f = _stencil(half, n, case["prec"], 2.75)
        real = {"f64": 8, "f32": 4}[case["prec"]]
        return {"bytes": iters * (4 * b + 5 * 24 * real * half * n) + 4 * n * v * canon, "flops": iters * 4 * f}
    if do == "multishift":
        b, f = _stencil(half, n, "f64", 2.75)
        return {"bytes": iters * (4 * b + canon * half * n * (3 + 4 * case["nshift"])), "flops": iters * 4 * f}
    total = sum(c for _, c in _requests(case, 0))
    b, f = _stencil(half, total, "f32", 2.75)
    return {"bytes": iters * (4 * b + 5 * 96 * half * total), "flops": iters * 4 * f}


# ---------------------------------------------------------------------------
# the same in plain FP64 torch: fields are (columns, t, z, y, x, spin, colour)
# ---------------------------------------------------------------------------

# gamma_mu as (source spin, phase) per spin, chiral basis
_GAMMA = (((3, 1j), (2, 1j), (1, -1j), (0, -1j)), ((3, -1), (2, 1), (1, 1), (0, -1)),
          ((2, 1j), (3, -1j), (0, -1j), (1, 1j)), ((2, 1), (3, 1), (0, 1), (1, 1)))


def _gamma_matrix(mu):
    m = torch.zeros((4, 4), dtype=torch.complex128)
    for s, (q, ph) in enumerate(_GAMMA[mu]):
        m[s, q] = ph
    return m


def _project(p, mu, sign):
    """(1 + sign gamma_mu) p"""
    return torch.stack([p[..., s, :] + (sign * ph) * p[..., q, :] for s, (q, ph) in enumerate(_GAMMA[mu])], dim=-2)


def _colour(u, h):
    return sum(u[..., None, :, k] * h[..., k, None] for k in range(3))


class _Matrix:
    """The fermion matrix of one gauge field on full-lattice arrays."""

    def __init__(self, case, links, kappa, mu):
        x, y, z, t = _dims(case)
        self.shape, self.kappa, self.mu = (t, z, y, x), kappa, mu
        self.u = links.reshape(4, t, z, y, x, 3, 3)
        c = [torch.arange(d, device=DEVICE) for d in (t, z, y, x)]
        odd = (c[0][:, None, None, None] + c[1][:, None, None] + c[2][:, None] + c[3]) % 2
        self.odd = odd.to(torch.float64)[None, ..., None, None]
        self.plaquette = 0.0
        self.clover = self._clover()
        self.inverse = None

    def grid(self, a):
        return a.reshape(a.shape[0], *self.shape, 4, 3)

    def _clover(self):
        """T as two 6x6 blocks per site: (t, z, y, x, block, 6, 6)."""
        u = self.u
        at = lambda a, mu, d: torch.roll(a, -d, dims=3 - mu)  # noqa: E731  a(x + d mu)
        dag = lambda a: a.conj().transpose(-1, -2)  # noqa: E731
        mul = lambda *m: m[0] if len(m) == 1 else mul(_matmul3(m[0], m[1]), *m[2:])  # noqa: E731
        out = torch.zeros((*self.shape, 2, 6, 6), dtype=torch.complex128, device=DEVICE)
        out += torch.eye(6, dtype=torch.complex128, device=DEVICE)
        for m in range(4):
            for n in range(m + 1, 4):
                a, b = u[m], u[n]
                plaq = mul(a, at(b, m, 1), dag(at(a, n, 1)), dag(b))
                self.plaquette += float(plaq.diagonal(dim1=-2, dim2=-1).real.mean()) / 6.0
                q = plaq
                q = q + mul(b, dag(at(at(a, n, 1), m, -1)), dag(at(b, m, -1)), at(a, m, -1))
                am, bmn, amn = at(a, m, -1), at(at(b, m, -1), n, -1), at(at(a, m, -1), n, -1)
                q = q + mul(dag(am), dag(bmn), amn, at(b, n, -1))
                bn, an = at(b, n, -1), at(a, n, -1)
                q = q + mul(dag(bn), an, at(at(b, n, -1), m, 1), dag(a))
                g = -0.125j * (q - dag(q))
                g = g - (g.diagonal(dim1=-2, dim2=-1).sum(-1) / 3.0)[..., None, None] * torch.eye(3, device=DEVICE)
                gm, gn = _gamma_matrix(m), _gamma_matrix(n)
                sigma = 0.5j * (gm @ gn - gn @ gm)
                for blk in range(2):
                    for i in range(2):
                        for k in range(2):
                            c = complex(sigma[2 * blk + i, 2 * blk + k])
                            if c:
                                out[..., blk, 3 * i:3 * i + 3, 3 * k:3 * k + 3] += (self.kappa * CSW * c) * g
        return out

    def T(self, p, inverse=False):
        if inverse and self.inverse is None:  # Gauss-Jordan on the Hermitian positive definite blocks
            a = torch.cat([self.clover, torch.eye(6, dtype=torch.complex128, device=DEVICE).expand_as(self.clover)], -1)
            for k in range(6):
                row = a[..., k, :] / a[..., k, k, None]
                a = a - a[..., :, k, None] * row[..., None, :]
                a[..., k, :] = row
            self.inverse = a[..., 6:].contiguous()
        c = self.inverse if inverse else self.clover
        q = p.reshape(*p.shape[:-2], 2, 6)
        return sum(c[..., :, k] * q[..., k, None] for k in range(6)).reshape(p.shape)

    def D(self, p, dagger=False):
        s = 1 if dagger else -1
        out = torch.zeros_like(p)
        for mu in range(4):
            axis = 4 - mu
            fwd, bwd = torch.roll(p, -1, dims=axis), _colour(self.u[mu].conj().transpose(-1, -2), _project(p, mu, -s))
            bwd = torch.roll(bwd, 1, dims=axis)
            if mu == 3:
                e = math.exp(-self.mu if dagger else self.mu)
                fwd, bwd = fwd * e, bwd / e
                fwd[:, -1] *= T_BC
                bwd[:, 0] *= T_BC
            out += _colour(self.u[mu], _project(fwd, mu, s)) + bwd
        return out

    def M(self, p, dagger=False):
        return self.T(p) - self.kappa * self.D(p, dagger)

    def K1(self, p, dagger=False):
        return self.T((1 - self.odd) * self.D(self.odd * p, dagger), inverse=True)

    def Mhat(self, p, dagger=False):
        return self.odd * (self.T(p) - self.kappa**2 * self.D(self.K1(p, dagger), dagger))


def _cg(a, b, tol=1e-14, most=3000):
    """CG on a Hermitian positive definite operator, every column with scalars of its own."""
    dot = lambda p, q: (p.conj() * q).real.flatten(1).sum(1)  # noqa: E731
    col = lambda c: c[:, None, None, None, None, None, None]  # noqa: E731
    x, r, p = torch.zeros_like(b), b.clone(), b.clone()
    rho = dot(r, r)
    stop = rho * tol**2
    for _ in range(most):
        if bool((rho <= stop).all()):
            break
        q = a(p)
        alpha = rho / dot(p, q).clamp_min(1e-300)
        x += col(alpha) * p
        r -= col(alpha) * q
        new = dot(r, r)
        p = r + col(new / rho.clamp_min(1e-300)) * p
        rho = new
    return x


def exact(case, seed):
    do = case["do"]
    if do == "transfer":
        return _source(case, seed, case["nrhs"])
    if do in ("solve", "multishift") and _volume(case) * case["nrhs"] * case.get("nshift", 1) > 2_000_000:
        return None
    links = _links(case, seed)
    if do == "serve":
        out = []
        for k, (kappa, n) in enumerate(_requests(case, seed)):
            m, b = _Matrix(case, links, kappa, 0.0), _source(case, seed, n, salt=10 + k)
            x = _cg(lambda p: m.M(m.M(p), dagger=True), m.M(m.grid(b), dagger=True))
            out.append(x.reshape(b.shape))
        return out
    if do in ("apply", "configuration"):
        m = _Matrix(case, links, 0.124, 0.1)
    else:
        m = _Matrix(case, links, case["kappa"], case.get("mu", 0.0))
    b = _source(case, seed, case["nrhs"])
    p = m.grid(b)
    if do == "configuration":
        return {"plaquette": m.plaquette, "clover": m.T(p).reshape(b.shape)}
    if do == "apply":
        x = {"M": lambda: m.M(p), "Mdag": lambda: m.M(p, dagger=True), "Mhat": lambda: m.Mhat(m.odd * p),
             "MhatdagMhat": lambda: m.Mhat(m.Mhat(m.odd * p), dagger=True), "K1": lambda: m.K1(p),
             "clover": lambda: m.T(p)}[case["kind"]]()
        return [x.reshape(b.shape)]
    if do == "solve":
        return [_cg(lambda q: m.M(m.M(q), dagger=True), m.M(p, dagger=True)).reshape(b.shape)]
    b_odd = m.odd * p
    return [_cg(lambda q: m.Mhat(m.Mhat(q), dagger=True) + s * q, b_odd).reshape(b.shape) for s in _shifts(case)]
