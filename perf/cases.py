"""Performance cases of the framework's public entry points (``paper_1405_4524_amd.a2a``).

A case is one call, or one short sequence of calls, that a program built on the library makes:
solves of noise sources on a resident field, a whole configuration from links to correlators, a
mixed batch through the serving engine, an operator application on a fresh field, and the
contractions (pion, pi-pi, momentum-projected, outer-product fill, diagrams with point
propagators).  ``listed`` holds the sizes of the named workloads and studies, ``draw`` more of the
same ranges.  Inputs are drawn on the GPU from the seed: near-identity SU(3) links exp(i eps H)
with H Gaussian, traceless and Hermitian, complex-Z2 noise, and, for the contractions alone,
Gaussian solution fields on top of the noise.  ``exact`` evaluates the definitions in complex128
with plain torch.
"""
import math
import weakref

import numpy as np
import torch

DEVICE = "cuda" if torch.cuda.is_available() else "cpu"
C128, F64 = torch.complex128, torch.float64
PREC = {"f64": 0, "f32": 1, "f16": 2, "bf16": 3}
REAL_BYTES = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}
SCHEME = {"none": 0, "t": 1, "sc": 2, "tsc": 3}
MOMS = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (1, 1, 0), (1, 1, 1), (2, 0, 0)]
TOL = 1e-10
NOMINAL_ITERS = 40  # BiCGStab iterations to 1e-10 at the workloads' kappa (35-48)


# ------------------------------------------------------------------------------------------
# cases
# ------------------------------------------------------------------------------------------
def _solve(name, L, T, n, prec, kappa, csw, eps):
    return dict(name=name, kind="solve", X=L, Y=L, Z=L, T=T, n=n, prec=prec, kappa=kappa, csw=csw, eps=eps)


def listed():
    return [
        # smallest solve: a user's first call and the smoke test; launches and latency count
        _solve("solve_4c8_f16_n4", 4, 8, 4, "f16", 0.120, 1.0, 0.20),
        # a serving-sized request: 20 sources are one 16-lane group and four per-slot sources
        _solve("solve_8c16_f16_n20", 8, 16, 20, "f16", 0.125, 1.2, 0.30),
        # the plain FP64 method on the solver + pi-pi workload
        _solve("solve_16c32_f64_n16", 16, 32, 16, "f64", 0.125, 1.2, 0.30),
        # BF16 inner solves of 32 sources, two lane tiles
        _solve("solve_24c48_bf16_n32", 24, 48, 32, "bf16", 0.130, 1.5, 0.35),
        # the headline workload: one configuration from links to pion and pi-pi correlators
        dict(name="config_32c64_f16_n48", kind="config", X=32, Y=32, Z=32, T=64, n=48, prec="f16", kappa=0.130,
             csw=1.5, eps=0.35),
        # continuous batching: requests on three resident lattices in one engine, any batch shape
        dict(name="serve_3lattices_f16", kind="serve", L1=8, T1=16, n1=26, L2=16, T2=32, n2=31, L3=24, T3=48, n3=30,
             prec="f16", kappa=0.130, csw=1.5, eps=0.35),
        # full operator on a fresh field with unequal ragged extents: field ingest, clover, apply
        dict(name="apply_12x10x6x14_f64_n3", kind="apply", X=12, Y=10, Z=6, T=14, n=3, prec="f64", dagger=True,
             kappa=0.125, csw=1.2, eps=0.30),
        # pion correlator and operators of the smallest lattice: pure call latency
        dict(name="pion_4c8_n4", kind="pion", X=4, Y=4, Z=4, T=8, n=4),
        # pi-pi diagrams and pion of the headline workload's sources and solutions
        dict(name="pipi_32c64_n48", kind="pipi", X=32, Y=32, Z=32, T=64, n=48),
        # time-spin-colour diluted sources of four noise vectors, six momenta
        dict(name="momentum_8c16_tsc_n768", kind="momentum", X=8, Y=8, Z=8, T=16, nv=4, scheme="tsc", nmom=6),
        # outer-product fill of one (t, t_src) block of the all-to-all propagator
        dict(name="fill_8c16_n1024", kind="fill", X=8, Y=8, Z=8, T=16, n=1024, dagger=False),
        # Sec. 8 diagrams from 12 point solutions and two noise sets
        dict(name="mixed_8c16_n256", kind="mixed", X=8, Y=8, Z=8, T=16, n1=256, n2=256, t0=3),
    ]


def _even(rng, lo, hi):
    """An even number, spread over the logarithm of [lo, hi]."""
    return max(lo, min(hi, 2 * round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / 2)))


def _count(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def _dims(rng, lo, hi, t_hi):
    L = _even(rng, lo, hi)
    near = lambda: max(2, min(hi, L + rng.choice((-2, 0, 0, 2))))  # noqa: E731
    return dict(X=near(), Y=near(), Z=near(), T=_even(rng, 4, t_hi))


def draw(rng):
    kind = rng.choice(("solve", "solve", "solve", "config", "serve", "apply", "pion", "pipi", "momentum", "fill", "mixed"))
    phys = dict(kappa=round(rng.uniform(0.120, 0.130), 4), csw=round(rng.uniform(1.0, 1.5), 2), eps=round(rng.uniform(0.20, 0.35), 2))
    if kind in ("solve", "config"):
        c = dict(kind=kind, prec=rng.choice(("f16", "f16", "bf16", "f32", "f64")), **_dims(rng, 4, 24, 48), **phys)
        V = c["X"] * c["Y"] * c["Z"] * c["T"]
        # the FP64 and FP32 modes cost three and two times the 16-bit ones
        most = (24**3 * 48 * 32) // {"f64": 8, "f32": 4}.get(c["prec"], 1)
        c["n"] = _count(rng, 1, max(1, min(96, most // V)))
        if kind == "config":
            c["n"] = max(4, min(96, c["n"] // 4 * 4))
        return c
    if kind == "serve":
        L = [_even(rng, 4, 16) for _ in range(3)]
        c = dict(kind=kind, prec=rng.choice(("f16", "bf16")), **phys)
        for k in range(3):
            c.update({"L%d" % (k + 1): L[k], "T%d" % (k + 1): _even(rng, 4, 32), "n%d" % (k + 1): _count(rng, 1, 64)})
        return c
    if kind == "apply":
        return dict(kind=kind, prec="f64", dagger=rng.random() < 0.5, n=_count(rng, 1, 24),
                    **_dims(rng, 4, 24, 32), **phys)
    if kind in ("pion", "pipi"):
        c = dict(kind=kind, **_dims(rng, 4, 32, 64))
        most = max(4, (32**3 * 64 * 48) // (c["X"] * c["Y"] * c["Z"] * c["T"]))
        c["n"] = _count(rng, 2, min(128, most)) if kind == "pion" else 4 * _count(rng, 1, min(32, most // 4))
        return c
    if kind == "momentum":
        c = dict(kind=kind, scheme=rng.choice(("none", "t", "sc", "tsc")), nmom=rng.randint(1, 6), **_dims(rng, 4, 12, 16))
        pieces = {"none": 1, "t": c["T"], "sc": 12, "tsc": 12 * c["T"]}[c["scheme"]]
        room = min(768, (768 * 8**3 * 16) // (c["X"] * c["Y"] * c["Z"] * c["T"]))
        c["nv"] = _count(rng, 2, max(2, min(64, room // pieces)))
        return c
    if kind == "fill":
        return dict(kind=kind, n=_count(rng, 8, 1024), dagger=rng.random() < 0.5, **_dims(rng, 4, 8, 16))
    c = dict(kind="mixed", n1=_count(rng, 4, 256), n2=_count(rng, 4, 256), **_dims(rng, 4, 8, 16))
    c["t0"] = rng.randrange(c["T"])
    return c


# ------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------
def _generator(seed, stream):
    return torch.Generator(DEVICE).manual_seed(int(seed) * 64 + stream)


def _matmul3(a, b):
    return (a[..., :, :, None] * b[..., None, :, :]).sum(-2)


def _links(dims, eps, seed, stream=0):
    """[T][Z][Y][X][4][3][3] links exp(i eps H): Taylor series of the exponential of an eighth,
    squared three times."""
    X, Y, Z, T = dims
    gen = _generator(seed, stream)
    U = torch.empty((T, Z, Y, X, 4, 3, 3), dtype=C128, device=DEVICE)
    for mu in range(4):
        a = torch.view_as_complex(torch.randn((T, Z, Y, X, 3, 3, 2), dtype=F64, device=DEVICE, generator=gen))
        h = 0.5 * (a + a.mH)
        eye = torch.eye(3, dtype=C128, device=DEVICE)
        h = h - (torch.diagonal(h, dim1=-2, dim2=-1).sum(-1) / 3)[..., None, None] * eye
        m = (1j * eps / 8) * h
        u = eye + m / 14
        for k in range(13, 0, -1):
            u = eye + _matmul3(m, u) / k
        for _ in range(3):
            u = _matmul3(u, u)
        U[..., mu, :, :] = u
    return U


def _noise(dims, n, seed, stream=1):
    """n complex-Z2 sources (+-1 +- i)/sqrt(2), [n][T][Z][Y][X][4][3]."""
    X, Y, Z, T = dims
    gen = _generator(seed, stream)
    out = torch.empty((n, T, Z, Y, X, 4, 3, 2), dtype=F64, device=DEVICE)
    for s in range(n):
        bits = torch.randint(0, 2, out.shape[1:], dtype=torch.int8, device=DEVICE, generator=gen)
        out[s] = (1 - 2 * bits.double()) * math.sqrt(0.5)
    return torch.view_as_complex(out)


def _fields(dims, n, seed, stream=2):
    """n Gaussian fields, [n][T][Z][Y][X][4][3]."""
    X, Y, Z, T = dims
    gen = _generator(seed, stream)
    out = torch.empty((n, T, Z, Y, X, 4, 3, 2), dtype=F64, device=DEVICE)
    for s in range(n):
        out[s] = torch.randn(out.shape[1:], dtype=F64, device=DEVICE, generator=gen)
    return torch.view_as_complex(out)


def _solutions(noise, seed, stream=2):
    """Stand-ins for the solutions of the noise sources: the noise itself plus a Gaussian field."""
    n, T, Z, Y, X = noise.shape[:5]
    out = _fields((X, Y, Z, T), n, seed, stream)
    out.mul_(0.5)
    for s in range(n):
        out[s] += noise[s]
    return out


def _dilute(noise, scheme):
    """Every noise vector split into its pieces, in the order of the dilution index."""
    n, T = noise.shape[:2]
    if scheme == "none":
        return noise
    D = {"t": T, "sc": 12, "tsc": 12 * T}[scheme]
    out = torch.zeros((n, D) + tuple(noise.shape[1:]), dtype=C128, device=noise.device)
    for d in range(D):
        t = d if scheme == "t" else d // 12
        s, c = (d % 12) // 3, d % 3
        if scheme == "t":
            out[:, d, t] = noise[:, t]
        elif scheme == "sc":
            out[:, d, ..., s, c] = noise[..., s, c]
        else:
            out[:, d, t, ..., s, c] = noise[:, t, ..., s, c]
    return out.reshape((n * D,) + tuple(noise.shape[1:]))


def _case_dims(case):
    return (case["X"], case["Y"], case["Z"], case["T"])


def _inputs(case, seed):
    """The tensors of a case, from the seed alone."""
    kind = case["kind"]
    if kind == "serve":
        lat = [(case["L%d" % k],) * 3 + (case["T%d" % k],) for k in (1, 2, 3)]
        return dict(dims=lat, links=[_links(d, case["eps"], seed, 8 * k) for k, d in enumerate(lat)],
                    src=[_noise(d, case["n%d" % (k + 1)], seed, 8 * k + 1) for k, d in enumerate(lat)])
    dims = _case_dims(case)
    if kind in ("solve", "config"):
        return dict(dims=dims, links=_links(dims, case["eps"], seed), src=_noise(dims, case["n"], seed))
    if kind == "apply":
        return dict(dims=dims, links=_links(dims, case["eps"], seed), src=_fields(dims, case["n"], seed))
    if kind == "momentum":
        src = _dilute(_noise(dims, case["nv"], seed), case["scheme"])
        return dict(dims=dims, src=src, sol=_fields(dims, src.shape[0], seed))
    if kind == "mixed":
        src = [_noise(dims, case["n1"], seed, 1), _noise(dims, case["n2"], seed, 3)]
        return dict(dims=dims, src=src, sol=[_solutions(src[0], seed, 2), _solutions(src[1], seed, 4)],
                    point=_fields(dims, 12, seed, 5))
    src = _noise(dims, case["n"], seed)
    return dict(dims=dims, src=src, sol=_solutions(src, seed))


# ------------------------------------------------------------------------------------------
# what a program keeps, and one pass
# ------------------------------------------------------------------------------------------
class _Session:
    """The context of a process, shared by its states, as a program keeps one per GPU."""

    current = None  # weak reference

    def __init__(self):
        from paper_1405_4524_amd import a2a

        self.a2a = a2a
        self.ctx = a2a.Context(0)

    def __del__(self):
        self.ctx.finalize()

    @classmethod
    def get(cls):
        s = cls.current() if cls.current else None
        if s is None:
            s = cls()
            cls.current = weakref.ref(s)
        return s


class _State:
    """One program's inputs, output buffers, resident fields and engine."""

    def __init__(self, case, seed):
        self.case = case
        self.session = _Session.get()
        self.gauges, self.clovers, self.engine = [], [], None
        self.__dict__.update(_inputs(case, seed))
        kind = case["kind"]
        if DEVICE == "cuda":
            torch.cuda.synchronize()
        if kind == "solve":
            self.resident(self.links, self.dims)
        if kind == "serve":
            for U, d in zip(self.links, self.dims):
                self.resident(U, d)
            self.engine = self.session.ctx.engine_create('{"max_slots": 256}')
            self.sol = [torch.zeros_like(s) for s in self.src]
        if kind in ("solve", "serve"):
            self.links = None
        if kind in ("solve", "config", "apply"):
            self.sol = torch.zeros_like(self.src)
        if kind == "fill":
            M = 12 * case["X"] * case["Y"] * case["Z"]
            self.S = torch.empty((M, M), dtype=C128, device=DEVICE)

    def resident(self, links, dims):
        ctx = self.session.ctx
        self.gauges.append(ctx.load_gauge_dev(links, dims, -1))
        self.clovers.append(ctx.load_clover(self.gauges[-1], self.case["csw"]))

    def __del__(self):
        if self.engine is not None:
            self.engine.destroy()
        for g in self.gauges:
            self.session.ctx.unload(g)


def prepare(case, seed):
    return _State(case, seed)


def run(state):
    s, case, ctx, a2a = state, state.case, state.session.ctx, state.session.a2a
    kind = case["kind"]
    if kind == "solve":
        ctx.solve_propagators_dev(s.clovers[0], s.src, s.sol, case["n"], case["kappa"], case["csw"], tol=TOL,
                                  prec=PREC[case["prec"]])
        return s.sol
    if kind == "config":
        g = ctx.load_gauge_dev(s.links, s.dims, -1)
        c = ctx.load_clover(g, case["csw"])
        ctx.solve_propagators_dev(c, s.src, s.sol, case["n"], case["kappa"], case["csw"], tol=TOL,
                                  prec=PREC[case["prec"]])
        d, v, p = ctx.contract_pipi_2pt_dev(s.src, s.sol, case["n"], s.dims, want_pion=True)
        ctx.unload(g)
        return {"solutions": s.sol, "pipi": d, "loops": v, "pion": p}
    if kind == "serve":
        n = [case["n%d" % k] for k in (1, 2, 3)]
        tickets = [s.engine.submit(c, case["kappa"], x, k, TOL, PREC[case["prec"]], 100000, y)
                   for c, x, k, y in zip(s.clovers, s.src, n, s.sol)]
        while True:
            s.engine.step(8)
            if all(s.engine.poll(t, k)[0] != 0 for t, k in zip(tickets, n)):
                return s.sol
    if kind == "apply":
        g = ctx.load_gauge_dev(s.links, s.dims, -1)
        c = ctx.load_clover(g, case["csw"])
        ctx.dslash_clover_dev(c, case["kappa"], s.src, s.sol, case["n"], op=a2a.OP_FULL_D, dagger=case["dagger"],
                              prec=PREC[case["prec"]])
        ctx.unload(g)
        return s.sol
    if kind == "pion":
        return ctx.contract_pion_2pt_dev(s.src, s.sol, case["n"], s.dims, want_O=True)
    if kind == "pipi":
        return ctx.contract_pipi_2pt_dev(s.src, s.sol, case["n"], s.dims, want_pion=True)
    if kind == "momentum":
        return ctx.contract_pion_mom_dev(s.src, s.sol, s.src.shape[0], s.dims, MOMS[:case["nmom"]],
                                         scheme=SCHEME[case["scheme"]])
    if kind == "fill":
        ctx.fill_propagator_dev(s.sol, s.src, case["n"], s.dims, 0, case["T"] // 2, s.S, dagger=case["dagger"])
        return s.S
    return ctx.contract_pipi_mixed_dev(s.point, case["t0"], s.src[0], s.sol[0], case["n1"], s.src[1], s.sol[1],
                                       case["n2"], s.dims)


# ------------------------------------------------------------------------------------------
# bytes and operations a pass cannot do without
# ------------------------------------------------------------------------------------------
def _solve_work(V, n, prec):
    """Links, sources and solutions once in FP64; per iteration two Schur operators, each two
    half-lattice stencils (1320 flop and a clover product of 504 per site) that read and write one
    half-lattice spinor of the storage format, and the Krylov updates' eight half-lattice spinors."""
    b = REAL_BYTES[prec]
    half = V * n * 12 * b  # one half-lattice spinor of every source
    return dict(bytes=V * 4 * 144 + 2 * V * n * 192 + NOMINAL_ITERS * 16 * half,
                flops=NOMINAL_ITERS * V * n * 2 * (1320 + 504 + 96))


def _gram_work(V, n, m):
    """n x m inner products on every timeslice: both operands once, 8 flop a complex product."""
    return dict(bytes=192 * V * (n + m), flops=96 * V * n * m)


def work(case):
    kind = case["kind"]
    if kind == "serve":
        parts = [_solve_work(case["L%d" % k] ** 3 * case["T%d" % k], case["n%d" % k], case["prec"]) for k in (1, 2, 3)]
        return {key: sum(p[key] for p in parts) for key in ("bytes", "flops")}
    V, T = case["X"] * case["Y"] * case["Z"] * case["T"], case["T"]
    if kind == "solve":
        return _solve_work(V, case["n"], case["prec"])
    if kind == "config":
        a, b = _solve_work(V, case["n"], case["prec"]), _gram_work(V, case["n"], case["n"])
        return {key: a[key] + b[key] for key in a}
    if kind == "apply":
        return dict(bytes=V * 4 * 144 + 2 * V * case["n"] * 192, flops=V * case["n"] * (1320 + 504 + 48) + V * 50000)
    if kind in ("pion", "pipi"):
        return _gram_work(V, case["n"], case["n"])
    if kind == "momentum":
        pieces = {"none": 1, "t": T, "sc": 12, "tsc": 12 * T}[case["scheme"]]
        n = case["nv"] * pieces
        # O(t, p) and O(t, -p); a time-diluted source contributes on its own timeslice only
        on_t = T if case["scheme"] in ("t", "tsc") else 1
        return dict(bytes=192 * V * (n + n // on_t), flops=2 * case["nmom"] * 96 * V * n * n // on_t)
    M = 12 * V // T
    if kind == "fill":
        return dict(bytes=16 * (2 * M * case["n"] + M * M), flops=8 * M * M * case["n"])
    n1, n2 = case["n1"], case["n2"]
    return dict(bytes=192 * V * (2 * n1 + 2 * n2 + 12), flops=2 * 96 * V * n1 * n2 + 96 * V * 12 * (n2 + 12))


# ------------------------------------------------------------------------------------------
# the definitions in complex128
# ------------------------------------------------------------------------------------------
def _gammas():
    """gamma_1..4 in the chiral basis, gamma_k = [[0, -i s_k], [i s_k, 0]], gamma_4 = [[0, 1], [1, 0]]."""
    s = [np.array([[0, 1], [1, 0]], complex), np.array([[0, -1j], [1j, 0]]), np.array([[1, 0], [0, -1]], complex)]
    z, one = np.zeros((2, 2)), np.eye(2)
    return [np.block([[z, -1j * m], [1j * m, z]]) for m in s] + [np.block([[z, one], [one, z]]).astype(complex)]


AXIS = (3, 2, 1, 0)  # lattice axis of direction mu in a [T][Z][Y][X] array


class _Dirac:
    """D = A - kappa H on vectors [T][Z][Y][X][4][3][n]."""

    def __init__(self, U, kappa, csw):
        self.U, self.kappa, self.gammas = U, kappa, _gammas()
        dims = U.shape[:4]
        A = torch.zeros(tuple(dims) + (4, 3, 4, 3), dtype=C128, device=U.device)
        for mu in range(4):
            for nu in range(mu + 1, 4):
                F = self.field_strength(mu, nu)
                sigma = 0.5j * (self.gammas[mu] @ self.gammas[nu] - self.gammas[nu] @ self.gammas[mu])
                for a, b in zip(*np.nonzero(sigma)):
                    A[..., a, :, b, :] += 1j * kappa * csw * complex(sigma[a, b]) * F
        A = A.reshape(tuple(dims) + (12, 12))
        A += torch.eye(12, dtype=C128, device=U.device)
        self.A = A.reshape(-1, 12, 12)

    def field_strength(self, mu, nu):
        """(Q - Q^dag) / 8 over the four counter-clockwise leaves of the plane."""
        at = lambda m, d_mu, d_nu: torch.roll(self.U[..., m, :, :], (-d_mu, -d_nu), (AXIS[mu], AXIS[nu]))  # noqa: E731
        mul = lambda *f: _matmul3(_matmul3(f[0], f[1]), _matmul3(f[2], f[3]))  # noqa: E731
        Q = mul(at(mu, 0, 0), at(nu, 1, 0), at(mu, 0, 1).mH, at(nu, 0, 0).mH)
        Q += mul(at(nu, 0, 0), at(mu, -1, 1).mH, at(nu, -1, 0).mH, at(mu, -1, 0))
        Q += mul(at(mu, -1, 0).mH, at(nu, -1, -1).mH, at(mu, -1, -1), at(nu, 0, -1))
        Q += mul(at(nu, 0, -1).mH, at(mu, 0, -1), at(nu, 1, -1), at(mu, 0, 0).mH)
        return (Q - Q.mH) / 8

    def hop_one(self, mu, psi):
        """The two hops of one direction."""
        U, g, ax = self.U[..., mu, :, :], self.gammas[mu], AXIS[mu]
        col = [int(np.nonzero(g[r])[0][0]) for r in range(4)]
        val = [complex(g[r, col[r]]) for r in range(4)]

        def spin(v, sign):  # (1 + sign gamma_mu) v
            return torch.stack([v[..., r, :, :] + sign * val[r] * v[..., col[r], :, :] for r in range(4)], -3)

        def colour(W, v):
            return torch.stack([sum(W[..., a, b, None, None] * v[..., b, :] for b in range(3)) for a in range(3)], -2)

        f = torch.roll(psi, -1, ax)
        if mu == 3:
            f[-1] = -f[-1]
        out = spin(colour(U, f), -1)
        b = torch.roll(colour(U.mH, psi), 1, ax)
        if mu == 3:
            b[0] = -b[0]
        return out + spin(b, +1)

    def __call__(self, psi):
        n = psi.shape[-1]
        out = torch.matmul(self.A, psi.reshape(-1, 12, n)).reshape(psi.shape)
        for mu in range(4):
            out -= self.kappa * self.hop_one(mu, psi)
        return out


def _solve_exact(D, b, tol=1e-13):
    """BiCGStab on all columns of b at once, restarted from the true residual."""
    dot = lambda u, v: (u.conj() * v).reshape(-1, u.shape[-1]).sum(0)  # noqa: E731
    norm = lambda u: dot(u, u).real.sqrt()  # noqa: E731
    x, bn = torch.zeros_like(b), norm(b)
    for _ in range(3):
        r = b - D(x)
        if bool((norm(r) <= tol * bn).all()):
            break
        rh, p, rho = r.clone(), r.clone(), dot(r, r)
        for _ in range(400):
            v = D(p)
            alpha = rho / dot(rh, v)
            s = r - alpha * v
            t = D(s)
            omega = dot(t, s) / dot(t, t)
            x += alpha * p + omega * s
            r = s - omega * t
            if bool((norm(r) <= tol * bn).all()):
                break
            new = dot(rh, r)
            p = r + (new / rho) * (alpha / omega) * (p - omega * v)
            rho = new
    return x


def _last(v):
    """[n][T][Z][Y][X][4][3] -> [T][Z][Y][X][4][3][n]."""
    return v.movedim(0, -1).contiguous()


def _first(v):
    return v.movedim(-1, 0).contiguous()


def _propagators(links, src, kappa, csw):
    """D^-1 of the sources, sixteen at a time; None where it would take too long."""
    if links.shape[:4].numel() * src.shape[0] > 16**3 * 32 * 32:
        return None
    D = _Dirac(links, kappa, csw)
    return torch.cat([_first(_solve_exact(D, _last(src[k:k + 16]))) for k in range(0, src.shape[0], 16)])


def _timeslices(v):
    """[n][T][...] -> [T][n][12 Z Y X]."""
    return v.reshape(v.shape[0], v.shape[1], -1).movedim(1, 0)


def _gram(a, b, weight=None):
    """[T][na][nb] inner products <a_i, w b_j>_t."""
    A, B = _timeslices(a), _timeslices(b)
    return torch.stack([torch.matmul(A[t].conj(), (B[t] * weight if weight is not None else B[t]).T)
                        for t in range(A.shape[0])])


def _gamma5(dims):
    g5 = torch.tensor([1.0] * 6 + [-1.0] * 6, dtype=C128, device=DEVICE)
    return g5.repeat(dims[0] * dims[1] * dims[2])


def _correlate(Op, Om, keep, norm):
    """sum_t0 sum_ab keep_ab Op[t0 + dt]_ab Om[t0]_ba / norm."""
    K = Om.transpose(1, 2) * keep
    T = Op.shape[0]
    return np.array([complex((torch.roll(Op, -dt, 0) * K).sum()) / norm for dt in range(T)])


def _pion_of(O):
    T, n = O.shape[:2]
    keep = 1.0 - torch.eye(n, dtype=F64, device=O.device)
    return _correlate(O, O, keep, T * n * (n - 1))


def _pipi_of(O):
    T, n = O.shape[:2]
    m = n // 4
    B = lambda g, h: O[:, g * m:(g + 1) * m, h * m:(h + 1) * m]  # noqa: E731
    loop = lambda g, h, sh: torch.einsum("tij,tji->t", torch.roll(B(g, h), -sh, 0), B(h, g)) / m**2  # noqa: E731
    v12, v34 = loop(0, 1, 0), loop(2, 3, 0)
    b12, b23, b34, b41 = B(0, 1), B(1, 2), B(2, 3), B(3, 0)
    d = np.empty((4, T), complex)
    mm = lambda *f: torch.matmul(torch.matmul(f[0], f[1]), torch.matmul(f[2], f[3]))  # noqa: E731
    tr = lambda M: torch.diagonal(M, dim1=-2, dim2=-1).sum(-1)  # noqa: E731
    for dt in range(T):
        at = lambda M: torch.roll(M, -dt, 0).contiguous()  # noqa: B023, E731
        d[0, dt] = complex((loop(0, 1, dt) * loop(2, 3, dt)).mean())
        d[1, dt] = complex((torch.roll(v12, -dt) * v34).mean())
        d[2, dt] = complex(tr(mm(b12.contiguous(), at(b23), at(b34), b41.contiguous())).mean()) / m**4
        d[3, dt] = complex(tr(mm(at(b12), at(b23), b34.contiguous(), b41.contiguous())).mean()) / m**4
    return d, v12.cpu().numpy()


def _mixed_exact(s, case):
    """Sec. 8's traces in factorised form: every propagator is a sum of outer products, so a trace over
    sites and spin-colour is a product of inner products."""
    t0, n1, n2 = case["t0"], case["n1"], case["n2"]
    (e1, e2), (x1, x2), P = s["src"], s["sol"], s["point"]
    G, F, Pn = _gram(e1, e2), _gram(x1, x2), _gram(P, P)
    A, B = _gram(P, x1)[t0], _gram(x2, P)
    T = G.shape[0]
    d, pc = np.empty((4, T), complex), np.empty((3, T), complex)
    c0 = complex(torch.trace(Pn[t0]))
    for dt in range(T):
        t = (t0 + dt) % T
        cs = complex((G[t0] * F[t].conj()).sum()) / (n1 * n2)
        lp = complex((G[t] * F[t].conj()).sum()) / (n1 * n2)
        d2 = complex((G[t] * torch.matmul(B[t], A).T).sum()) / (n1 * n2)
        cp = complex(torch.trace(Pn[t]))
        d[:, dt] = (cp * cs, lp * c0, d2, d2.conjugate())
        pc[:, dt] = (cp, cs, lp)
    return d, pc


def _momentum_exact(s, case):
    X, Y, Z, T = s["dims"]
    n = s["src"].shape[0]
    group = n // case["nv"]
    who = torch.arange(n, device=DEVICE) // group
    keep = (who[:, None] != who[None, :]).to(F64)
    g5 = _gamma5(s["dims"])
    z, y, x = torch.meshgrid(*(torch.arange(k, dtype=F64, device=DEVICE) for k in (Z, Y, X)), indexing="ij")
    out = np.empty((case["nmom"], T), complex)
    for m, p in enumerate(MOMS[:case["nmom"]]):
        w = torch.exp(-2j * math.pi * (p[0] * x / X + p[1] * y / Y + p[2] * z / Z)).reshape(-1).repeat_interleave(12)
        Op, Om = _gram(s["src"], s["sol"], g5 * w), _gram(s["src"], s["sol"], g5 * w.conj())
        out[m] = _correlate(Op, Om, keep, T * case["nv"] * (case["nv"] - 1))
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("solve", "config"):  # not those whose solves take too long
        if case["X"] * case["Y"] * case["Z"] * case["T"] * case["n"] > 16**3 * 32 * 32:
            return None
    s = _inputs(case, seed)
    dims = s["dims"]
    if kind == "solve":
        return _propagators(s["links"], s["src"], case["kappa"], case["csw"])
    if kind == "config":
        sol = _propagators(s["links"], s["src"], case["kappa"], case["csw"])
        O = _gram(s["src"], sol, _gamma5(dims))
        d, v = _pipi_of(O)
        return {"solutions": sol, "pipi": d, "loops": v, "pion": _pion_of(O)}
    if kind == "serve":
        return [_propagators(U, b, case["kappa"], case["csw"]) for U, b in zip(s["links"], s["src"])]
    if kind == "apply":
        D = _Dirac(s["links"], case["kappa"], case["csw"])
        g5 = torch.tensor([1.0, 1.0, -1.0, -1.0], dtype=C128, device=DEVICE)[:, None, None]
        v = _last(s["src"])
        return _first(g5 * D(g5 * v) if case["dagger"] else D(v))
    if kind in ("pion", "pipi"):
        O = _gram(s["src"], s["sol"], _gamma5(dims))
        if kind == "pion":
            return _pion_of(O), O.cpu().numpy()
        return (*_pipi_of(O), _pion_of(O))
    if kind == "momentum":
        return _momentum_exact(s, case)
    if kind == "fill":
        T = case["T"]
        P = s["sol"][:, T // 2].reshape(case["n"], -1)
        Q = s["src"][:, 0].reshape(case["n"], -1)
        S = torch.matmul(P.T, Q.conj()) / case["n"]
        if case["dagger"]:  # the spin-colour dagger of every 12 x 12 block
            m = S.shape[0] // 12
            S = S.reshape(m, 12, m, 12).transpose(1, 3).conj().reshape(S.shape).contiguous()
        return S
    return _mixed_exact(s, case)
