"""Performance cases of the library: the calls a program that estimates disconnected loops makes.

A case names one public entry point and its sizes.  `listed` gives the fixed set, `draw` more of the same
ranges, `prepare` the inputs and handles a program holds before the call, `run` one pass, `work` the bytes and
operations a pass cannot do without, and `exact` the same outputs from plain torch in 64 bits.

Kinds: "apply" (an operator on given fields), "solve" (quark propagators from given sources), "loops" (per-noise
loop estimates), "tsm" (truncated solver method), "grad" (loops and their gradients through autograd), "batch"
(several lattices at once) and "smear" (Gaussian smearing of given fields).  Gauge fields are synthetic SU(3)
fields exp(i eps H) as in `synth`, made on the GPU; (eps, kappa) pairs and lattice shapes are those of
`synth.WORKLOADS` and shapes around them.
"""
import math

import numpy as np
import torch

import paper_1012_5168_amd as dl
from paper_1012_5168_amd.autograd import disconnected_loops

PREC = {"f64": dl.DL_F64, "f32": dl.DL_F32, "f16": dl.DL_F16, "bf16": dl.DL_BF16}
BYTES = {"f64": 16, "f32": 8, "f16": 4, "bf16": 4}  # of one stored complex number
OPS = {"dhop": dl.DL_OP_DHOP, "m": dl.DL_OP_M, "mdag": dl.DL_OP_MDAG, "mhat": dl.DL_OP_MHAT}
SPIN_COLOUR, CUBIC, EVEN_ODD, SPIN = dl.DL_DIL_SPIN_COLOUR, dl.DL_DIL_CUBIC, dl.DL_DIL_EVEN_ODD, dl.DL_DIL_SPIN
ALPHA = 0.5  # of the Gaussian smearing

# (eps, kappa) of the workloads
FIELDS = [(0.5, 0.12), (0.30, 0.145), (0.35, 0.148), (0.35, 0.150), (0.40, 0.150)]


def _case(name, kind, dims, eps, kappa, **more):
    c = {"kind": kind, "X": dims[0], "Y": dims[1], "Z": dims[2], "T": dims[3], "eps": eps, "kappa": kappa}
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the exact loops at one site of the smallest lattice: latency and launches
        _case("loops_point_4x4x4x4", "loops", (4, 4, 4, 4), 0.5, 0.12, source="point", noises=1, scheme=0, prec="f64",
              tol=1e-12, gammas=16),
        # a few noises on a small lattice, mixed precision: a first look at an ensemble
        _case("loops_f32_8x8x8x16", "loops", (8, 8, 8, 16), 0.30, 0.145, source="z2", noises=4, scheme=SPIN_COLOUR,
              prec="f32", tol=1e-10, gammas=2),
        # the plain estimate on the paper's lattice: 24 spin-colour-diluted noises, 288 solves
        _case("loops_f64_16x16x16x32", "loops", (16, 16, 16, 32), 0.35, 0.150, source="z2", noises=24,
              scheme=SPIN_COLOUR, prec="f64", tol=1e-10, gammas=2),
        # two diluted noises on the largest lattice, mixed precision
        _case("loops_f32_24x24x24x48", "loops", (24, 24, 24, 48), 0.35, 0.148, source="z2", noises=2,
              scheme=SPIN_COLOUR, prec="f32", tol=1e-10, gammas=2),
        # one operator application inside a caller's own solver
        _case("apply_m_f64_1rhs", "apply", (16, 16, 16, 32), 0.35, 0.150, op="m", prec="f64", nrhs=1),
        # the hopping term on a block of fields
        _case("apply_dhop_f64_96rhs", "apply", (16, 16, 16, 32), 0.35, 0.150, op="dhop", prec="f64", nrhs=96),
        # the Schur operator in single precision on a ragged lattice and an odd number of fields
        _case("apply_mhat_f32_ragged", "apply", (10, 6, 14, 18), 0.40, 0.150, op="mhat", prec="f32", nrhs=7),
        # a propagator: the 12 columns of given sources, mixed precision
        _case("solve_f32_12x12x12x24", "solve", (12, 12, 12, 24), 0.35, 0.148, prec="f32", tol=1e-10, nrhs=12),
        # the truncated solver method: 400 truncated solves in 16-bit storage and 16 corrections
        _case("tsm_f16_16x16x16x32", "tsm", (16, 16, 16, 32), 0.35, 0.150, lp="f16", iters=25, n_lp=400, n_hp=16,
              gammas=2),
        # forward and backward through the autograd function: loops, links' and kappa's gradients
        _case("grad_8x8x8x16", "grad", (8, 8, 8, 16), 0.35, 0.148, noises=2, scheme=SPIN_COLOUR, gammas=2),
        # three lattices in one batched call, graph replay on
        _case("batch_f32_3_lattices", "batch", (16, 16, 16, 32), 0.40, 0.150, noises=8, scheme=SPIN_COLOUR,
              prec="f32", tol=1e-10, graph=True, gammas=2),
        # smearing the columns of two propagators
        _case("smear_16x16x16x32", "smear", (16, 16, 16, 32), 0.35, 0.150, iters=10, nrhs=24),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _dims(rng, lo, hi):
    """Even extents of a lattice of about exp(uniform(log lo, log hi)) sites, time extent the longest or near it."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    base = (v / 2.0) ** 0.25
    ext = [max(4, 2 * int(round(base * rng.uniform(0.8, 1.25) / 2))) for _ in range(3)]
    t = max(4, 2 * int(round(v / (ext[0] * ext[1] * ext[2]) / 2)))
    return ext[0], ext[1], ext[2], min(t, 96)


def _rhs(rng, dims, most, cap):
    """A number of right-hand sides: at most `most`, and at most `cap` sites in all."""
    v = dims[0] * dims[1] * dims[2] * dims[3]
    return max(1, min(_log_int(rng, 1, most), cap // v))


def draw(rng):
    eps, kappa = rng.choice(FIELDS)
    kind = rng.choice(["apply", "apply", "solve", "loops", "loops", "loops", "tsm", "grad", "batch", "smear"])
    if kind == "apply":
        d = _dims(rng, 256, 300000)
        return _case("", kind, d, eps, kappa, op=rng.choice(sorted(OPS)), prec=rng.choice(["f64", "f64", "f32", "bf16"]),
                     nrhs=_rhs(rng, d, 200, 16_000_000))
    if kind == "solve":
        d = _dims(rng, 256, 300000)
        return _case("", kind, d, eps, kappa, prec=rng.choice(["f64", "f32"]), tol=rng.choice([1e-10, 1e-12]),
                     nrhs=_rhs(rng, d, 100, 8_000_000))
    if kind == "loops":
        d = _dims(rng, 256, 300000)
        if rng.random() < 0.2:
            return _case("", kind, d, eps, kappa, source="point", noises=1, scheme=0, prec=rng.choice(["f64", "f32"]),
                         tol=1e-10, gammas=16)
        scheme = rng.choice([0, SPIN, SPIN_COLOUR, SPIN_COLOUR, SPIN_COLOUR | EVEN_ODD])
        n = _rhs(rng, d, 32, 16_000_000 // _classes(scheme))
        return _case("", kind, d, eps, kappa, source="z2", noises=n, scheme=scheme, prec=rng.choice(["f64", "f32"]),
                     tol=rng.choice([1e-10, 1e-12]), gammas=rng.choice([1, 2, 16]))
    if kind == "tsm":
        d = _dims(rng, 256, 140000)
        n = max(16, _rhs(rng, d, 400, 40_000_000))
        # (float16 storage rounds differently in the two hopping kernels that the autotuner chooses from, so small
        # lattices, where either may win, are drawn in the formats whose results do not depend on the choice)
        return _case("", kind, d, eps, kappa, lp=rng.choice(["bf16", "f32"]), iters=rng.choice([10, 15, 25]),
                     n_lp=n, n_hp=max(2, n // 25), gammas=2)
    if kind == "grad":
        d = _dims(rng, 256, 40000)
        return _case("", kind, d, eps, kappa, noises=rng.choice([1, 2, 3]), scheme=rng.choice([0, SPIN, SPIN_COLOUR]), gammas=2)
    if kind == "batch":
        d = _dims(rng, 2000, 140000)
        return _case("", kind, d, eps, kappa, noises=_log_int(rng, 1, 8), scheme=rng.choice([0, SPIN_COLOUR]), prec="f32",
                     tol=1e-10, graph=rng.random() < 0.5, gammas=2)
    d = _dims(rng, 256, 300000)
    return _case("", kind, d, eps, kappa, iters=rng.choice([1, 5, 20, 50]), nrhs=_rhs(rng, d, 48, 8_000_000))


def _classes(scheme):
    return ((12 if scheme & SPIN_COLOUR else 1) * (4 if scheme & SPIN else 1) * (8 if scheme & CUBIC else 1)
            * (2 if scheme & EVEN_ODD else 1))


def _shape(case):
    return case["X"], case["Y"], case["Z"], case["T"]


def _batch_shapes(case):
    """The case's lattice and two smaller ones (about 3/4 and 1/2 of its extents)."""
    d = _shape(case)
    return [tuple(max(4, 2 * int(round(f * x / 2))) for x in d) for f in (0.5, 0.75, 1.0)]


def _gammas(case):
    return {1: [15], 2: [0, 15], 16: list(range(16))}[case["gammas"]]


# ------------------------------------------------------------------ inputs


def _mul3(a, b):
    """Products of 3x3 matrices, elementwise over the leading extents."""
    return (a[..., :, :, None] * b[..., None, :, :]).sum(-2)


def _gauge_links(dims, eps, seed):
    """SU(3) links exp(i eps H), H = sum_a h_a lambda_a with unit-normal h_a: complex128 [4][V][3][3] on the GPU."""
    V = dims[0] * dims[1] * dims[2] * dims[3]
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    h = torch.randn((4 * V, 8), generator=gen, dtype=torch.float64, device="cuda")
    H = torch.zeros((4 * V, 3, 3), dtype=torch.complex128, device="cuda")
    s3 = 1.0 / math.sqrt(3.0)
    H[:, 0, 0] = h[:, 2] + s3 * h[:, 7]
    H[:, 1, 1] = -h[:, 2] + s3 * h[:, 7]
    H[:, 2, 2] = -2.0 * s3 * h[:, 7]
    for (i, j), (re, im) in {(0, 1): (0, 1), (0, 2): (3, 4), (1, 2): (5, 6)}.items():
        H[:, i, j] = torch.complex(h[:, re], -h[:, im])
        H[:, j, i] = torch.complex(h[:, re], h[:, im])
    A = H * (1j * eps / 16.0)
    U = torch.eye(3, dtype=torch.complex128, device="cuda").expand(4 * V, 3, 3)
    for k in range(12, 0, -1):  # exp(A) by Horner's rule, then four squarings
        U = _mul3(A, U) / k + torch.eye(3, dtype=torch.complex128, device="cuda")
    for _ in range(4):
        U = _mul3(U, U)
    r0 = U[:, 0] / torch.linalg.vector_norm(U[:, 0], dim=-1, keepdim=True)
    r1 = U[:, 1] - (r0.conj() * U[:, 1]).sum(-1, keepdim=True) * r0
    r1 = r1 / torch.linalg.vector_norm(r1, dim=-1, keepdim=True)
    r2 = torch.stack([r0[:, 1] * r1[:, 2] - r0[:, 2] * r1[:, 1], r0[:, 2] * r1[:, 0] - r0[:, 0] * r1[:, 2],
                      r0[:, 0] * r1[:, 1] - r0[:, 1] * r1[:, 0]], dim=-1).conj()
    return torch.stack([r0, r1, r2], dim=-2).reshape(4, V, 3, 3).contiguous()


def _fields(dims, nrhs, seed):
    """Gaussian spinor fields, complex128 [nrhs][V][4][3] on the GPU."""
    V = dims[0] * dims[1] * dims[2] * dims[3]
    gen = torch.Generator(device="cuda").manual_seed(int(seed) + 77)
    return torch.randn((nrhs, V, 4, 3), generator=gen, dtype=torch.complex128, device="cuda")


def _noise_seed(seed, k=0):
    return 1_000_003 * int(seed) + 2000 + k


def _cotangent(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed) + 99)
    return torch.randn((case["noises"], len(_gammas(case)), case["T"]), generator=gen, dtype=torch.complex128, device="cuda")


def prepare(case, seed):
    kind, dims = case["kind"], _shape(case)
    state = {"case": case}
    if kind == "batch":
        state["gauges"] = [dl.Gauge(dl.Lattice(d), _gauge_links(d, case["eps"], seed + 10 * k), precs=(dl.DL_F64, dl.DL_F32))
                           for k, d in enumerate(_batch_shapes(case))]
        state["sources"] = [dl.z2_sources(_noise_seed(seed, k), case["noises"], scheme=case["scheme"]) for k in range(3)]
        state["params"] = dl.solve_params(prec=PREC[case["prec"]], tol=case["tol"], maxiter=2000, use_graph=case["graph"])
        return state
    links = _gauge_links(dims, case["eps"], seed)
    if kind == "grad":
        state["kappa"] = torch.tensor(case["kappa"], dtype=torch.float64, requires_grad=True)
        state["links"] = links.requires_grad_(True)
        state["sources"] = dl.z2_sources(_noise_seed(seed), case["noises"], scheme=case["scheme"])
        state["cotangent"] = _cotangent(case, seed)
        return state
    precs = {dl.DL_F64, PREC[case.get("prec") or case.get("lp") or "f64"]}
    if kind == "tsm":
        precs.add(dl.DL_F32)
    state["gauge"] = dl.Gauge(dl.Lattice(dims), links, precs=sorted(precs))
    if kind in ("apply", "solve", "smear"):
        state["fields"] = _fields(dims, case["nrhs"], seed)
    if kind == "solve":
        state["params"] = dl.solve_params(prec=PREC[case["prec"]], tol=case["tol"], maxiter=2000)
    if kind == "loops":
        state["sources"] = _sources(case, seed)
        state["params"] = dl.solve_params(prec=PREC[case["prec"]], tol=case["tol"], maxiter=2000)
    if kind == "tsm":
        state["sources"] = dl.z2_sources(_noise_seed(seed), case["n_lp"] + case["n_hp"])
        state["lp"] = dl.solve_params(solver=dl.DL_CGNR, prec=PREC[case["lp"]], fixed_iters=case["iters"])
        state["hp"] = dl.solve_params(prec=dl.DL_F32, tol=1e-10, maxiter=2000)
    return state


def _point_site(case, seed):
    return (int(seed) * 7919) % (case["X"] * case["Y"] * case["Z"] * case["T"])


def _sources(case, seed):
    if case["source"] == "point":
        return dl.point_sources(_point_site(case, seed))
    return dl.z2_sources(_noise_seed(seed), case["noises"], scheme=case["scheme"])


# ------------------------------------------------------------------ one pass


def run(state):
    case = state["case"]
    kind, kappa = case["kind"], case["kappa"]
    if kind == "apply":
        return dl.apply(state["gauge"], kappa, OPS[case["op"]], state["fields"], prec=PREC[case["prec"]])
    if kind == "solve":
        x, stats = dl.solve(state["gauge"], kappa, state["fields"], state["params"])
        return {"x": x, "status": np.array([s[0] for s in stats])}
    if kind == "smear":
        return dl.smear(state["gauge"], ALPHA, case["iters"], state["fields"])
    if kind == "loops":
        loops, stats = dl.loops(state["gauge"], kappa, state["sources"], _gammas(case), state["params"])
        return {"loops": loops, "status": np.array([s[0] for s in stats])}
    if kind == "tsm":
        lp, hp, hl, stats = dl.loops_tsm(state["gauge"], kappa, state["sources"], case["n_lp"], case["n_hp"], _gammas(case),
                                         state["lp"], state["hp"])
        est, var = dl.tsm_estimate(lp, hp, hl)
        return {"lp": lp, "hp": hp, "hl": hl, "est": est, "var": var, "status": np.array([s[0] for s in stats])}
    if kind == "batch":
        loops, stats = dl.batch_loops(state["gauges"], [kappa] * 3, state["sources"], _gammas(case), state["params"])
        return {"loops": loops, "status": [np.array([s[0] for s in st]) for st in stats]}
    loops = disconnected_loops(state["kappa"], state["links"], _shape(case), state["sources"], _gammas(case))
    gk, gl = torch.autograd.grad(loops, (state["kappa"], state["links"]), grad_outputs=state["cotangent"])
    return {"loops": loops, "grad_kappa": gk, "grad_links": gl}


# ------------------------------------------------------------------ bytes and operations

HOP_FLOPS = 1320  # of the hopping term at one site


def _iterations(tol):
    """BiCGStab iterations, about: the workloads gain a factor e in the residual per iteration."""
    return math.log(1.0 / tol)


def _solve_work(sites, nrhs, tol, prec):
    """A tolerance-driven solve: per iteration two applications of the Schur operator (a hop at every site each), and
    14 half fields moved: p and rhat read, v written; r and v read, t written; x, r, p, v, t read, x, r, p written."""
    it = _iterations(tol)
    return (nrhs * it * 14 * (sites // 2) * 12 * BYTES[prec] + 4 * sites * 6 * BYTES[prec], nrhs * it * 2 * sites * HOP_FLOPS)


def work(case):
    kind, dims = case["kind"], _shape(case)
    V = dims[0] * dims[1] * dims[2] * dims[3]
    if kind == "apply":  # the fields in and out, the links
        return {"bytes": case["nrhs"] * 2 * V * 12 * 16 + 4 * V * 6 * BYTES[case["prec"]], "flops": case["nrhs"] * V * HOP_FLOPS}
    if kind == "smear":  # the fields in and out and the spatial links; six colour products of four spins a site and step
        return {"bytes": case["nrhs"] * 2 * V * 12 * 16 + 3 * V * 6 * 16,
                "flops": case["iters"] * case["nrhs"] * V * (6 * 4 * 72 + 48)}
    if kind == "solve":
        b, f = _solve_work(V, case["nrhs"], case["tol"], case["prec"])
        return {"bytes": b + case["nrhs"] * 2 * V * 12 * 16, "flops": f}
    if kind == "loops":
        n = 12 if case["source"] == "point" else case["noises"] * _classes(case["scheme"])
        b, f = _solve_work(V, n, case["tol"], case["prec"])
        return {"bytes": b, "flops": f}
    if kind == "tsm":
        n = case["n_lp"] + case["n_hp"]
        b, f = _solve_work(V, case["n_hp"], 1e-10, "f32")
        # truncated CG on the normal equations: p read, t written; t and r read, r written; x, p, r read, x, p written
        b += n * case["iters"] * 10 * (V // 2) * 12 * BYTES[case["lp"]]
        return {"bytes": b, "flops": f + n * case["iters"] * 2 * V * HOP_FLOPS}
    if kind == "batch":
        n = case["noises"] * _classes(case["scheme"])
        parts = [_solve_work(d[0] * d[1] * d[2] * d[3], n, case["tol"], case["prec"]) for d in _batch_shapes(case)]
        return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}
    n = case["noises"] * _classes(case["scheme"])
    b, f = _solve_work(V, 4 * n, 1e-12, "f64")  # the loops, and the loops, adjoint and kappa solves of the gradient
    return {"bytes": b + 2 * 4 * V * 9 * 16, "flops": f}


# ------------------------------------------------------------------ plain torch in 64 bits

_SIGMA = [[[0, 1], [1, 0]], [[0, -1j], [1j, 0]], [[1, 0], [0, -1]]]


def _gamma_matrices():
    g = torch.zeros((4, 4, 4), dtype=torch.complex128)
    for k in range(3):
        for r in range(2):
            for c in range(2):
                g[k, r, 2 + c] = -1j * _SIGMA[k][r][c]
                g[k, 2 + r, c] = 1j * _SIGMA[k][r][c]
    for r in range(2):
        g[3, r, 2 + r] = g[3, 2 + r, r] = 1
    return g


def _gamma_product(n):
    g, out = _gamma_matrices(), torch.eye(4, dtype=torch.complex128)
    for mu in range(4):
        if (n >> mu) & 1:
            out = out @ g[mu]
    return out


def _spin(m, psi):
    """The 4x4 spin matrix m applied to [.., 4, 3], over its non-zero entries."""
    rows = []
    for a in range(4):
        acc = None
        for b in range(4):
            z = complex(m[a, b])
            if z != 0:
                t = z * psi[..., b, :]
                acc = t if acc is None else acc + t
        rows.append(torch.zeros_like(psi[..., 0, :]) if acc is None else acc)
    return torch.stack(rows, dim=-2)


def _colour(u, psi, dag):
    """U psi or U^+ psi for u [V][3][3], psi [n][V][4][3]."""
    out = []
    for i in range(3):
        out.append(sum((u[:, j, i].conj() if dag else u[:, i, j])[None, :, None] * psi[..., j] for j in range(3)))
    return torch.stack(out, dim=-1)


class _Lattice:
    """Site tables and the plain Wilson operator of one lattice (antiperiodic in time)."""

    def __init__(self, dims, links):
        self.dims, self.U = dims, links
        X, Y, Z, T = dims
        t, z, y, x = torch.meshgrid(*[torch.arange(n, device="cuda") for n in (T, Z, Y, X)], indexing="ij")
        self.x = [a.reshape(-1) for a in (x, y, z, t)]
        self.V = X * Y * Z * T
        self.par = (x + y + z + t).reshape(-1) & 1

        def index(c):
            return c[0] + X * (c[1] + Y * (c[2] + Z * c[3]))

        self.fwd, self.bwd, self.sf, self.sb = [], [], [], []
        for mu in range(4):
            up, dn = list(self.x), list(self.x)
            up[mu], dn[mu] = (self.x[mu] + 1) % dims[mu], (self.x[mu] - 1) % dims[mu]
            self.fwd.append(index(up))
            self.bwd.append(index(dn))
            one = torch.ones(self.V, dtype=torch.float64, device="cuda")
            self.sf.append(torch.where((self.x[mu] == dims[mu] - 1) & (mu == 3), -one, one)[None, :, None, None])
            self.sb.append(torch.where((self.x[mu] == 0) & (mu == 3), -one, one)[None, :, None, None])

    def dhop(self, psi, dag=False, U=None):
        U = self.U if U is None else U
        g, eye, out = _gamma_matrices(), torch.eye(4, dtype=torch.complex128), torch.zeros_like(psi)
        s = -1.0 if dag else 1.0
        for mu in range(4):
            out = out + self.sf[mu] * _spin(eye - s * g[mu], _colour(U[mu], psi[:, self.fwd[mu]], False))
            out = out + self.sb[mu] * _spin(eye + s * g[mu], _colour(U[mu][self.bwd[mu]], psi[:, self.bwd[mu]], True))
        return out

    def keep(self, psi, parity):
        return psi * (self.par == parity).to(torch.float64)[None, :, None, None]

    def m(self, psi, kappa, dag=False):
        return psi - kappa * self.dhop(psi, dag)

    def mhat(self, psi, kappa, dag=False):
        e = self.keep(psi, 0)
        return e - kappa * kappa * self.keep(self.dhop(self.keep(self.dhop(e, dag), 1), dag), 0)

    def solve(self, b, kappa):
        """M^-1 b: conjugate gradients on the normal equations of the Schur system, to rounding."""
        rhs = self.keep(b, 0) + kappa * self.keep(self.dhop(self.keep(b, 1)), 0)
        x = self.cgnr(rhs, kappa, 400, 1e-15)
        return x + self.keep(b, 1) + kappa * self.keep(self.dhop(x), 1)

    def cgnr(self, rhs, kappa, iters, tol=0.0):
        r = self.mhat(rhs, kappa, True)
        x, p, rr = torch.zeros_like(r), r.clone(), _norm2(r)
        first = rr.clone()
        for _ in range(iters):
            t = self.mhat(p, kappa)
            q = self.mhat(t, kappa, True)
            tt = _norm2(t)
            alpha = torch.where(tt > 0, rr / tt, torch.zeros_like(tt))
            x, r = x + alpha * p, r - alpha * q
            new = _norm2(r)
            p = r + torch.where(rr > 0, new / rr, torch.zeros_like(rr)) * p
            rr = new
            if tol and bool((rr <= tol * tol * first).all()):
                break
        return x

    def truncated(self, b, kappa, iters):
        x = self.cgnr(self.keep(b, 0) + kappa * self.keep(self.dhop(self.keep(b, 1)), 0), kappa, iters)
        return x + self.keep(b, 1) + kappa * self.keep(self.dhop(x), 1)

    def contract(self, eta, s, gammas):
        """sum_{x in t} eta^+ Gamma s per right-hand side: [n][n_gamma][T]."""
        n, T = eta.shape[0], self.dims[3]
        return torch.stack([(eta.conj() * _spin(_gamma_product(g), s)).reshape(n, T, -1).sum(-1) for g in gammas], dim=1)

    def z2(self, seed, noises, scheme):
        """The diluted complex Z2 sources of the noises, [len * classes][V][4][3]."""
        site = torch.arange(self.V, device="cuda", dtype=torch.int64)[:, None, None]
        sp = torch.arange(4, device="cuda", dtype=torch.int64)[None, :, None]
        co = torch.arange(3, device="cuda", dtype=torch.int64)[None, None, :]
        cls = torch.zeros((self.V, 4, 3), dtype=torch.int64, device="cuda")
        x = [a[:, None, None] for a in self.x]
        if scheme & SPIN_COLOUR:
            cls = cls * 12 + 3 * sp + co
        if scheme & SPIN:
            cls = cls * 4 + sp
        if scheme & CUBIC:
            cls = cls * 8 + (x[0] & 1) + 2 * (x[1] & 1) + 4 * (x[2] & 1)
        if scheme & EVEN_ODD:
            cls = cls * 2 + (self.par[:, None, None] & 1)
        out = []
        for n in noises:
            r = _splitmix64(seed, ((n * self.V + site) * 4 + sp) * 3 + co)
            a = math.sqrt(0.5)
            eta = torch.complex(a * (1.0 - 2.0 * (r & 1).double()), a * (1.0 - 2.0 * ((r >> 1) & 1).double()))
            out += [eta * (cls == d) for d in range(_classes(scheme))]
        return torch.stack(out)

    def point(self, site):
        b = torch.zeros((12, self.V, 4, 3), dtype=torch.complex128, device="cuda")
        for d in range(12):
            b[d, site, d // 3, d % 3] = 1
        return b


def _norm2(a):
    return torch.view_as_real(a).square().sum(dim=(1, 2, 3, 4))[:, None, None, None]


def _signed(v):
    v &= (1 << 64) - 1
    return v - (1 << 64) if v >> 63 else v


def _splitmix64(seed, n):
    """Output number n of the SplitMix64 stream, as 64-bit patterns in int64."""
    z = n * _signed(0x9E3779B97F4A7C15) + _signed(seed + 0x9E3779B97F4A7C15)
    z = (z ^ ((z >> 30) & ((1 << 34) - 1))) * _signed(0xBF58476D1CE4E5B9)
    z = (z ^ ((z >> 27) & ((1 << 37) - 1))) * _signed(0x94D049BB133111EB)
    return z ^ ((z >> 31) & ((1 << 33) - 1))


def _per_noise(z, noises):
    return z.reshape(noises, -1, *z.shape[1:]).sum(1)


def _exact_loops(lat, eta, kappa, gammas, noises):
    """In chunks of right-hand sides, summed over each noise's classes."""
    step = max(1, 3_000_000 // lat.V)
    parts = [lat.contract(e, lat.solve(e, kappa), gammas) for e in eta.split(step)]
    return _per_noise(torch.cat(parts), noises).cpu().numpy()


def exact(case, seed):
    kind, dims, kappa = case["kind"], _shape(case), case["kappa"]
    V = dims[0] * dims[1] * dims[2] * dims[3]
    most = 3_500_000  # site-solves that plain torch does in the time there is
    if kind == "batch":
        n = case["noises"] * _classes(case["scheme"])
        if 1.6 * n * V > most:
            return None
        out = []
        for k, d in enumerate(_batch_shapes(case)):
            lat = _Lattice(d, _gauge_links(d, case["eps"], seed + 10 * k))
            eta = lat.z2(_noise_seed(seed, k), range(case["noises"]), case["scheme"])
            out.append(_exact_loops(lat, eta, kappa, _gammas(case), case["noises"]))
        return {"loops": out, "status": [None] * 3}
    solves = {"solve": case.get("nrhs", 0), "loops": 12 if case.get("source") == "point" else case.get("noises", 0) * _classes(case.get("scheme", 0)),
              "tsm": case.get("n_lp", 0) / 2, "grad": 3 * case.get("noises", 0) * _classes(case.get("scheme", 0))}.get(kind, 0)
    if solves * V > most:
        return None
    lat = _Lattice(dims, _gauge_links(dims, case["eps"], seed))
    if kind == "apply":
        out = []
        for psi in _fields(dims, case["nrhs"], seed).split(max(1, 3_000_000 // V)):
            if case["op"] == "dhop":
                out.append(lat.dhop(psi))
            elif case["op"] == "mhat":
                out.append(lat.mhat(psi, kappa))
            else:
                out.append(lat.m(psi, kappa, case["op"] == "mdag"))
        return torch.cat(out)
    if kind == "smear":
        out = []
        for psi in _fields(dims, case["nrhs"], seed).split(max(1, 3_000_000 // V)):
            for _ in range(case["iters"]):
                hop = sum(_colour(lat.U[i], psi[:, lat.fwd[i]], False)
                          + _colour(lat.U[i][lat.bwd[i]], psi[:, lat.bwd[i]], True) for i in range(3))
                psi = (psi + ALPHA * hop) / (1.0 + 6.0 * ALPHA)
            out.append(psi)
        return torch.cat(out)
    if kind == "solve":
        b = _fields(dims, case["nrhs"], seed)
        return {"x": torch.cat([lat.solve(p, kappa) for p in b.split(max(1, 3_000_000 // V))]), "status": None}
    if kind == "loops":
        if case["source"] == "point":
            site = _point_site(case, seed)
            return {"loops": _exact_loops(lat, lat.point(site), kappa, _gammas(case), 1), "status": None}
        eta = lat.z2(_noise_seed(seed), range(case["noises"]), case["scheme"])
        return {"loops": _exact_loops(lat, eta, kappa, _gammas(case), case["noises"]), "status": None}
    if kind == "tsm":
        lp, hp, step = [], [], max(1, 3_000_000 // V)
        total = case["n_lp"] + case["n_hp"]
        for k in range(0, total, step):
            eta = lat.z2(_noise_seed(seed), range(k, min(total, k + step)), 0)
            lp.append(lat.contract(eta, lat.truncated(eta, kappa, case["iters"]), _gammas(case)))
        for k in range(case["n_lp"], total, step):
            eta = lat.z2(_noise_seed(seed), range(k, min(total, k + step)), 0)
            hp.append(lat.contract(eta, lat.solve(eta, kappa), _gammas(case)))
        lp, hp = torch.cat(lp), torch.cat(hp)
        a, c = lp[: case["n_lp"]], lp[case["n_lp"]:]
        est = a.mean(0) + (hp - c).mean(0)
        return {"lp": a.cpu().numpy(), "hp": hp.cpu().numpy(), "hl": c.cpu().numpy(), "est": est.cpu().numpy(),
                "var": (_variance(a) / len(a) + _variance(hp - c) / len(c)).cpu().numpy(), "status": None}
    # grad: dF = Re kappa a^+ dD s with s = M^-1 eta and a = M^-+ (sum_g W_g Gamma_g^+ P_t eta)
    eta = lat.z2(_noise_seed(seed), range(case["noises"]), case["scheme"])
    W = _cotangent(case, seed).repeat_interleave(_classes(case["scheme"]), dim=0)
    s = lat.solve(eta, kappa)
    loops = _per_noise(lat.contract(eta, s, _gammas(case)), case["noises"])
    src = sum(W[:, k, lat.x[3]][:, :, None, None] * _spin(_gamma_product(g).conj().T, eta) for k, g in enumerate(_gammas(case)))
    g5 = _gamma_product(15)
    a = _spin(g5, lat.solve(_spin(g5, src), kappa))
    links = lat.U.clone().requires_grad_(True)
    F = (a.conj() * lat.dhop(s, U=links)).sum().real
    (gl,) = torch.autograd.grad(F, links)
    return {"loops": loops, "grad_kappa": F.detach().cpu(), "grad_links": kappa * gl}


def _variance(z):
    return torch.view_as_real(z - z.mean(0)).square().sum(-1).sum(0) / (len(z) - 1)
