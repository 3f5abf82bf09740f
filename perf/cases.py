"""Performance cases: what a user of this library has it do, through its public entry points.

Lattice sizes and couplings are those of the tests and of bench.py (4^4, 16^3 x 32, 24^3 x 48,
48^3 x 96 with c_sw 1.0 .. 1.2), or generic ragged extents.  `exact` restates every path in
plain torch complex128.
"""
import math

import torch

from paper_2407_08092_amd import api
from paper_2407_08092_amd.autograd import dirac_schur

DEV = "cuda"
PREC = {"f64": api.DDQ_F64, "f32": api.DDQ_F32, "f16": api.DDQ_F16, "bf16": api.DDQ_BF16}
DTYPE = {"f64": torch.complex128, "f32": torch.complex64, "f16": torch.float16, "bf16": torch.bfloat16}
BYTES = {"f64": 16, "f32": 8, "f16": 4, "bf16": 4}  # of a stored complex number
OMEGA = 0.16  # about 0.8 / |lambda_max(D_S)| on these fields


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def _lattice_case(name, kind, dims, **more):
    lx, ly, lz, lt = dims
    case = {"kind": kind, "lx": lx, "ly": ly, "lz": lz, "lt": lt, "eps": 0.5, "c_sw": 1.0, "m0": -0.2}
    case.update(more)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # the smallest call: one FP64 operator application on the 4^4 lattice of the smoke test
        # (unit tests, coarse levels of a hierarchy); latency and launches
        _lattice_case("apply_f64_4x4x4x4", "apply", (4, 4, 4, 4), prec="f64", nrhs=1, dagger=False),
        # a ragged lattice, a few right-hand sides and the adjoint: an inner product or a
        # normal-equation step on a small test configuration
        _lattice_case("apply_dag_f32_x3_12x10x6x14", "apply", (12, 10, 6, 14), prec="f32", nrhs=3, dagger=True),
        # the FP64 residual of an iterative refinement on a production-shaped lattice
        _lattice_case("apply_f64_24x48", "apply", (24, 24, 24, 48), prec="f64", nrhs=1, dagger=False),
        # the benchmark's work: FP32 Richardson sweeps on the largest lattice
        _lattice_case("sweeps_f32_48x96", "sweeps", (48, 48, 48, 96), prec="f32", nrhs=1, link12=False, n=4, c_sw=1.2, m0=-0.25),
        # a 16-bit preconditioner's sweeps inside a mixed-precision solve
        _lattice_case("sweeps_f16_24x48", "sweeps", (24, 24, 24, 48), prec="f16", nrhs=1, link12=False, n=8),
        # forward and backward of the differentiable operator: gradients of the vector and of the
        # links (force of a molecular-dynamics step, learned preconditioners)
        _lattice_case("backward_16x32", "backward", (16, 16, 16, 32), eps=0.4, m0=-0.1),
        # a new gauge configuration: links packed, clover built and inverted, then the operator
        # applied in FP64 and FP32 (every step of a molecular-dynamics trajectory)
        _lattice_case("setup_16x32", "setup", (16, 16, 16, 32)),
        # a whole mixed-precision solve to 1e-10: FP64 refinement, FP32 operator, FP16 sweeps
        _lattice_case("gmres_mixed_16x32", "gmres", (16, 16, 16, 32), inner="f32", smoother="f16", sweeps=12, passes=1),
        # the odd-even smoother M_nu on full vectors (the fine-level smoother of the multigrid)
        _lattice_case("smoother_f32_24x48", "smoother", (24, 24, 24, 48), prec="f32", nrhs=1, n=3),
        # the Schwarz smoother SAP(1, 4) on 4^4 blocks with FP32 block solves
        _lattice_case("sap_f32_24x48", "sap", (24, 24, 24, 48), prec="f32", link12=False, n=1, m=4),
        # twelve right-hand sides (one propagator) in the interleaved layout
        _lattice_case("mrhs12_24x48", "mrhs", (24, 24, 24, 48), nrhs=12, n=0),
        # the coarse-grid operator of 48^3 x 96 with 4^4 aggregates on one propagator's vectors
        {"name": "coarse_nv24_x12_12x24", "kind": "coarse", "lx": 12, "ly": 12, "lz": 12, "lt": 24, "nv": 24, "nrhs": 12, "storage": "f32"},
    ]


def _draw_dims(rng, lo, hi, step=2):
    """Four extents (multiples of step) whose product is spread evenly over log [lo, hi]."""
    while True:
        side = math.exp(rng.uniform(math.log(lo), math.log(hi))) ** 0.25
        d = [max(step, step * round(side * math.exp(rng.uniform(-0.5, 0.5)) / step)) for _ in range(4)]
        if lo <= math.prod(d) <= hi:
            return tuple(d)


def draw(rng):
    kind = rng.choice(["apply", "apply", "sweeps", "sweeps", "backward", "setup", "gmres", "smoother", "sap", "mrhs", "mrhs", "coarse"])
    big, mid = 24 ** 3 * 48, 16 ** 3 * 32
    if kind == "apply":
        prec = rng.choice(["f64", "f64", "f32", "f32", "f16", "bf16"])
        dagger = prec in ("f64", "f32") and rng.random() < 0.5
        return _lattice_case(None, kind, _draw_dims(rng, 256, big), prec=prec, nrhs=rng.choice([1, 1, 1, 2, 3, 5]), dagger=dagger)
    if kind == "sweeps":
        prec = rng.choice(["f64", "f32", "f32", "f16", "bf16"])
        return _lattice_case(None, kind, _draw_dims(rng, 4096, 4 * big), prec=prec, nrhs=rng.choice([1, 1, 1, 2]),
                             link12=prec == "f32" and rng.random() < 0.5, n=rng.randint(1, 8))
    if kind == "backward":
        return _lattice_case(None, kind, _draw_dims(rng, 256, 2 * mid), eps=0.4, m0=-0.1)
    if kind == "setup":
        return _lattice_case(None, kind, _draw_dims(rng, 256, big))
    if kind == "gmres":
        inner, smoother = rng.choice([("f64", "f64"), ("f32", "f32"), ("f32", "f16")])
        return _lattice_case(None, kind, _draw_dims(rng, 256, mid), inner=inner, smoother=smoother, sweeps=rng.randint(2, 12), passes=rng.choice([1, 2]))
    if kind == "smoother":
        return _lattice_case(None, kind, _draw_dims(rng, 1024, big), prec=rng.choice(["f64", "f32"]), nrhs=rng.choice([1, 1, 2]), n=rng.randint(1, 8))
    if kind == "sap":
        prec = rng.choice(["f64", "f32", "f32"])
        return _lattice_case(None, kind, _draw_dims(rng, 4096, big, 4), prec=prec, link12=prec == "f32" and rng.random() < 0.5,
                             n=rng.randint(1, 2), m=rng.randint(1, 5))
    if kind == "mrhs":
        return _lattice_case(None, kind, _draw_dims(rng, 4096, big), nrhs=rng.randint(1, 16), n=rng.choice([0, 0, 1, 2, 4]))
    lx, ly, lz, lt = (rng.randint(3, 12) for _ in range(4))
    return {"kind": kind, "lx": lx, "ly": ly, "lz": lz, "lt": lt, "nv": rng.choice([8, 16, 20, 24, 28, 32]), "nrhs": rng.randint(1, 64),
            "storage": rng.choice(["f32", "f32", "f16", "bf16"])}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _dims(case):
    return case["lx"], case["ly"], case["lz"], case["lt"]


def _shape(case):
    return case["lt"], case["lz"], case["ly"], case["lx"]


def _normal(shape, gen, dtype=torch.complex128):
    """Complex numbers with Re and Im each N(0, 1)."""
    real = torch.float64 if dtype == torch.complex128 else torch.float32
    return torch.view_as_complex(torch.randn(tuple(shape) + (2,), generator=gen, dtype=real, device=DEV))


def _mul3(a, b):
    return (a.unsqueeze(-1) * b.unsqueeze(-3)).sum(-2)


def _links(case, gen, chunk=1 << 21):
    """U = exp(i eps sum_k a_k T_k) per link, a_k ~ N(0, 1), T_k the su(3) generators of
    tr(T_a T_b) = delta_ab / 2: scaled Taylor series and squarings."""
    n = math.prod(_dims(case)) * 4
    out = torch.empty((n, 3, 3), dtype=torch.complex128, device=DEV)
    r3 = 1 / math.sqrt(3)
    eye = torch.eye(3, dtype=torch.complex128, device=DEV)
    for s in range(0, n, chunk):
        m = min(chunk, n - s)
        a = torch.randn((8, m), generator=gen, dtype=torch.float64, device=DEV) * (0.5 * case["eps"] / 64)
        x = torch.zeros((m, 3, 3), dtype=torch.complex128, device=DEV)
        for i, j, re, im in ((0, 1, 0, 1), (0, 2, 3, 4), (1, 2, 5, 6)):  # i H: the off-diagonal generators
            x[:, i, j] = torch.complex(a[im], a[re])
            x[:, j, i] = torch.complex(-a[im], a[re])
        x[:, 0, 0].imag.copy_(a[2] + r3 * a[7])
        x[:, 1, 1].imag.copy_(-a[2] + r3 * a[7])
        x[:, 2, 2].imag.copy_(-2 * r3 * a[7])
        u = eye + x / 7
        for k in range(6, 0, -1):
            u = eye + _mul3(x, u) / k
        for _ in range(6):
            u = _mul3(u, u)
        out[s:s + m] = u
    return out.reshape(_shape(case) + (4, 3, 3))


def _layout(v, prec):
    """[..., 12, V/2] complex128 in the parity layout of prec, rounded to it."""
    lead, vh = v.shape[:-2], v.shape[-1]
    if prec == "f64":
        return v.contiguous()
    if prec == "f32":
        return v.reshape(lead + (6, 2, vh)).transpose(-1, -2).to(torch.complex64).contiguous()
    q = torch.view_as_real(v.reshape(lead + (3, 4, vh)).transpose(-1, -2).contiguous())
    return q.to(DTYPE[prec]).contiguous()


def _unlayout(v, prec):
    """The inverse of _layout, in complex128."""
    if prec == "f64":
        return v
    if prec == "f32":
        q = v.to(torch.complex128)
    else:
        q = torch.view_as_complex(v.to(torch.float64))
    q = q.transpose(-1, -2)
    return q.reshape(q.shape[:-3] + (12, q.shape[-1]))


def _keep(case):
    """The stored precisions and link form that a program of this case asks for."""
    kind, prec = case["kind"], case.get("prec", "f64")
    store = {"f64", prec}
    if kind in ("setup", "mrhs"):
        store |= {"f32"}
    if kind == "gmres":
        store |= {case["inner"], case["smoother"]}
    return tuple(PREC[p] for p in sorted(store)), bool(case.get("link12"))


def _inputs(case, seed):
    """Everything that is random in a case, from the seed alone."""
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    kind = case["kind"]
    vol = math.prod(_dims(case))
    if kind == "coarse":
        n2 = 2 * case["nv"]
        return {"blocks": _normal((vol, 9, n2, n2), gen, torch.complex64) / (6 * n2) ** 0.5,
                "v": _normal((vol, n2, case["nrhs"]), gen, torch.complex64)}
    d = {"U": _links(case, gen)}
    vh, many = vol // 2, case.get("nrhs", 1)
    parity = ((many,) if many > 1 else ()) + (12, vh)
    full = ((many,) if many > 1 else ()) + _shape(case) + (4, 3)
    if kind == "apply":
        d["x"] = _layout(_normal(parity, gen), case["prec"])
    elif kind == "sweeps":
        d["x"] = _layout(_normal(parity, gen), case["prec"])
        d["b"] = _layout(_normal(parity, gen), case["prec"])
    elif kind == "backward":
        d["phi"], d["g"] = _normal(parity, gen), _normal(parity, gen)
    elif kind == "setup":
        d["x"] = _normal(parity, gen)
    elif kind == "gmres":
        d["sol"] = _normal(full, gen)
    elif kind == "smoother":
        d["r"] = _normal(full, gen)
    elif kind == "sap":
        d["x"], d["b"] = _normal(full, gen), _normal(full, gen)
    elif kind == "mrhs":
        d["x"] = _normal((vh, 6, many, 2), gen, torch.complex64)
        d["b"] = _normal((vh, 6, many, 2), gen, torch.complex64)
    return d


def prepare(case, seed):
    d = _inputs(case, seed)
    state = {"case": case, **d}
    if case["kind"] == "coarse":
        state["op"] = api.CoarseOperator(_dims(case), d["blocks"], PREC[case["storage"]])
        del state["blocks"]
        return state
    lat = api.create_lattice(_dims(case))
    if case["kind"] != "setup":  # there the links are new on every pass
        store, link12 = _keep(case)
        api.set_gauge(lat, d["U"], store=store, link12=link12)
        api.set_clover(lat, case["c_sw"], case["m0"])
    state["lat"] = lat
    if case["kind"] == "gmres":
        state["b"] = _Plain(case, d["U"]).dirac(d["sol"])
        del state["sol"]
    if case["kind"] == "backward":
        state["phi"].requires_grad_(True)
        state["U"].requires_grad_(True)
    else:
        if case["kind"] != "setup":
            del state["U"]
    return state


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "coarse":
        return state["op"].apply(state["v"])
    lat = state["lat"]
    if kind == "apply":
        return api.apply_schur(lat, state["x"], dagger=case["dagger"])
    if kind == "sweeps":  # in place: a smoother goes on from where it was
        return api.richardson_smooth(lat, state["x"], state["b"], case["n"], OMEGA)
    if kind == "backward":
        y = dirac_schur(state["phi"], state["U"], lat)
        grads = torch.autograd.grad(y, (state["phi"], state["U"]), grad_outputs=state["g"])
        return {"y": y.detach(), "phi": grads[0], "U": grads[1]}
    if kind == "setup":
        store, link12 = _keep(case)
        api.set_gauge(lat, state["U"], store=store, link12=link12)
        api.set_clover(lat, case["c_sw"], case["m0"])
        x32 = api.convert_parity(lat, state["x"], torch.complex64)
        return {"y64": api.apply_schur(lat, state["x"]), "y32": api.apply_schur(lat, x32)}
    if kind == "gmres":
        x, _, _ = api.oe_gmres_solve(lat, state["b"], m=30, tol=1e-10, inner_prec=PREC[case["inner"]], smoother_sweeps=case["sweeps"],
                                     omega=OMEGA, smoother_prec=PREC[case["smoother"]], orth_passes=case["passes"])
        return x
    if kind == "smoother":
        return api.oe_smoother(lat, state["r"], case["n"], OMEGA, prec=PREC[case["prec"]])
    if kind == "sap":  # in place, as the sweeps
        return api.sap_smooth(lat, state["b"], state["x"], case["n"], case["m"], prec=PREC[case["prec"]])
    if case["n"] == 0:
        return api.mrhs_apply_schur(lat, state["x"])
    return api.mrhs_richardson_smooth(lat, state["x"], state["b"], case["n"], OMEGA)


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    """Bytes: links, clover blocks and vectors once per operator application (a sweep needs the
    whole vector of the one before).  Flops per pair of sites: 3672 per D_S, of which 1152 the
    two clover products."""
    kind = case["kind"]
    vol = math.prod(_dims(case))
    if kind == "coarse":
        n2 = 2 * case["nv"]
        store = 8 if case["storage"] == "f32" else 4
        return {"bytes": vol * (9 * n2 * n2 * store + 2 * n2 * case["nrhs"] * 8), "flops": 8 * vol * 9 * n2 * n2 * case["nrhs"]}
    vh, many = vol // 2, case.get("nrhs", 1)
    prec = case.get("prec", "f64")
    link = 48 if (case.get("link12") or prec in ("f16", "bf16")) else 72  # complex numbers per pair of sites
    fields = link + 72

    def schur(size, vectors, link=fields, k=1):
        return vh * size * (link + 12 * k * vectors)

    if kind == "apply":
        return {"bytes": schur(BYTES[prec], 2, k=many), "flops": 3672 * vh * many}
    if kind == "sweeps":
        return {"bytes": case["n"] * schur(BYTES[prec], 3, k=many), "flops": case["n"] * 3744 * vh * many}
    if kind == "mrhs":
        n = max(1, case["n"])
        return {"bytes": n * schur(8, 3 if case["n"] else 2, k=many), "flops": n * 3744 * vh * many}
    if kind == "backward":
        # y, the adjoint apply, kernel A twice for the force; 24 leaves of 4 products per link
        return {"bytes": 2 * schur(16, 2) + vol * 16 * (72 + 24 + 72), "flops": 3 * 3672 * vh + vol * 4 * 24 * 4 * 198}
    if kind == "setup":
        # canonical links read, packed (FP64 and FP32) and clover (three FP64 fields, two FP32)
        # written, two applications
        return {"bytes": vol * 16 * (36 + 72 + 36 + 54 + 18) + schur(16, 2) + schur(8, 2), "flops": vol * (24 * 4 * 198 + 2 * 1500) + 2 * 3672 * vh}
    if kind == "gmres":
        # about eight Krylov steps of one operator application and the sweeps
        lo = 4 if case["smoother"] in ("f16", "bf16") else BYTES[case["smoother"]]
        step = schur(BYTES[case["inner"]], 2, 144) + (case["sweeps"] - 1) * schur(lo, 3, 120 if lo == 4 else 144)
        return {"bytes": 8 * step, "flops": 8 * case["sweeps"] * 3672 * vh}
    if kind == "smoother":
        return {"bytes": case["n"] * schur(BYTES[prec], 3, k=many) + vh * 16 * (72 + 36 + 96 * many), "flops": (case["n"] + 1) * 3672 * vh * many}
    # sap: per sweep the FP64 residual's fields and vectors and the block solves' fields
    return {"bytes": case["n"] * vh * (16 * (144 + 6 * 12) + BYTES[prec] * (link // 2 + 72)), "flops": case["n"] * (case["m"] + 2) * 3672 * vh}


# ---------------------------------------------------------------------------
# the same in plain torch, 64 bits
# ---------------------------------------------------------------------------
class _Plain:
    """Wilson-clover D = A - H, A = (4 + m0) + (i c_sw / 4) sum sigma_munu F_munu, in the chiral
    basis, antiperiodic in t; fields shaped [t, z, y, x, ...]."""

    # gamma_mu = [[0, B], [B^H, 0]]: B of x, y, z, t
    B = (((0, -1j), (-1j, 0)), ((0, -1), (1, 0)), ((-1j, 0), (0, 1j)), ((1, 0), (0, 1)))
    SPIN = (((0, 1), (1, 0)), ((0, -1j), (1j, 0)), ((1, 0), (0, -1)))

    def __init__(self, case, U):
        self.U = [U[..., mu, :, :] for mu in range(4)]
        t, z, y, x = torch.meshgrid(*(torch.arange(n, device=DEV) for n in _shape(case)), indexing="ij")
        self.even = ((t + z + y + x) % 2 == 0).reshape(-1)
        self.shape = _shape(case)
        self.A = self._clover(case["c_sw"], case["m0"])

    @staticmethod
    def roll(f, mu, step, signed=False):
        """f(x + step mu); signed: with the antiperiodic sign of a hop across t."""
        g = torch.roll(f, -step, 3 - mu)
        if signed and mu == 3:
            sign = torch.ones(f.shape[0], dtype=torch.float64, device=f.device)
            sign[-1 if step > 0 else 0] = -1
            g = g * sign.reshape((-1,) + (1,) * (f.dim() - 1))
        return g

    def _field(self, mu, nu):
        a, b, r = self.U[mu], self.U[nu], self.roll
        m = _mul3
        am, bm = r(a, mu, -1), r(b, mu, -1)
        an, bn = r(a, nu, -1), r(b, nu, -1)
        amn, bmn = r(am, nu, -1), r(bm, nu, -1)
        q = m(m(m(a, r(b, mu, 1)), r(a, nu, 1).mH), b.mH)
        q = q + m(m(m(b, r(am, nu, 1).mH), bm.mH), am)
        q = q + m(m(m(am.mH, bmn.mH), amn), bn)
        q = q + m(m(m(bn.mH, an), r(bn, mu, 1)), a.mH)
        return (q - q.mH) / 8

    def _clover(self, c_sw, m0):
        """The two 6 x 6 blocks per site, [V, 2, 6, 6]."""
        fs = {}
        for mu in range(4):
            for nu in range(mu + 1, 4):
                fs[mu, nu] = self._field(mu, nu)
        electric = (fs[0, 3], fs[1, 3], fs[2, 3])
        magnetic = (fs[1, 2], -fs[0, 2], fs[0, 1])
        vol = math.prod(self.shape)
        blocks = []
        for sign in (1, -1):
            rows = [[0, 0], [0, 0]]
            for s, e, h in zip(self.SPIN, electric, magnetic):
                for i in range(2):
                    for j in range(2):
                        if s[i][j]:
                            rows[i][j] = rows[i][j] + (0.5j * c_sw * s[i][j]) * (sign * e - h)
            blk = torch.cat([torch.cat(r, -1) for r in rows], -2).reshape(vol, 6, 6)
            blocks.append(blk + (4 + m0) * torch.eye(6, dtype=torch.complex128, device=DEV))
        return torch.stack(blocks, 1)

    @staticmethod
    def site(A, v):
        """Two 6 x 6 blocks times [..., 4, 3] spinors."""
        w = v.reshape(v.shape[:-2] + (2, 1, 6))
        return (A * w).sum(-1).reshape(v.shape)

    def hop(self, v, dagger=False):
        """H v = 1/2 sum_mu (1 - g) U v(x + mu) + (1 + g) U^H(x - mu) v(x - mu); dagger: 1 -+ g exchanged."""
        sf = 1.0 if dagger else -1.0
        out = None
        for mu in range(4):
            b = torch.tensor(self.B[mu], dtype=torch.complex128, device=DEV)
            for sign, step in ((sf, 1), (-sf, -1)):
                if step > 0:
                    p = self.roll(v, mu, 1, True)
                    h = p[..., :2, :] + sign * _spin(b, p[..., 2:, :])
                    u = (self.U[mu].unsqueeze(-3) * h.unsqueeze(-2)).sum(-1)
                else:
                    h = v[..., :2, :] + sign * _spin(b, v[..., 2:, :])
                    u = (self.U[mu].mH.unsqueeze(-3) * h.unsqueeze(-2)).sum(-1)
                    u = self.roll(u, mu, -1, True)
                term = torch.cat((u, sign * _spin(b.mH, u)), -2)
                out = term if out is None else out + term
        return 0.5 * out

    def dirac(self, v):
        many = v.dim() == 7
        got = [self.site(self.A.reshape(self.shape + (2, 6, 6)), w) - self.hop(w) for w in (v if many else [v])]
        return torch.stack(got) if many else got[0]

    def split(self, v):
        """The parity halves [12, V/2] of a full vector."""
        w = v.reshape(-1, 12)
        return w[self.even].T, w[~self.even].T

    def join(self, e, o):
        w = torch.zeros((self.even.numel(), 12), dtype=torch.complex128, device=DEV)
        if e is not None:
            w = w.index_put((self.even.nonzero()[:, 0],), e.T)
        if o is not None:
            w = w.index_put(((~self.even).nonzero()[:, 0],), o.T)
        return w.reshape(self.shape + (4, 3))

    def block(self, odd, inverse=False):
        A = self.A[~self.even if odd else self.even]
        return torch.linalg.inv(A) if inverse else A

    def on_site(self, A, v):
        return self.site(A, v.T.reshape(-1, 4, 3)).reshape(-1, 12).T

    def H_to(self, odd, v, dagger=False):
        """H from one parity's vector to the other (odd: to the odd sites)."""
        full = self.join(v, None) if odd else self.join(None, v)
        return self.split(self.hop(full, dagger))[1 if odd else 0]

    def set_blocks(self):
        self.Ae, self.Ao_inv = self.block(False), self.block(True, True)
        return self

    def schur(self, v, dagger=False):
        u = self.on_site(self.Ao_inv, self.H_to(True, v, dagger))
        return self.on_site(self.Ae, v) - self.H_to(False, u, dagger)


def _spin(b, v):
    return (b.unsqueeze(-1) * v.unsqueeze(-3)).sum(-2)


def _each(f, *vs):
    """f on every right-hand side of [12, V/2] or [nrhs, 12, V/2] vectors."""
    if vs[0].dim() == 2:
        return f(*vs)
    return torch.stack([f(*v) for v in zip(*vs)])


def _layout64(v, prec):
    """_layout without the rounding."""
    lead, vh = v.shape[:-2], v.shape[-1]
    if prec == "f64":
        return v.contiguous()
    if prec == "f32":
        return v.reshape(lead + (6, 2, vh)).transpose(-1, -2).contiguous()
    return torch.view_as_real(v.reshape(lead + (3, 4, vh)).transpose(-1, -2).contiguous())


def _sap_blocks(case):
    """Colour of every site's 4^4 block, [t, z, y, x]."""
    t, z, y, x = torch.meshgrid(*(torch.arange(n, device=DEV) // 4 for n in _shape(case)), indexing="ij")
    return (t + z + y + x) % 2, t, z, y, x


def _sap(plain, case, x, b, n, m):
    """SAP(n, m): per colour r = b - D x, then on each 4^4 block of the colour the odd-even
    Minimal Residual on its Schur complement, hops that leave the block dropped."""
    colour, *coords = _sap_blocks(case)
    ids = coords[0]
    for c, size in zip(coords[1:], case_blocks(case)[1:]):
        ids = ids * size + c
    ids = ids.reshape(-1)
    shape = plain.shape
    # links of hops that stay inside a block
    inner = _Plain.__new__(_Plain)
    inner.shape, inner.even, inner.A = shape, plain.even, plain.A
    inner.U = []
    for mu in range(4):
        same = torch.ones(shape, dtype=torch.bool, device=DEV)
        for c in coords:
            same &= torch.roll(c, -1, 3 - mu) == c
        inner.U.append(plain.U[mu] * same[..., None, None])
    inner.set_blocks()
    ids_e = ids[plain.even]
    count = int(ids.max()) + 1

    def dot(a, v):  # per block, spread over its even sites
        s = (a.conj() * v).sum(0)
        tot = torch.zeros(count, dtype=torch.complex128, device=DEV)
        return tot.index_add(0, ids_e, s)[ids_e]

    x = x.clone()
    for _ in range(n):
        for col in (0, 1):
            mask = (colour == col)[..., None, None]
            re, ro = plain.split((b - plain.dirac(x)) * mask)
            r = re + inner.H_to(False, inner.on_site(inner.Ao_inv, ro))
            e = torch.zeros_like(r)
            for _ in range(m):
                q = inner.schur(r)
                den = dot(q, q).real
                alpha = torch.where(den > 0, dot(q, r) / den.clamp_min(1e-300), torch.zeros((), dtype=torch.complex128, device=DEV))
                e = e + alpha * r
                r = r - alpha * q
            eo = inner.on_site(inner.Ao_inv, ro + inner.H_to(True, e))
            x = x + plain.join(e, eo) * mask
    return x


def case_blocks(case):
    return tuple(n // 4 for n in _shape(case))


def _coarse_exact(case, d):
    cd = _dims(case)
    n2, nrhs = 2 * case["nv"], case["nrhs"]
    v = d["v"].to(torch.complex128).reshape(cd[3], cd[2], cd[1], cd[0], n2, nrhs)
    dtype = {"f32": None, "f16": torch.float16, "bf16": torch.bfloat16}[case["storage"]]
    y = torch.zeros((math.prod(cd), n2, nrhs), dtype=torch.complex128, device=DEV)
    for k in range(9):
        w = v if k == 0 else torch.roll(v, 1 if (k - 1) & 1 else -1, 3 - (k - 1) // 2)
        w = w.reshape(-1, n2, nrhs)
        for s in range(0, y.shape[0], 4096):
            a = d["blocks"][s:s + 4096, k]
            if dtype is not None:  # the stored blocks are rounded once
                a = torch.view_as_complex(torch.view_as_real(a).to(dtype).to(torch.float64))
            y[s:s + 4096] += torch.bmm(a.to(torch.complex128), w[s:s + 4096].contiguous())
    return y


def exact(case, seed):
    d = _inputs(case, seed)
    kind = case["kind"]
    if kind == "coarse":
        return _coarse_exact(case, d)
    if kind == "gmres":
        return d["sol"]
    if kind == "backward":
        U = d["U"].requires_grad_(True)
        phi = d["phi"].requires_grad_(True)
        y = _Plain(case, U).set_blocks().schur(phi)
        grads = torch.autograd.grad(y, (phi, U), grad_outputs=d["g"])
        return {"y": y.detach(), "phi": grads[0], "U": grads[1]}
    plain = _Plain(case, d["U"]).set_blocks()

    def sweeps(x, b, n):
        for _ in range(n):
            x = x + OMEGA * (b - plain.schur(x))
        return x

    if kind == "apply":
        y = _each(lambda v: plain.schur(v, case["dagger"]), _unlayout(d["x"], case["prec"]))
        return _layout64(y, case["prec"])
    if kind == "sweeps":
        x = _each(lambda v, b: sweeps(v, b, case["n"]), _unlayout(d["x"], case["prec"]), _unlayout(d["b"], case["prec"]))
        return _layout64(x, case["prec"])
    if kind == "setup":
        y32 = plain.schur(d["x"].to(torch.complex64).to(torch.complex128))
        return {"y64": plain.schur(d["x"]), "y32": _layout64(y32, "f32")}
    if kind == "mrhs":
        # [V/2, 6, nrhs, 2] <-> [nrhs, 12, V/2]
        def rows(v):
            return v.to(torch.complex128).permute(2, 1, 3, 0).reshape(v.shape[2], 12, v.shape[0])

        x, b = rows(d["x"]), rows(d["b"])
        y = _each(plain.schur, x) if case["n"] == 0 else _each(lambda v, w: sweeps(v, w, case["n"]), x, b)
        return y.reshape(y.shape[0], 6, 2, -1).permute(3, 1, 0, 2).contiguous()
    if kind == "smoother":
        def smooth(r):
            re, ro = plain.split(r)
            bt = re + plain.H_to(False, plain.on_site(plain.Ao_inv, ro))
            xe = sweeps(torch.zeros_like(bt), bt, case["n"])
            return plain.join(xe, plain.on_site(plain.Ao_inv, ro + plain.H_to(True, xe)))

        return smooth(d["r"]) if case["nrhs"] == 1 else torch.stack([smooth(r) for r in d["r"]])
    return _sap(plain, case, d["x"], d["b"], case["n"], case["m"])
