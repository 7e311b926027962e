"""The timed cases of the library: what a lattice program asks of it, through its
public entry points, from the smallest lattice to a full-size one.

A program holds one handle per lattice (`Lattice`), sets a gauge field and a
flavour on it, and then applies the Schur operator, its preconditioners and its
solvers to sources.  Each case is one such call on lattices of the shapes that
the workload recipes name (8 x 4^3, 32 x 16^3, 48 x 24^3, 64 x 32^3) or on
ragged ones; `draw` gives others between them.

`exact` evaluates the same quantities in complex128 from the definitions
(Sec. 2.1, 2.3 and 4.4 of arXiv:1908.11673) in plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1908_11673_amd as qxd

PREC = {"f64": qxd.F64, "f32": qxd.F32, "bf16": qxd.BF16}
SIZE = {"f64": 8, "f32": 4, "bf16": 2}
# the two quarks of the sample run
FLAVOURS = {
    "d": dict(qhat=-2, invqel=6.0, kappa=0.136377, su3csw=1.909520, u1csw=1.0),
    "u": dict(qhat=4, invqel=6.0, kappa=0.137312, su3csw=1.909520, u1csw=1.0),
}
CHANNELS = (24, 32, 32, 24)  # of the learned preconditioner
TAPS = 81


def _case(name, op, L, cstar=3, tanti=0, flavour="d", **more):
    return dict({"name": name, "op": op, "L0": L[0], "L1": L[1], "L2": L[2], "L3": L[3], "cstar": cstar,
                 "tanti": tanti, "flavour": flavour}, **more)


def listed():
    return [
        # the smallest lattice of the recipes: the operator is all launch and latency
        _case("dhat-f64-8x4", "dhat", (8, 4, 4, 4), cstar=1, prec="f64", dagger=0),
        # a lattice whose half volume is no multiple of a workgroup, antiperiodic time, the adjoint operator
        _case("dhatdag-f32-ragged", "dhat", (18, 10, 14, 12), cstar=2, tanti=1, flavour="u", prec="f32", dagger=1),
        # the operator at full size, the headline quantity
        _case("dhat-f64-64x32", "dhat", (64, 32, 32, 32), prec="f64", dagger=0),
        # a new gauge configuration (what every trajectory or measurement starts with), then the
        # first applications of its operator in both precisions a mixed solve needs
        _case("setup-64x32", "setup", (64, 32, 32, 32), flavour="u"),
        # the preconditioner of the fastest full-size solver: 2 cycles of 8 plain block steps
        _case("sap-plain-64x32", "sap", (64, 32, 32, 32), ncy=2, nmr=8, eo=0),
        # the paper's setting: 5 cycles of 5 even-odd preconditioned block steps (the solver's default block solver)
        _case("sap-eo-32x16", "sap", (32, 16, 16, 16), flavour="u", ncy=5, nmr=5, eo=1),
        # the learned preconditioner: one application at full size (encode), one training batch (backward)
        _case("nn-apply-64x32", "nn", (64, 32, 32, 32)),
        _case("nn-grad-32x16", "nngrad", (32, 16, 16, 16), pairs=4, loss=1),
        # the deflated preconditioner
        _case("dfl-apply-32x16", "dfl", (32, 16, 16, 16), ns=16, nit=3, nc=16, ncy=2, nmr=8, eo=0),
        # whole solves from a canonical source to a canonical solution: the smallest (latency of an
        # iteration), a mixed-precision one, and the shifted systems of a rational approximation
        _case("cg-f64-8x4", "cg", (8, 4, 4, 4), cstar=1, inner="f64", res=1e-11),
        _case("fgcr-f32-32x16", "fgcr", (32, 16, 16, 16), inner="f32", res=1e-11, ncy=0, nmr=0, eo=0),
        _case("mscg-32x16", "mscg", (32, 16, 16, 16), flavour="u", res=1e-11, shifts=4, mu0=0.01),
    ]


# the largest extended volume drawn for each kind of case
_VMAX = {"dhat": 1 << 22, "dw": 1 << 22, "setup": 1 << 22, "sap": 1 << 22, "nn": 1 << 22, "nngrad": 1 << 18,
         "dfl": 1 << 18, "cg": 1 << 16, "fgcr": 1 << 18, "mscg": 1 << 18}


def _extents(rng, op, cstar, vmax):
    """Physical extents whose extended volume is spread over its logarithm up to vmax."""
    blocks = op in ("sap", "dfl") or (op == "fgcr" and rng.random() < 0.3)
    step = 8 if blocks else 2
    lo = 8 ** 4 if blocks else 512
    want = math.exp(rng.uniform(math.log(2 * lo), math.log(vmax)))
    for _ in range(400):
        L = []
        for mu in range(4):
            c = (want / (2 if cstar else 1)) ** 0.25 * math.exp(rng.uniform(-0.5, 0.5)) * (1.6 if mu == 0 else 0.9)
            unit = step if mu != 1 or not blocks else (8 if cstar >= 2 or cstar == 0 else 4)
            L.append(max(unit, 4, int(round(c / unit)) * unit))
        v = L[0] * L[1] * L[2] * L[3] * (2 if cstar else 1)
        if want / 2 <= v <= min(vmax, 2 * want):
            return L, blocks
    return ([8, 8, 8, 8], True) if blocks else ([8, 4, 4, 4], False)


def draw(rng):
    op = rng.choice(["dhat", "dhat", "dw", "setup", "sap", "sap", "nn", "nngrad", "dfl", "cg", "fgcr", "fgcr", "mscg"])
    cstar = rng.choice([0, 1, 2, 3, 3, 3])
    L, blocks = _extents(rng, op, cstar, _VMAX[op])
    c = dict(op=op, L0=L[0], L1=L[1], L2=L[2], L3=L[3], cstar=cstar, tanti=rng.choice([0, 0, 1]),
             flavour=rng.choice(["d", "u"]))
    if op in ("dhat", "dw"):
        c["prec"] = rng.choice(["f64", "f64", "f32", "f32", "bf16"])
        if op == "dhat":
            c["dagger"] = rng.choice([0, 1])
    elif op == "sap":
        c["eo"] = rng.choice([0, 1])
        c["ncy"], c["nmr"] = rng.choice([(1, 4), (1, 8), (2, 4), (2, 5), (3, 4), (2, 7)])
    elif op == "nngrad":
        c["pairs"], c["loss"] = rng.choice([1, 2, 3]), rng.choice([0, 1, 1])
    elif op == "dfl":
        c.update(ns=rng.choice([4, 8, 12, 16, 20]), nit=rng.choice([1, 2, 3]), nc=rng.choice([4, 8, 12]),
                 ncy=rng.choice([1, 2]), nmr=rng.choice([4, 6, 8]), eo=rng.choice([0, 1]))
    elif op == "cg":
        c.update(inner=rng.choice(["f64", "f32", "bf16"]), res=1e-11)
    elif op == "fgcr":
        sap = blocks and rng.random() < 0.8
        c.update(inner=rng.choice(["f32", "f32", "bf16"] + ([] if sap else ["f64"])), res=1e-11,
                 ncy=rng.choice([1, 2, 3]) if sap else 0, nmr=rng.choice([4, 6, 8]) if sap else 0,
                 eo=rng.choice([0, 1]) if sap else 0)
    elif op == "mscg":
        c.update(shifts=rng.choice([1, 2, 3, 4]), mu0=rng.choice([0.01, 0.02, 0.05]), res=1e-11)
    return c


# ---------------------------------------------------------------------------
# inputs (made on the GPU from the seed alone)


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _crandn(g, *shape):
    """Gaussian complex numbers, real and imaginary parts of variance 1/2."""
    return torch.randn(*shape, dtype=torch.complex128, device="cuda", generator=g)


def _geometry(case):
    L = [case["L%d" % m] for m in range(4)]
    Le = [L[0], 2 * L[1] if case["cstar"] else L[1], L[2], L[3]]
    return L, Le, L[0] * L[1] * L[2] * L[3], Le[0] * Le[1] * Le[2] * Le[3]


def _gauge(g, vphys):
    """SU(3) links near unity (rows of 1 + an anti-Hermitian Gaussian matrix
    made orthonormal, the third the conjugate cross product) and Gaussian U(1)
    angles: [4][vphys][3][3] complex128, [4][vphys] float64."""
    m = _crandn(g, 4, vphys, 3, 3).mul_(0.2)
    m = m - m.transpose(-1, -2).conj()
    a = m[..., 0, :].clone()
    b = m[..., 1, :].clone()
    del m
    a[..., 0] += 1
    b[..., 1] += 1
    a = a / a.abs().square().sum(-1, keepdim=True).sqrt()
    b = b - (a.conj() * b).sum(-1, keepdim=True) * a
    b = b / b.abs().square().sum(-1, keepdim=True).sqrt()
    u = torch.stack([a, b, torch.linalg.cross(a, b).conj()], dim=-2).contiguous()
    return u, 0.3 * torch.randn(4, vphys, dtype=torch.float64, device="cuda", generator=g)


def _weights(seed):
    """He-scaled network weights with a small last layer, layers packed [81][cout][cin]."""
    rng = np.random.default_rng(int(seed))
    parts = []
    for k in range(3):
        ci, co = CHANNELS[k], CHANNELS[k + 1]
        parts.append(rng.standard_normal(TAPS * co * ci) * math.sqrt(2.0 / (TAPS * ci)) * (0.05 if k == 2 else 1.0))
    return np.concatenate(parts).astype(np.float32)


def _inputs(case, seed):
    """The arrays a case starts from: gauge field and sources."""
    L, Le, vphys, V = _geometry(case)
    g = _gen(seed)
    U, A = _gauge(g, vphys)
    op, half = case["op"], 12 * (V // 2)
    d = {"U": U, "A": A}
    if op == "dhat" or op == "dw":
        x = _crandn(g, (2 if op == "dw" else 1) * half)
        if case["prec"] == "f32":
            x = x.to(torch.complex64)
        elif case["prec"] == "bf16":
            x = torch.view_as_real(x).reshape(-1).to(torch.bfloat16)
        d["x"] = x
    elif op == "setup":
        d["x"] = _crandn(g, half)
        d["x32"] = d["x"].to(torch.complex64)
    elif op in ("sap", "nn"):
        d["x"] = _crandn(g, half).to(torch.complex64)
    elif op == "dfl":
        d["x"] = _crandn(g, half).to(torch.complex64)
        d["start"] = _crandn(g, case["ns"], 2 * half).to(torch.complex64)
    elif op == "nngrad":
        d["e"] = _crandn(g, case["pairs"], half).to(torch.complex64)
    elif op in ("cg", "fgcr"):
        d["b"] = _crandn(g, V, 4, 3)
    else:
        d["b"] = _crandn(g, half)
    if op in ("nn", "nngrad"):
        d["w"] = _weights(seed)
    return d


class _Owned:
    """Keeps a network or deflation handle beside its lattice and frees it with the state."""

    def __init__(self, handle, destroy):
        self.handle, self.destroy = handle, destroy

    def __del__(self):
        self.destroy(self.handle)


def prepare(case, seed):
    d = _inputs(case, seed)
    op, fl = case["op"], FLAVOURS[case["flavour"]]
    lat = qxd.Lattice([case["L%d" % m] for m in range(4)], case["cstar"], bool(case["tanti"]))
    lat.setup(d["U"], d["A"], fl)
    st = {"case": case, "lat": lat, "in": d}
    if op != "setup":
        del d["U"], d["A"]
    if op == "dhat":
        st["out"] = lat.field(PREC[case["prec"]], zero=False)
    elif op == "dw":
        st["out"] = lat.field(PREC[case["prec"]], full=True, zero=False)
    elif op == "setup":
        st["out"], st["out32"] = lat.field(qxd.F64, zero=False), lat.field(qxd.F32, zero=False)
    elif op == "sap":
        st["out"] = lat.field(qxd.F32, zero=False)
    elif op in ("nn", "nngrad"):
        net = st["net"] = _Owned(qxd.qxd_nn_create(lat.h), qxd.qxd_nn_destroy)
        qxd.qxd_nn_set_weights(net.handle, d["w"])
        qxd.qxd_nn_set_skip(net.handle, 2 * fl["kappa"])
        st["out"] = lat.field(qxd.F32, zero=False)
        if op == "nngrad":  # pairs as harvested: D_hat e = r
            d["r"] = torch.empty_like(d["e"])
            for k in range(case["pairs"]):
                qxd.qxd_dw_eo_schur(lat.h, qxd.F32, 0, d["r"][k], d["e"][k])
    elif op == "dfl":
        dfl = st["dfl"] = _Owned(qxd.qxd_dfl_create(lat.h, case["ns"]), qxd.qxd_dfl_destroy)
        qxd.qxd_dfl_generate(lat.h, dfl.handle, d.pop("start"), case["nit"], 4, 4)
        st["out"] = lat.field(qxd.F32, zero=False)
    elif op in ("cg", "fgcr"):
        st["x"] = lat.field(qxd.F64, full=True, zero=False)
        st["params"] = qxd.solver_params(res=case["res"], inner_prec=PREC[case["inner"]], sap_ncy=case.get("ncy", 0),
                                         sap_nmr=case.get("nmr", 0), sap_plain=1 - case.get("eo", 0))
    else:
        st["shifts"] = _shifts(case)
        st["xs"] = [lat.field(qxd.F64, zero=False) for _ in st["shifts"]]
        st["params"] = qxd.solver_params(res=case["res"])
    return st


def _shifts(case):
    return [(case["mu0"] * 3.0 ** j) ** 2 for j in range(case["shifts"])]


def run(st):
    case, lat, d = st["case"], st["lat"], st["in"]
    op = case["op"]
    if op == "dhat":
        qxd.qxd_dw_eo_schur(lat.h, PREC[case["prec"]], case["dagger"], st["out"], d["x"])
        return st["out"]
    if op == "dw":
        qxd.qxd_dw_apply(lat.h, PREC[case["prec"]], st["out"], d["x"])
        return st["out"]
    if op == "setup":
        lat.setup(d["U"], d["A"], FLAVOURS[case["flavour"]])
        qxd.qxd_dw_eo_schur(lat.h, qxd.F64, 0, st["out"], d["x"])
        qxd.qxd_dw_eo_schur(lat.h, qxd.F32, 0, st["out32"], d["x32"])
        return st["out"], st["out32"]
    if op == "sap":
        qxd.qxd_sap_apply(lat.h, case["ncy"], case["nmr"], case["eo"], st["out"], d["x"])
        return st["out"]
    if op == "nn":
        qxd.qxd_nn_apply(lat.h, st["net"].handle, st["out"], d["x"])
        return st["out"]
    if op == "nngrad":
        return qxd.qxd_nn_loss_grad(lat.h, st["net"].handle, d["r"], d["e"], case["pairs"], case["loss"])
    if op == "dfl":
        qxd.qxd_dfl_apply(lat.h, st["dfl"].handle, case["nc"], case["ncy"], case["nmr"], case["eo"], st["out"], d["x"])
        return st["out"]
    if op == "cg":
        qxd.qxd_solve_cg(lat.h, st["params"], st["x"], lat.pack(d["b"]))
        return lat.unpack(st["x"])
    if op == "fgcr":
        qxd.qxd_solve_fgcr(lat.h, st["params"], None, st["x"], lat.pack(d["b"]))
        return lat.unpack(st["x"])
    qxd.qxd_solve_mscg(lat.h, st["params"], st["shifts"], st["xs"], d["b"])
    return st["xs"]


def work(case):
    """Inputs read once, outputs written once, and the arithmetic of the
    definitions: per site a hop sum is 1320 flops, a clover block pair 600."""
    L, Le, vphys, V = _geometry(case)
    Ve, op = V // 2, case["op"]
    schur = 2 * 1320 + 2 * 600 + 48  # flops per even site of one D_hat
    if op == "dhat":  # psi_e, out, links, H_e, H_o^-1
        return {"bytes": Ve * ((48 + 144) * SIZE[case["prec"]] + 144 * max(4, SIZE[case["prec"]])), "flops": Ve * schur}
    if op == "dw":
        return {"bytes": V * ((48 + 72) * SIZE[case["prec"]] + 72 * max(4, SIZE[case["prec"]])), "flops": V * 1970}
    if op == "setup":  # gauge field in; links, H, H_o^-1 in FP64 and what FP32 D_hat reads; then both applications
        bytes_ = vphys * 4 * (144 + 8) + V * (72 + 72 + 36) * 8 + Ve * 288 * 4 + Ve * 336 * 12
        return {"bytes": bytes_, "flops": V * 21000 + Ve * 4000 + 2 * Ve * schur}
    if op == "sap":
        return {"bytes": V * 4 * (72 + 72 + (18 if case["eo"] else 0)) + Ve * 192,
                "flops": V * case["ncy"] * (case["nmr"] + 1 + case["eo"]) * 1970}
    conv = (V * 41 * 24 * 32 + V * TAPS * 32 * 32 + Ve * TAPS * 32 * 24) * 2
    if op == "nn":
        return {"bytes": Ve * 192 + 207360 * 4, "flops": conv}
    if op == "nngrad":
        return {"bytes": case["pairs"] * Ve * 192 + 207360 * 8 + V * 4 * 144, "flops": 3 * case["pairs"] * conv}
    if op == "dfl":  # the basis twice, the little operator, the operator, source and result
        nblk, ns = V // 256, case["ns"]
        return {"bytes": 2 * V * 96 * ns + nblk * 72 * ns * ns + V * 4 * 144 + Ve * 192,
                "flops": V * 8 * 24 * ns + case["nc"] * nblk * 72 * ns * ns + V * 1970 * (1 + case["ncy"] * (case["nmr"] + 1))}
    # solves: source, solution and the operator once; the arithmetic of about 100 (FGCR), 300 (CG) operator applications
    n = {"cg": 300, "fgcr": 100, "mscg": 500}[op]
    return {"bytes": Ve * (192 * 4 + 288 * 8), "flops": n * Ve * schur}


# ---------------------------------------------------------------------------
# the same quantities in complex128 from their definitions

_S = [torch.tensor(m, dtype=torch.complex128) for m in ([[0, 1], [1, 0]], [[0, -1j], [1j, 0]], [[1, 0], [0, -1]])]


def _gammas():
    z = torch.zeros(2, 2, dtype=torch.complex128)
    one = torch.eye(2, dtype=torch.complex128)
    g = [torch.cat([torch.cat([z, -one], 1), torch.cat([-one, z], 1)], 0)]
    for s in _S:
        g.append(torch.cat([torch.cat([z, -1j * s], 1), torch.cat([1j * s, z], 1)], 0))
    return g


def _mm(a, b):
    return (a.unsqueeze(-1) * b.unsqueeze(-3)).sum(-2)


def _dag(a):
    return a.transpose(-1, -2).conj()


class _Exact:
    """The operator on the extended lattice; fields are [..., X0, X1, X2, X3, 4, 3]."""

    def __init__(self, case, U, A):
        self.L, self.Le, vphys, self.V = _geometry(case)
        self.cstar, self.tanti = case["cstar"], case["tanti"]
        f = FLAVOURS[case["flavour"]]
        U = U.reshape(4, *self.L, 3, 3)
        A = A.reshape(4, *self.L)
        if self.cstar:
            U = torch.cat([U, U.conj()], 2)
            A = torch.cat([A, -A], 2)
        self.gam = [g.cuda() for g in _gammas()]
        one = torch.eye(4, dtype=torch.complex128, device="cuda")
        self.pm = [(one - g, one + g) for g in self.gam]
        # one 6 x 6 block of the site-diagonal term for each chirality
        self.H = torch.zeros(*self.Le, 2, 6, 6, dtype=torch.complex128, device="cuda")
        self.H[..., :, :, :] += torch.eye(6, dtype=torch.complex128, device="cuda") / (2 * f["kappa"])
        for mu in range(4):
            for nu in range(mu + 1, 4):
                E = f["su3csw"] * self._field_strength(U, mu, nu)
                a = f["u1csw"] * f["qhat"] * self._abelian(A, mu, nu)
                E = E + 1j * a[..., None, None] * torch.eye(3, dtype=torch.complex128, device="cuda")
                sig = 0.5j * (self.gam[mu] @ self.gam[nu] - self.gam[nu] @ self.gam[mu])
                for c in (0, 1):
                    s = 0.5j * sig[2 * c:2 * c + 2, 2 * c:2 * c + 2]
                    k = s[:, None, :, None] * E[..., None, :, None, :]
                    self.H[..., c, :, :] += k.reshape(*self.Le, 6, 6)
                del E
        self.W = [U[m] * torch.exp(1j * f["qhat"] * A[m])[..., None, None] for m in range(4)]
        self.Wb = [_dag(self.shift(self.W[m], m, -1, 2)) for m in range(4)]
        x = torch.meshgrid(*[torch.arange(n, device="cuda") for n in self.Le], indexing="ij")
        self.par = (x[0] + x[1] + x[2] + x[3]) & 1
        self.even = (self.par == 0)[..., None, None].to(torch.float64)
        self.x = x
        self._inv = None

    def shift(self, f, mu, d, tail):
        """f(x + d mu); `tail` trailing dimensions follow the four of the lattice."""
        dims = [f.dim() - tail - 4 + m for m in range(4)]
        r = torch.roll(f, -d, dims[mu])
        if mu >= 2 and self.cstar >= mu:  # the wrapped slice comes from the mirror half
            i = self.Le[mu] - 1 if d > 0 else 0
            s = r.narrow(dims[mu], i, 1)
            s.copy_(torch.roll(s, self.L[1], dims[1]))
        return r

    def _field_strength(self, U, mu, nu):
        S = lambda f, m, d: self.shift(f, m, d, 2)  # noqa: E731
        um, un = U[mu], U[nu]
        um_n, un_m = S(um, nu, 1), S(un, mu, 1)
        plaq = _mm(_mm(um, un_m), _mm(_dag(um_n), _dag(un)))  # corner x
        Q = plaq
        # corner x - mu, seen from x: U_nu(x) U_mu(x-mu+nu)^+ U_nu(x-mu)^+ U_mu(x-mu)
        t = S(_mm(_mm(_dag(um_n), _dag(un)), um), mu, -1)
        Q = Q + _mm(un, t)
        # corner x - nu: U_nu(x-nu)^+ U_mu(x-nu) U_nu(x-nu+mu) U_mu(x)^+
        t = S(_mm(_mm(_dag(un), um), un_m), nu, -1)
        Q = Q + _mm(t, _dag(um))
        # corner x - mu - nu: U_mu(x-mu)^+ U_nu(x-mu-nu)^+ U_mu(x-mu-nu) U_nu(x-nu)
        t = S(_mm(_dag(un), um), nu, -1)  # at x - nu, still to be moved to x - mu
        t = S(_mm(_dag(um), t), mu, -1)
        Q = Q + _mm(t, S(un, nu, -1))
        return (Q - _dag(Q)) / 8

    def _abelian(self, A, mu, nu):
        S = lambda f, m, d: self.shift(f, m, d, 0)  # noqa: E731
        s = torch.sin(A[mu] + S(A[nu], mu, 1) - S(A[mu], nu, 1) - A[nu])
        s = s + S(s, mu, -1)
        return 0.25 * (s + S(s, nu, -1))

    def clover(self, f, H=None):
        H = self.H if H is None else H
        v = f.reshape(*f.shape[:-2], 2, 1, 6)
        return (H * v).sum(-1).reshape(f.shape)

    @property
    def Hinv(self):
        if self._inv is None:  # Gauss-Jordan; the blocks are dominated by their diagonal
            M = self.H.clone()
            R = torch.eye(6, dtype=torch.complex128, device="cuda").expand_as(M).clone()
            for k in range(6):
                p = 1 / M[..., k, k]
                M[..., k, :] *= p[..., None]
                R[..., k, :] *= p[..., None]
                for i in range(6):
                    if i != k:
                        q = M[..., i, k].clone()[..., None]
                        M[..., i, :] -= q * M[..., k, :]
                        R[..., i, :] -= q * R[..., k, :]
            self._inv = R
        return self._inv

    def hop(self, f, inside=False):
        """inside: hops that stay in their 4^4 block only."""
        out = torch.zeros_like(f)
        for mu in range(4):
            for d, W in ((1, self.W[mu]), (-1, self.Wb[mu])):
                s = self.shift(f, mu, d, 2)
                if mu == 0 and self.tanti:
                    s.narrow(s.dim() - 6, self.Le[0] - 1 if d > 0 else 0, 1).neg_()
                s = (W.unsqueeze(-3) * s.unsqueeze(-2)).sum(-1)
                if inside:
                    s = s * ((self.x[mu] & 3) != (3 if d > 0 else 0))[..., None, None]
                p = self.pm[mu][0 if d > 0 else 1]
                out += (p[:, :, None] * s.unsqueeze(-3)).sum(-2)
        return out

    def dirac(self, f):
        return self.clover(f) - 0.5 * self.hop(f)

    def schur(self, f, dagger=False):
        """D_hat on fields that vanish on the odd sites."""
        if dagger:
            return self.g5(self.schur(self.g5(f)))
        t = self.clover(self.hop(f), self.Hinv) * (1 - self.even)
        return (self.clover(f) - 0.25 * self.hop(t)) * self.even

    def g5(self, f):
        return torch.cat([f[..., :2, :], -f[..., 2:, :]], -2)

    def normal_cg(self, b, shift=0.0, tol=1e-14, nmx=2500):
        """(D_hat^+ D_hat + shift) x = b."""
        x, r = torch.zeros_like(b), b.clone()
        p, rr = r.clone(), float(r.abs().square().sum())
        stop = tol * tol * rr
        for _ in range(nmx):
            t = self.schur(p)
            w = self.schur(t, True)
            den = float(t.abs().square().sum()) + shift * float(p.abs().square().sum())
            a = rr / den
            x += a * p
            r -= a * (w + shift * p)
            new = float(r.abs().square().sum())
            if new <= stop:
                break
            p = r + (new / rr) * p
            rr = new
        return x

    def solve(self, b):
        bo = b * (1 - self.even)
        bh = (b + 0.5 * self.hop(self.clover(bo, self.Hinv))) * self.even
        xe = torch.zeros_like(b)
        for _ in range(2):  # the second pass takes out the rounding of the first
            xe = xe + self.normal_cg(self.schur(bh - self.schur(xe), True), tol=1e-13)
        return xe + self.clover(bo + 0.5 * self.hop(xe) * (1 - self.even), self.Hinv) * (1 - self.even)

    # -- the Schwarz preconditioner on 4^4 blocks

    def _blocks(self, f):
        """[..., nblk, sites of a block, 12]"""
        n = [e // 4 for e in self.Le]
        lead = f.shape[:-6]
        f = f.reshape(*lead, n[0], 4, n[1], 4, n[2], 4, n[3], 4, 12)
        k = len(lead)
        f = f.permute(*range(k), *[k + i for i in (0, 2, 4, 6, 1, 3, 5, 7, 8)])
        return f.reshape(*lead, n[0] * n[1] * n[2] * n[3], 256, 12)

    def _unblocks(self, f):
        n = [e // 4 for e in self.Le]
        lead = f.shape[:-3]
        k = len(lead)
        f = f.reshape(*lead, *n, 4, 4, 4, 4, 12)
        f = f.permute(*range(k), *[k + i for i in (0, 4, 1, 5, 2, 6, 3, 7, 8)])
        return f.reshape(*lead, *self.Le, 4, 3)

    def _minres(self, op, rho, nmr):
        e = torch.zeros_like(rho)
        for _ in range(nmr):
            v = op(rho)
            num = self._blocks(v.conj() * rho).sum((-1, -2))
            den = self._blocks(v.abs().square().to(v.dtype)).sum((-1, -2)).real
            al = torch.where(den > 0, num / torch.where(den > 0, den, 1.0), 0.0)
            al = self._unblocks(al[..., None, None].expand(*al.shape, 256, 12))
            e = e + al * rho
            rho = rho - al * v
        return e

    def sap(self, eta, ncy, nmr, eo):
        colour = ((self.x[0] >> 2) + (self.x[1] >> 2) + (self.x[2] >> 2) + (self.x[3] >> 2)) & 1
        odd = 1 - self.even
        x = torch.zeros_like(eta)
        hop = lambda f: self.hop(f, inside=True)  # noqa: E731
        for _ in range(ncy):
            for c in (0, 1):
                r = (eta - self.dirac(x)) * (colour == c)[..., None, None]
                if not eo:
                    e = self._minres(lambda f: self.clover(f) - 0.5 * hop(f), r, nmr)
                else:
                    def dhat(f):
                        return (self.clover(f) - 0.25 * hop(self.clover(hop(f), self.Hinv) * odd)) * self.even
                    ro = r * odd
                    rho = (r + 0.5 * hop(self.clover(ro, self.Hinv))) * self.even
                    e = self._minres(dhat, rho, nmr)
                    e = e + self.clover(ro + 0.5 * hop(e) * odd, self.Hinv) * odd
                x = x + e
        return x

    def deflated(self, eta, start, case):
        vs = start
        for _ in range(case["nit"]):
            vs = self.sap(vs, 4, 4, 0)
            vs = vs / vs.abs().square().sum(tuple(range(1, vs.dim())), keepdim=True).sqrt()
        vs = self._blocks(vs).flatten(-2)  # [ns, nblk, 3072]
        W = []
        for v in vs:
            for _ in range(2):
                for w in W:
                    v = v - (w.conj() * v).sum(-1, keepdim=True) * w
            W.append(v / v.abs().square().sum(-1, keepdim=True).sqrt())
        W = torch.stack(W)
        restrict = lambda f: (W.conj() * self._blocks(f).flatten(-2)).sum(-1)  # noqa: E731
        prolong = lambda c: self._unblocks((c[..., None] * W).sum(0).unflatten(-1, (256, 12)))  # noqa: E731
        r = restrict(eta)
        c = torch.zeros_like(r)
        zs, ws = [], []
        for _ in range(case["nc"]):
            z = r.clone()
            w = restrict(self.dirac(prolong(z)))
            be = [(wj.conj() * w).sum() for wj in ws]
            for b, wj, zj in zip(be, ws, zs):
                w, z = w - b * wj, z - b * zj
            n = w.abs().square().sum().sqrt()
            w, z = w / n, z / n
            a = (w.conj() * r).sum()
            c, r = c + a * z, r - a * w
            zs.append(z)
            ws.append(w)
        psi = prolong(c)
        return psi + self.sap(eta - self.dirac(psi), case["ncy"], case["nmr"], case["eo"])

    # -- layouts of the half and full fields

    def unpack(self, v, group, parities=1):
        """eo layout ([12 / group][Ve][group] per parity) -> field; missing parities are zero."""
        out = torch.zeros(self.V, 12, dtype=torch.complex128, device="cuda")
        v = v.reshape(parities, 12 // group, self.V // 2, group)
        for p in range(parities):
            out[(self.par == p).reshape(-1)] = v[p].permute(1, 0, 2).reshape(self.V // 2, 12).to(torch.complex128)
        return out.reshape(*self.Le, 4, 3)

    def pack(self, f, group, parities=1):
        f = f.reshape(self.V, 12)
        out = [f[(self.par == p).reshape(-1)].reshape(self.V // 2, 12 // group, group).permute(1, 0, 2).reshape(-1)
               for p in range(parities)]
        return torch.cat(out)

    # -- the learned preconditioner

    def _conv(self, h, W):
        out = torch.zeros(*h.shape[:-1], W.shape[1], dtype=h.dtype, device=h.device)
        for tap in range(TAPS):
            s = h
            for mu, d in enumerate((tap // 27 - 1, tap // 9 % 3 - 1, tap // 3 % 3 - 1, tap % 3 - 1)):
                if d:
                    s = self.shift(s, mu, d, 1)
            out = out + s @ W[tap].T
        return out

    def network(self, f, W, skip):
        """N(f) + skip f on the even sites for a field that vanishes on the odd ones."""
        h = torch.view_as_real(f.reshape(*self.Le, 12)).reshape(*self.Le, 24)
        for k in range(3):
            h = self._conv(h, W[k])
            if k < 2:
                h = torch.relu(h)
        y = torch.view_as_complex(h.reshape(*self.Le, 12, 2)).reshape(*self.Le, 4, 3)
        return (y + skip * f) * self.even


def _layers(w):
    out, at = [], 0
    for k in range(3):
        n = TAPS * CHANNELS[k] * CHANNELS[k + 1]
        out.append(torch.from_numpy(w[at:at + n]).cuda().double().reshape(TAPS, CHANNELS[k + 1], CHANNELS[k]))
        at += n
    return out


_GROUP = {"f64": 1, "f32": 2, "bf16": 4}


def exact(case, seed):
    d = _inputs(case, seed)
    op = case["op"]
    X = _Exact(case, d["U"], d["A"])
    del d["U"], d["A"]
    if op in ("dhat", "dw"):
        x, n = d["x"], _GROUP[case["prec"]]
        if case["prec"] == "bf16":
            x = torch.view_as_complex(x.double().reshape(-1, 2))
        parts = 2 if op == "dw" else 1
        f = X.unpack(x, n, parts)
        f = X.dirac(f) if op == "dw" else X.schur(f, bool(case["dagger"]))
        return X.pack(f, n, parts)
    if op == "setup":
        return X.pack(X.schur(X.unpack(d["x"], 1)), 1), X.pack(X.schur(X.unpack(d["x32"], 2)), 2)
    if op == "sap":
        return X.pack(X.sap(X.unpack(d["x"], 2), case["ncy"], case["nmr"], case["eo"]), 2)
    skip = 2 * FLAVOURS[case["flavour"]]["kappa"]
    if op == "nn":
        f = X.unpack(d["x"], 2)
        n = f.abs().square().sum().sqrt()
        return X.pack(n * X.network(f / n, _layers(d["w"]), skip), 2)
    if op == "nngrad":
        W = [w.requires_grad_() for w in _layers(d["w"])]
        total = 0.0
        for k in range(case["pairs"]):
            e = X.unpack(d["e"][k], 2)
            r = X.schur(e)
            n = r.abs().square().sum().sqrt()
            with torch.no_grad():
                rhat, ehat = r / n, e / n
            u = X.network(rhat, W, skip) - ehat
            if case["loss"] == 0:
                loss = u.abs().square().sum() / ehat.abs().square().sum()
            else:
                g = u.detach()
                v = X.schur(g)
                # the gradient of |D_hat u|^2 at u, handed on as a linear form
                loss = v.abs().square().sum()
                t = 2 * X.schur(v, True)
                form = (t.real * u.real + t.imag * u.imag).sum()
                (form / case["pairs"]).backward()
                total += float(loss) / case["pairs"]
                continue
            (loss / case["pairs"]).backward()
            total += float(loss) / case["pairs"]
        return total, torch.cat([w.grad.reshape(-1) for w in W])
    if op == "dfl":
        eta = X.unpack(d["x"], 2)
        start = torch.stack([X.unpack(v, 2, 2) for v in d["start"]])
        return X.pack(X.deflated(eta, start, case) * X.even, 2)
    if op in ("cg", "fgcr"):
        return X.solve(d["b"].reshape(*X.Le, 4, 3)).reshape(X.V, 4, 3)
    b = X.unpack(d["b"], 1)
    return [X.pack(X.normal_cg(b, s), 1) for s in _shifts(case)]
