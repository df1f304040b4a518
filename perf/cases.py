"""The calls whose speed is measured: what a user's program has the library do.

Three kinds of work are covered, over the lattices, source counts and settings
of the tests and the benchmark:

* H_W alone on a batch of spinors (FP64 and FP32 arithmetic);
* sgn(H_W) b and D_ov(m_q) b through the shifted solver, in the forms and
  precisions a caller selects, one field at a time or several fields in one
  batched solve;
* the action |D_ov phi|^2 and its derivative with respect to the links
  (autograd forward and backward), with a new gauge field on every call.

A case is a dict of plain values; `prepare` makes seeded fields, sources and
the contexts a program keeps, `run` is one call, `exact` the same result from
plain torch in 64 bits.
"""
import math

import numpy as np
import torch

from paper_2204_01583_amd import ovl

M0, MQ = 1.4, 0.1
CIRCLE = (1.3, 1.2999, 1.0)      # centre, radius, vertical scaling (m0 = 1.4)
ELLIPSE = (1.2, 1.1999, 0.1)     # the paper's contour (m0 = 1)
BC = (1, 1, 1, -1)
FORMS = {"basis": ovl.FORM_BASIS, "twopass": ovl.FORM_TWOPASS, "fused": ovl.FORM_FUSED}


def _lat(dims):
    return {"lx": dims[0], "ly": dims[1], "lz": dims[2], "lt": dims[3]}


def _case(name, kind, dims, nrhs, **kw):
    c = {"kind": kind, **_lat(dims), "nrhs": nrhs, "rough": 0.3, **kw}
    return {"name": name, **c} if name else c


def _hw(name, dims, nrhs, prec="fp64", rough=0.3):
    return _case(name, "hw", dims, nrhs, prec=prec, rough=rough)


def _solve(name, kind, dims, nrhs, form="basis", prec="fp64", nq=64, contour="circle", tol=1e-12,
           rough=0.3):
    return _case(name, kind, dims, nrhs, form=form, prec=prec, nq=nq, contour=contour, tol=tol,
                 rough=rough)


def _batch(name, jobs, nrhs, prec="mixed", rough=0.3):
    # jobs: "8x8x8x8*16;12x12x12x12*2"
    return {**({"name": name} if name else {}), "kind": "batch", "jobs": jobs, "nrhs": nrhs,
            "form": "twopass", "prec": prec, "nq": 64, "contour": "circle", "tol": 1e-12,
            "rough": rough}


def _force(name, dims, prec="fp64", nq=64, rough=0.3):
    return _case(name, "force", dims, 1, form="basis", prec=prec, nq=nq, contour="circle",
                 tol=1e-12, rough=rough)


def listed():
    return [
        # the smallest call: one operator application on the smallest test
        # lattice, where launches and host work are all there is
        _hw("hw-smallest", (4, 4, 4, 4), 1),
        # an operator application as an outer (non-library) iteration does it,
        # at the benchmark's lattice and source count
        _hw("hw-ordinary", (16, 16, 16, 16), 4),
        # the FP32 operator on a ragged lattice (partial tiles and blocks)
        _hw("hw-fp32-ragged", (10, 6, 14, 9), 3, prec="fp32"),
        # the twelve spin-colour sources of a propagator on the largest lattice
        _hw("hw-propagator", (16, 16, 16, 32), 12),
        # the paper's own workload: one vector on its 8^4 lattice, its ellipse,
        # FP64 to 1e-14
        _solve("sign-paper", "sign", (8, 8, 8, 8), 1, nq=250, contour="ellipse", tol=1e-14),
        # FP64 sign function on a ragged lattice, a few sources
        _solve("sign-fp64-ragged", "sign", (12, 10, 6, 14), 2),
        # the settings a caller gets who chooses none (FP64, swept directions)
        _solve("sign-default", "sign", (12, 12, 12, 12), 2, form="fused"),
        # the benchmark: D_ov on four sources at 16^4, mixed precision
        _solve("dov-mixed", "dov", (16, 16, 16, 16), 4, prec="mixed", nq=128),
        # an ensemble of small fields in one batched solve
        _batch("batch-small", "8x8x8x8*16", 4),
        # fields of different sizes in one batched solve
        _batch("batch-uneven", "8x8x8x8*2;12x12x12x12*2;16x16x16x32*1", 4),
        # action and derivative of one pseudofermion, forward and backward,
        # small and ordinary lattice
        _force("force-small", (8, 8, 8, 8)),
        _force("force-ordinary", (16, 16, 16, 16), prec="mixed"),
    ]


def _extents(rng, vmax):
    """Random extents, volumes spread over their logarithm from 4^4 to vmax,
    even and odd; the last extent is the time direction."""
    v = math.exp(rng.uniform(math.log(256), math.log(vmax)))
    while True:
        d = []
        for i in range(4):
            top = 32 if i == 3 else 16
            d.append(min(top, max(3, round(v ** 0.25 * math.exp(rng.uniform(-0.5, 0.5))))))
        if rng.random() < 0.5:
            d = [min(x + (x & 1), 16 if i < 3 else 32) for i, x in enumerate(d)]
        V = d[0] * d[1] * d[2] * d[3]
        if 0.6 * v <= V <= min(1.4 * v, vmax):
            return tuple(d)


def draw(rng):
    kind = rng.choice(["hw", "hw", "basis", "basis", "basis", "fused", "batch", "force"])
    rough = round(rng.uniform(0.2, 0.4), 3)
    if kind == "hw":
        d = _extents(rng, 131072)
        n = max(1, round(math.exp(rng.uniform(0, math.log(12.4)))))
        return _hw(None, d, n, prec=rng.choice(["fp64", "fp64", "fp32"]), rough=rough)
    if kind == "basis":
        d = _extents(rng, 65536)
        return _solve(None, rng.choice(["sign", "dov"]), d, rng.randint(1, 4), form="basis",
                      prec=rng.choice(["fp64", "mixed"]), nq=2 * rng.randint(16, 64), rough=rough)
    if kind == "fused":
        d = _extents(rng, 20736)
        return _solve(None, "sign", d, rng.randint(1, 2), form="fused", nq=2 * rng.randint(8, 32),
                      prec=rng.choice(["fp64", "fp64", "mixed"]), rough=rough)
    if kind == "batch":
        jobs = []
        for _ in range(rng.randint(2, 4)):
            d = _extents(rng, 20736)
            jobs.append("%dx%dx%dx%d*%d" % (*d, rng.randint(1, 4 if math.prod(d) < 6000 else 1)))
        return _batch(None, ";".join(jobs), rng.randint(1, 4), prec=rng.choice(["fp64", "mixed"]),
                      rough=rough)
    d = _extents(rng, 30000)
    return _force(None, d, prec=rng.choice(["fp64", "mixed"]), nq=2 * rng.randint(8, 32),
                  rough=rough)


# ---- inputs ---------------------------------------------------------------
def _jobs(case):
    """[(dims, index)] of every field of the case."""
    if case["kind"] != "batch":
        return [(case["lx"], case["ly"], case["lz"], case["lt"])]
    out = []
    for part in case["jobs"].split(";"):
        d, n = part.split("*")
        out += [tuple(int(x) for x in d.split("x"))] * int(n)
    return out


def _gell_mann():
    g = np.zeros((8, 3, 3), dtype=np.complex128)
    g[0][0, 1] = g[0][1, 0] = 1
    g[1][0, 1], g[1][1, 0] = -1j, 1j
    g[2][0, 0], g[2][1, 1] = 1, -1
    g[3][0, 2] = g[3][2, 0] = 1
    g[4][0, 2], g[4][2, 0] = -1j, 1j
    g[5][1, 2] = g[5][2, 1] = 1
    g[6][1, 2], g[6][2, 1] = -1j, 1j
    g[7] = np.diag([1, 1, -2]) / math.sqrt(3)
    return g


def _mm(a, b):
    return (a.unsqueeze(-1) * b.unsqueeze(-3)).sum(-2)


def _field(dims, rough, gen):
    """SU(3) links exp(i rough sum_k a_k lambda_k), a_k normal, complex128
    [4][Lt][Lz][Ly][Lx][3][3]."""
    lx, ly, lz, lt = dims
    a = torch.randn((4, lt, lz, ly, lx, 8), generator=gen, dtype=torch.float64, device="cuda")
    lam = torch.from_numpy(_gell_mann()).cuda()
    A = (1j * rough / 64) * sum(a[..., k, None, None] * lam[k] for k in range(8))
    one = torch.eye(3, dtype=torch.complex128, device="cuda")
    E = one + A / 14
    for n in range(13, 0, -1):       # Taylor series of exp(A), then six squarings
        E = one + _mm(A, E) / n
    for _ in range(6):
        E = _mm(E, E)
    return E.contiguous()


def _sources(dims, n, gen):
    lx, ly, lz, lt = dims
    return torch.view_as_complex(torch.randn((n, lt, lz, ly, lx, 4, 3, 2), generator=gen,
                                             dtype=torch.float64, device="cuda"))


def _m0(case):
    return 1.0 if case.get("contour") == "ellipse" else M0


def _inputs(case, seed):
    """(links, sources) per field, from the seed alone."""
    out = []
    for i, dims in enumerate(_jobs(case)):
        gen = torch.Generator(device="cuda").manual_seed(int(seed) * 1009 + i)
        out.append((_field(dims, case["rough"], gen), _sources(dims, case["nrhs"], gen)))
    return out


def _context(case, dims):
    c = ovl.Context(dims, bc=BC, device=0)
    c.set_masses(_m0(case), MQ)
    if case["kind"] != "hw":
        c.set_contour(case["nq"], *(ELLIPSE if case["contour"] == "ellipse" else CIRCLE))
        c.set_solver(ovl.PREC_MIXED if case["prec"] == "mixed" else ovl.PREC_FP64,
                     FORMS[case["form"]], tol=case["tol"], maxiter=4000,
                     switch_res=1e-4 if case["kind"] == "force" else 1e-3)
    return c


def prepare(case, seed):
    fields = _inputs(case, seed)
    ctxs = [_context(case, d) for d in _jobs(case)]
    if case["kind"] == "force":
        return {"case": case, "ctx": ctxs[0], "U": fields[0][0].requires_grad_(),
                "phi": fields[0][1]}
    for c, (U, _) in zip(ctxs, fields):
        c.set_gauge(U)
    return {"case": case, "ctxs": ctxs, "ctx": ctxs[0], "b": [b for _, b in fields]}


def run(state):
    case, ctx = state["case"], state["ctx"]
    kind = case["kind"]
    if kind == "hw":
        b = state["b"][0]
        return ctx.apply_hw(b) if case["prec"] == "fp64" else ctx.apply_hw_fp32(b)
    if kind == "sign":
        return ctx.apply_sign(state["b"][0])[0]
    if kind == "dov":
        return ctx.apply_dov(state["b"][0])[0]
    if kind == "batch":
        return ovl.apply_sign_batched(state["ctxs"], state["b"])[0]
    S = ovl.OverlapAction.apply(state["U"], state["phi"], ctx)
    (G,) = torch.autograd.grad(S, state["U"])
    return {"action": S.detach(), "grad": G}


def work(case):
    """Every operator application reads its links (two rows of each, the third
    follows for SU(3)) and its input once and writes its output once; 1368
    floating point operations per site and source.  A solve is its operator
    applications (about 450 per solve to 1e-12 on the circle, 940 on the
    paper's ellipse to 1e-14; the mixed solves run three quarters of them in
    FP32); the derivative is two solves."""
    n = case["nrhs"]
    nbytes = flops = 0.0
    for d in _jobs(case):
        V = math.prod(d)
        if case["kind"] == "hw":
            es = 8 if case["prec"] == "fp32" else 16
            # caller's vectors are complex128 whatever the arithmetic
            nbytes += V * (24 * es + 24 * 16 * n)
            flops += 1368.0 * V * n
            continue
        its = 940 if case["contour"] == "ellipse" else 450
        its *= 2 if case["kind"] == "force" else 1
        es = 10 if case["prec"] == "mixed" else 16
        nbytes += its * V * es * (24 + 24 * n) + 24 * 16 * V * n
        flops += its * 1368.0 * V * n
        if case["kind"] == "force":
            nbytes += 2 * 36 * 16 * V
    return {"bytes": nbytes, "flops": flops}


# ---- the same results in plain torch --------------------------------------
def _gammas():
    s = np.array([[[0, 1], [1, 0]], [[0, -1j], [1j, 0]], [[1, 0], [0, -1]]], dtype=np.complex128)
    g = np.zeros((4, 4, 4), dtype=np.complex128)
    for k in range(3):
        g[k, :2, 2:], g[k, 2:, :2] = -1j * s[k], 1j * s[k]
    g[3, :2, 2:] = g[3, 2:, :2] = np.eye(2)
    return g


class _Wilson:
    """H_W = gamma5 D_W(-m0) on [n][Lt][Lz][Ly][Lx][4][3]."""

    def __init__(self, U, m0):
        self.U, self.kappa = U.detach(), 1.0 / (2.0 * (4.0 - m0))
        one = np.eye(4)
        g5 = np.diag([1.0, 1, -1, -1])
        self.g5 = torch.tensor([1.0, 1, -1, -1], dtype=torch.float64, device="cuda")[:, None]
        self.fwd = [torch.from_numpy(g5 @ (one - g)).cuda() for g in _gammas()]
        self.bwd = [torch.from_numpy(g5 @ (one + g)).cuda() for g in _gammas()]

    def phase(self, mu, edge):
        """Boundary factor of a hop in direction mu, at coordinate `edge`."""
        L = self.U.shape[4 - mu]
        p = torch.ones(L, dtype=torch.float64, device="cuda")
        p[edge] = BC[mu]
        shape = [1, 1, 1, 1]
        shape[3 - mu] = L
        return p.view(shape)[..., None, None]

    @staticmethod
    def spin(M, x):
        # the spin matrices have two entries a row
        rows = []
        for a in range(4):
            nz = [b for b in range(4) if M[a, b] != 0]
            rows.append(sum(M[a, b] * x[..., b, :] for b in nz))
        return torch.stack(rows, -2)

    @staticmethod
    def colour(u, x):
        # (u x)_a = sum_b u_ab x_b for every spin
        return sum(u[..., None, :, b] * x[..., b, None] for b in range(3))

    def __call__(self, x):
        out = self.g5 * x
        for mu in range(4):
            dim = x.dim() - 3 - mu
            u = self.U[mu]
            f = self.colour(u, torch.roll(x, -1, dim)) * self.phase(mu, -1)
            w = torch.roll(self.colour(u.mH, x), 1, dim) * self.phase(mu, 0)
            out = out - self.kappa * (self.spin(self.fwd[mu], f) + self.spin(self.bwd[mu], w))
        return out


def _nodes(case):
    g, r, al = ELLIPSE if case["contour"] == "ellipse" else CIRCLE
    nq = case["nq"]
    th = 2 * np.pi * (np.arange(1, nq + 1) - 0.5) / nq
    e, w = r * (np.cos(th) + 1j * al * np.sin(th)), r * (al * np.cos(th) + 1j * np.sin(th)) / nq
    return np.concatenate([g + e, -g + e]), np.concatenate([w, -w])


def _lanczos(H, b, coef):
    """Rows sum_i coef(T)[j, i] v_i |b| from the Lanczos vectors v_i of H and b
    (one source), coef a function of T's eigenvalues and eigenvectors; run
    until its last coefficients vanish."""
    nb = float(torch.linalg.vector_norm(b))
    v, prev, beta = b / nb, None, 0.0
    V, al, be = [v], [], []
    while True:
        w = H(v)
        a = float((v.conj() * w).sum().real)
        w = w - a * v - (beta * prev if prev is not None else 0)
        beta = float(torch.linalg.vector_norm(w))
        al.append(a)
        if len(al) % 48 == 0 or beta < 1e-13 or len(al) >= 2400:
            T = np.diag(al) + np.diag(be, 1) + np.diag(be, -1)
            lam, Q = np.linalg.eigh(T)
            y = coef(lam, Q)
            tail = np.abs(y[:, -24:]).max() / np.abs(y).max()
            if tail < 1e-14 or beta < 1e-13 or len(al) >= 2400:
                break
        be.append(beta)
        prev, v = v, w / beta
        V.append(v)
    y = torch.from_numpy(np.ascontiguousarray(nb * y)).cuda()
    out = torch.zeros((y.shape[0], b.numel()), dtype=torch.complex128, device="cuda")
    for i in range(0, len(V), 64):
        out += y[:, i:i + 64] @ torch.stack([t.reshape(-1) for t in V[i:i + 64]])
    return out


def _sign(case, H, b):
    z, c = _nodes(case)

    def coef(lam, Q):
        f = (c[:, None] / (z[:, None] - lam[None, :])).sum(0)
        return ((Q * f) @ Q[0])[None, :]

    return _lanczos(H, b, coef).view(b.shape)


def _shifted(z, H, b):
    """(z_j - H)^-1 b for every node, [J][*b.shape]."""
    def coef(lam, Q):
        return (Q[0] / (z[:, None] - lam[None, :])) @ Q.T

    return _lanczos(H, b, coef).view(len(z), *b.shape)


def _force_exact(case, U, phi):
    z, c = _nodes(case)
    H = _Wilson(U, M0)
    phi = phi[0]
    Y = _shifted(z, H, phi)
    ct = torch.from_numpy(c).cuda().view(-1, 1, 1, 1, 1, 1, 1)
    d = 0.5 * (1 + MQ) * phi + 0.5 * (1 - MQ) * H.g5 * (ct * Y).sum(0)
    psi = 0.5 * (1 - MQ) * H.g5 * d
    X = _shifted(z.conj(), H, psi)
    Xc = (X.conj() * ct)
    G = []
    for mu in range(4):
        dim = 1 + 3 - mu
        # dS = 2 Re sum_j c_j X_j^dag dH Y_j, dH = -kappa (hops with dU)
        A = torch.zeros(U.shape[1:], dtype=torch.complex128, device="cuda")
        B = torch.zeros_like(A)
        for j in range(len(z)):
            fy = H.spin(H.fwd[mu], torch.roll(Y[j:j + 1], -1, dim))[0]
            by = H.spin(H.bwd[mu], Y[j])
            xb = torch.roll(Xc[j:j + 1], -1, dim)[0]
            for s in range(4):
                A += Xc[j][..., s, :, None] * fy[..., s, None, :]
                B += xb[..., s, :, None] * by[..., s, None, :]
        G.append(-2 * H.kappa * H.phase(mu, -1) * (A.conj() + B.transpose(-1, -2)))
    return {"action": (d.abs() ** 2).sum(), "grad": torch.stack(G)}


def exact(case, seed):
    jobs = _jobs(case)
    if case["kind"] != "hw":
        # operator applications on one source take about 3 ms at 16^4 here
        sites = sum(math.prod(d) for d in jobs) * case["nrhs"]
        if sites > 300000 or (case["kind"] == "batch" and len(jobs) * case["nrhs"] > 16):
            return None
    with torch.no_grad():
        fields = _inputs(case, seed)
        if case["kind"] == "hw":
            return _Wilson(fields[0][0], M0)(fields[0][1])
        if case["kind"] == "force":
            return _force_exact(case, *fields[0])
        out = []
        for U, b in fields:
            H = _Wilson(U, _m0(case))
            s = torch.stack([_sign(case, H, b[i]) for i in range(b.shape[0])])
            if case["kind"] == "dov":
                s = 0.5 * (1 + MQ) * b + 0.5 * (1 - MQ) * H.g5 * s
            out.append(s)
        return out if case["kind"] == "batch" else out[0]
