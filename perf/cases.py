"""The work that users have this library do, as cases that can be timed and compared.

A case goes through the public entry points (the ctypes binding of the C ABI, or the
serving loop on top of it) with everything resident that a program keeps between calls:
a context, the gauge field, a server.  Kinds:

  solve   wilson_solve_ex on a resident field: plain FP64 or mixed precision, one or several
          right-hand sides, BiCGStab or CG on the normal equations, Wilson or clover matrix
  dslash  wilson_dslash_ex on a resident field: D on the whole lattice (parity 2) or one
          parity hop (0, 1), in any of the precisions
  plain   wilson_dslash: the two-call form, which takes the links with every call
  serve   requests with several right-hand sides through the continuous-batching server

Inputs follow the library's benchmark: links exp(i eps A) with Gaussian traceless Hermitian
A, complex Gaussian or point sources, a clover term of two chiral Hermitian blocks.
"""
import math

import numpy as np
import torch

from paper_1811_00893_amd import _lib as L
from paper_1811_00893_amd.serve import Request, make_server

FP64, FP32, FP16, FP16_L32 = L.WILSON_FP64, L.WILSON_FP32, L.WILSON_FP16, L.WILSON_FP16_L32


def _case(name, kind, dims, **more):
    c = {"name": name, "kind": kind, "lx": dims[0], "ly": dims[1], "lz": dims[2], "lt": dims[3], "kappa": 0.125,
         "eps": 0.3, "tol": 1e-10, "precision": FP64, "nrhs": 1}
    c.update(more)
    return c


def listed():
    return [
        # the smallest solve: everything is in the caches, launches and latency count
        _case("solve 8^4 fp64", "solve", (8, 8, 8, 8), kappa=0.12),
        # the flagship: one propagator column on an ordinary lattice, FP64 throughout
        _case("solve 32^3x64 fp64", "solve", (32, 32, 32, 64)),
        # an ordinary lattice in the lowest precision that keeps FP32 links
        _case("solve 32^3x64 fp16", "solve", (32, 32, 32, 64), precision=FP16_L32),
        # the largest lattice, FP32 inner iterations and FP64 defect correction
        _case("solve 48^3x96 fp32", "solve", (48, 48, 48, 96), precision=FP32),
        # a whole point-to-all propagator: the 12 spin-colour point sources in one call
        _case("solve 24^3x48 fp32 12 rhs", "solve", (24, 24, 24, 48), precision=FP32, nrhs=12, point=True),
        # the clover matrix in mixed precision
        _case("solve 24^3x48 clover fp32", "solve", (24, 24, 24, 48), precision=FP32, clover=True),
        # extents that fit no tile, the second Krylov method
        _case("solve 20x12x28x36 cgnr fp64", "solve", (20, 12, 28, 36), solver=L.WILSON_SOLVER_CGNR_EO),
        # the smallest operator call (a program's own Krylov method on a small lattice)
        _case("D 8^4 fp64", "dslash", (8, 8, 8, 8), parity=2),
        # the whole operator on an ordinary lattice (residual checks, a program's own solver)
        _case("D 32^3x64 fp64", "dslash", (32, 32, 32, 64), parity=2),
        # one parity hop of 12 right-hand sides in single precision (an outside even-odd solver)
        _case("hop 24^3x48 fp32 12 rhs", "dslash", (24, 24, 24, 48), precision=FP32, nrhs=12, parity=1),
        # the two-call form: links come with the call
        _case("plain D 16^3x32", "plain", (16, 16, 16, 32), parity=2),
        # three requests of 1, 4 and 5 right-hand sides, own kappa and tolerance each, answered on the host
        _case("serve 16^3x32 fp32", "serve", (16, 16, 16, 32), precision=FP32, nrhs=10, kappa=0.12),
    ]


def _dims(c):
    return (int(c["lx"]), int(c["ly"]), int(c["lz"]), int(c["lt"]))


def _volume(c):
    return math.prod(_dims(c))


# (kind, options, smallest and largest number of sites): what draw() picks from
_RANGES = [
    ("solve", {}, 8 ** 4, 32 ** 3 * 64),
    ("solve", {"precision": FP32}, 8 ** 4, 32 ** 3 * 64),
    ("solve", {"precision": FP16_L32}, 16 ** 4, 32 ** 3 * 64),
    ("solve", {"precision": FP32, "nrhs": 12}, 8 ** 4, 24 ** 3 * 48),
    ("solve", {"precision": FP32, "nrhs": 0}, 8 ** 4, 24 ** 3 * 48),
    ("solve", {"precision": FP32, "clover": True}, 8 ** 4, 24 ** 3 * 48),
    ("solve", {"solver": L.WILSON_SOLVER_CGNR_EO}, 8 ** 4, 24 ** 3 * 48),
    ("dslash", {"parity": 2}, 8 ** 4, 32 ** 3 * 64),
    ("dslash", {"parity": 2}, 8 ** 4, 16 ** 4),
    ("dslash", {"parity": 1, "precision": FP32, "nrhs": 0}, 8 ** 4, 24 ** 3 * 48),
    ("plain", {"parity": 2}, 8 ** 4, 24 ** 3 * 48),
    ("serve", {"precision": FP32, "nrhs": 10}, 8 ** 4, 24 ** 3 * 48),
]


def draw(rng):
    kind, more, lo, hi = rng.choice(_RANGES)
    more = dict(more)
    target = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    # even extents around the fourth root, t the longest, ragged more often than not
    side = (target / 2.0) ** 0.25
    while True:
        xyz = [max(4, 2 * round(side * math.exp(rng.uniform(-0.35, 0.35)) / 2.0)) for _ in range(3)]
        lt = max(4, 2 * round(target / math.prod(xyz) / 2.0))
        if lo <= math.prod(xyz) * lt <= hi:
            break
    if more.get("nrhs") == 0:
        more["nrhs"] = rng.choice([2, 3, 4, 5, 7, 12])
    c = _case("", kind, (*xyz, lt), kappa=round(rng.uniform(0.115, 0.125), 4), eps=round(rng.uniform(0.2, 0.4), 3), **more)
    if kind == "solve":
        c["tol"] = rng.choice([1e-8, 1e-10])
    del c["name"]
    return c


# ---- inputs ------------------------------------------------------------------------
def _randn(shape, gen):
    a = torch.randn((*shape, 2), generator=gen, device="cuda", dtype=torch.float64)
    return torch.view_as_complex(a)


def _mul3(a, b):
    """Products of 3x3 matrices, elementwise over the leading dimension."""
    return a[:, :, 0:1] * b[:, 0:1, :] + a[:, :, 1:2] * b[:, 1:2, :] + a[:, :, 2:3] * b[:, 2:3, :]


def _links(V, eps, gen):
    """exp(i eps A), A traceless Hermitian from Gaussian matrices, (V, 4, 3, 3)."""
    U = torch.empty((V, 4, 3, 3), dtype=torch.complex128, device="cuda")
    flat = U.view(-1, 3, 3)
    eye = torch.eye(3, dtype=torch.complex128, device="cuda")
    for i in range(0, flat.shape[0], 1 << 23):
        M = _randn(flat[i:i + (1 << 23)].shape, gen)
        H = 0.5 * (M + M.mH)
        H = H - (torch.diagonal(H, dim1=-2, dim2=-1).sum(-1).real / 3.0)[:, None, None] * eye
        X = (1j * eps / 16.0) * H
        E = eye.expand_as(X).clone()  # Taylor sum of exp(X) by Horner's rule, then four squarings
        for k in range(11, 0, -1):
            E = eye + _mul3(X, E) / k
        for _ in range(4):
            E = _mul3(E, E)
        flat[i:i + (1 << 23)] = E
    return U


_G5 = torch.tensor([[0., 0., -1., 0.], [0., 0., 0., -1.], [-1., 0., 0., 0.], [0., -1., 0., 0.]], dtype=torch.float64)


def _clover(V, gen, c=0.05):
    """A Hermitian 12x12 matrix per site that commutes with gamma5."""
    g5 = torch.kron(_G5, torch.eye(3, dtype=torch.float64)).to("cuda", torch.complex128)
    F = torch.empty((V, 12, 12), dtype=torch.complex128, device="cuda")
    for i in range(0, V, 1 << 18):
        M = _randn(F[i:i + (1 << 18)].shape, gen)
        G = 0.5 * (M + M.mH)
        F[i:i + (1 << 18)] = 0.5 * c * (G + g5 @ (G @ g5))  # the part of G that commutes with gamma5
    return F


def _inputs(case, seed):
    V, n = _volume(case), int(case["nrhs"])
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 7919 + 17)
    U = _links(V, float(case["eps"]), gen)
    F = _clover(V, gen) if case.get("clover") else None
    if case.get("point"):
        b = torch.zeros((n, V, 4, 3), dtype=torch.complex128, device="cuda")
        for k in range(n):
            b[k, 0, (k // 3) % 4, k % 3] = 1.0
    else:
        b = _randn((n, V, 4, 3), gen)
    return U, F, b


# the serving requests: right-hand sides, kappa relative to the case's, tolerance
_REQUESTS = [(1, 1.0, 1e-8), (4, 0.98, 1e-10), (5, 1.03, 1e-10)]


class _Session:
    """A context and a resident gauge field, released with the object."""

    def __init__(self, U, F, dims, bits):
        self.ctx = L.wilson_context_create()
        self.g = L.wilson_gauge_load(self.ctx, U, dims, bits)
        if F is not None:
            L.check(L.wilson_gauge_attach_clover(self.ctx, self.g, F, dims), "attach_clover")

    def __del__(self):
        L.wilson_gauge_free(self.ctx, self.g)
        L.wilson_context_destroy(self.ctx)


class _Server:
    """A server with one gauge field, closed with the object."""

    def __init__(self, U, dims):
        self.sch, self.eng = make_server(hbm_budget=100e9, nslots=12, step_iters=32, precision=FP32, turn_ms=3.0,
                                         max_heavy=2, host_results=True)
        torch.cuda.synchronize()  # the server's stream does not wait for the default one
        self.sch.register_gauge("field", dims, self.eng.load_gauge("field", U, dims))

    def __del__(self):
        self.sch.close()
        self.eng.close()


def prepare(case, seed):
    dims, kind = _dims(case), case["kind"]
    U, F, b = _inputs(case, seed)
    s = {"case": dict(case), "dims": dims, "b": b}
    if kind == "serve":
        s["server"] = _Server(U, dims)
        torch.cuda.synchronize()
    elif kind == "plain":
        s["U"], s["out"] = U, torch.zeros_like(b)
    else:
        bits = {FP64: L.WILSON_GAUGE_FP64, FP32: L.WILSON_GAUGE_FP32, FP16: L.WILSON_GAUGE_FP16,
                FP16_L32: L.WILSON_GAUGE_FP32}[case["precision"]]
        s["lib"] = _Session(U, F, dims, bits)
        s["out"] = torch.zeros_like(b)
        s["opts"] = {"solver": int(case.get("solver", L.WILSON_SOLVER_BICGSTAB_EO)), "precision": int(case["precision"]),
                     "maxiter": 10000}
    return s


def run(state):
    c, b, kind = state["case"], state["b"], state["case"]["kind"]
    if kind == "solve":
        lib = state["lib"]
        st, _ = L.wilson_solve_ex(lib.ctx, lib.g, state["out"], b, c["nrhs"], c["kappa"], c["tol"], state["opts"])
        if L.check(st, "wilson_solve_ex") != L.WILSON_OK:
            raise RuntimeError("the solve did not converge")
        return list(state["out"])
    if kind == "dslash":
        lib = state["lib"]
        L.check(L.wilson_dslash_ex(lib.ctx, lib.g, state["out"], b, c["kappa"], c["parity"], c["precision"], c["nrhs"]),
                "wilson_dslash_ex")
        return state["out"]
    if kind == "plain":
        L.check(L.wilson_dslash(state["out"], b, state["U"], c["kappa"], state["dims"], c["parity"]), "wilson_dslash")
        return state["out"]
    sch, k, reqs = state["server"].sch, 0, []
    for i, (n, f, tol) in enumerate(_REQUESTS):
        reqs.append(Request(rid=i, gauge_id="field", kappa=c["kappa"] * f, tol=tol, b=b[k:k + n]))
        k += n
        if not sch.submit(reqs[-1]):
            raise RuntimeError("request rejected")
    sch.run_until_idle()
    sch.completed.clear()
    if any(st != L.WILSON_OK for r in reqs for st in r.status):
        raise RuntimeError("a request did not converge")
    return [list(r.x) for r in reqs]


def work(case):
    """Bytes and flops of one pass: every input read once and every output written once; a
    Krylov iteration applies the even-odd operator twice, reads the links (two rows) once for
    each application and each of its vectors once per step that needs it."""
    V, n, kind = float(_volume(case)), float(case["nrhs"]), case["kind"]
    real = {FP64: 8.0, FP32: 4.0, FP16: 2.0, FP16_L32: 2.0}[case["precision"]]
    link = 4.0 if case["precision"] in (FP32, FP16_L32) else real
    site = 4.0 * 12.0 * link + (144.0 * real if case.get("clover") else 0.0)
    if kind == "plain":
        return {"bytes": V * (4 * 18 * 8 + 2 * 192.0), "flops": 1368.0 * V}
    if kind == "dslash":
        one = case["parity"] != 2
        spinors = 192.0 if one else 384.0  # half the lattice in, half out, or all of both
        return {"bytes": V * (4.0 * 12.0 * link + spinors * n), "flops": (660.0 if one else 1368.0) * V * n}
    # iterations to these tolerances at kappa 0.12-0.125 (measured: 19-28); BiCGStab reads or
    # writes 10 half-lattice vectors an iteration besides the two operator applications
    # (in, out each), CG on the normal equations 6 and needs about 1.4 times as many
    iters, vecs = (26.0, 14.0) if case.get("solver", 0) == 0 else (36.0, 10.0)
    half = 12.0 * real * V  # one half-lattice vector: 24 reals on V / 2 sites
    return {"bytes": 384.0 * V * n + iters * (2.0 * V * site + n * vecs * half),
            "flops": iters * n * V * (2.0 * 1368.0 + vecs * 24.0)}


# ---- the same results in plain torch, 64 bits ----------------------------------------
def _gammas():
    s = [np.array([[0, 1], [1, 0]], complex), np.array([[0, -1j], [1j, 0]]), np.array([[1, 0], [0, -1]], complex)]
    z = np.zeros((2, 2))
    return [np.block([[z, -1j * m], [1j * m, z]]) for m in s] + [np.diag([1, 1, -1, -1]).astype(complex)]


def _gamma_times(mu):
    """gamma_mu psi as a permutation of the spins with phases."""
    g = _gammas()[mu]
    perm = [int(np.flatnonzero(g[r])[0]) for r in range(4)]
    phase = torch.tensor([g[r, perm[r]] for r in range(4)], dtype=torch.complex128, device="cuda")[:, None]
    return lambda p: p[..., perm, :] * phase


def _colour(U, h, adjoint):
    """U h or U^dagger h: U (..., 3, 3), h (..., 4, 3)."""
    out = None
    for k in range(3):
        col = U[..., k, :].conj() if adjoint else U[..., :, k]
        t = col[..., None, :] * h[..., :, k, None]
        out = t if out is None else out.add_(t)
    return out


class _Exact:
    def __init__(self, dims, U, F, kappa):
        self.shape, self.kappa, self.F = (dims[3], dims[2], dims[1], dims[0]), kappa, F
        self.U = U.view(*self.shape, 4, 3, 3)
        self.gamma = [_gamma_times(mu) for mu in range(4)]

    def hop(self, psi):
        p = psi.view(*self.shape, 4, 3)
        out = torch.zeros_like(p)
        for mu in range(4):
            axis, g, U = 3 - mu, self.gamma[mu], self.U[..., mu, :, :]
            f = torch.roll(p, -1, axis)
            if mu == 3:
                f[-1].neg_()
            out += _colour(U, f - g(f), False)
            w = torch.roll(_colour(U, p + g(p), True), 1, axis)
            if mu == 3:
                w[0].neg_()
            out += w
        return out.view_as(psi)

    def D(self, psi):
        out = psi - self.kappa * self.hop(psi)
        if self.F is not None:
            v = psi.reshape(-1, 12)
            out += sum(self.F[:, :, k] * v[:, k:k + 1] for k in range(12)).view_as(out)
        return out

    def solve(self, b):
        """BiCGStab on the full system to rounding, restarted until the residual stays down."""
        dot = lambda u, v: torch.vdot(u.reshape(-1), v.reshape(-1))  # noqa: E731
        x, bn = torch.zeros_like(b), torch.linalg.vector_norm(b).item()
        for _ in range(4):
            r = b - self.D(x)
            if torch.linalg.vector_norm(r).item() < 2e-14 * bn:
                break
            rh, p = torch.randn_like(r), r.clone()  # (a point source as its own shadow breaks down)
            rho = dot(rh, r)
            stop = max(1e-8 * torch.linalg.vector_norm(r).item(), 1e-15 * bn)
            for _ in range(2000):
                v = self.D(p)
                alpha = rho / dot(rh, v)
                r = r - alpha * v
                t = self.D(r)
                omega = dot(t, r) / dot(t, t)
                x += alpha * p + omega * r
                r = r - omega * t
                if not torch.linalg.vector_norm(r).item() >= stop:
                    break
                new = dot(rh, r)
                p = r + (new / rho * alpha / omega) * (p - omega * v)
                rho = new
        return x


def _parity_mask(dims):
    t, z, y, x = torch.meshgrid(*[torch.arange(d, device="cuda") for d in reversed(dims)], indexing="ij")
    return ((x + y + z + t) % 2).reshape(-1)


def exact(case, seed):
    dims, kind = _dims(case), case["kind"]
    U, F, b = _inputs(case, seed)
    if kind == "serve":
        out, k = [], 0
        for n, f, _ in _REQUESTS:
            e = _Exact(dims, U, None, case["kappa"] * f)
            out.append([e.solve(v) if j == 0 else None for j, v in enumerate(b[k:k + n])])
            k += n
        return out
    e = _Exact(dims, U, F, case["kappa"])
    if kind == "solve":  # (one right-hand side of each call: the others would take too long)
        return [e.solve(v) if k == len(b) - 1 else None for k, v in enumerate(b)]
    if case["parity"] == 2:
        return torch.stack([e.D(v) for v in b])
    on = (_parity_mask(dims) == case["parity"])[:, None, None]
    return torch.stack([torch.where(on, -case["kappa"] * e.hop(v), 0.0) for v in b])
