"""Cases that time the framework's public entry points on one GPU.

A case is a dict of plain values: the kind of work, the lattice, the number of
right-hand sides, the inner precision and the physics parameters.  The kinds:

  apply    `Lattice.apply_dev`: the distance-preconditioned operator D' + M (or
           its adjoint, or the even-site Schur operator) on device spinors
  newconf  what a measurement program does with each configuration of an
           ensemble before its solves: links in, clover term built, operator
           applied (the new mass's inverse clover is built on the way)
  solve    `Lattice.solve_dev`: point-source columns to the residue r, with the
           restored propagator and C_PP
  sap      `Lattice.solve_sap_dev`: SAP+GCR on one column
  serve    `Batch`: the served stream's loop (admit, step, harvest) over a few
           requests of different masses, profiles, sources and column counts

Lattices, masses, profiles, residues and c_sw are those of the synthetic
workloads (synth/configs.py), the served stream and the SAP study; links are
drawn as in synth/fields.py, on the GPU.
"""
import math
import random

import numpy as np
import torch

import paper_1006_4028_amd as dp

CSW = 1.6


# ------------------------------------------------------------------ cases

def _case(kind, dims, name=None, **kw):
    c = dict(kind=kind, T=dims[0], L1=dims[1], L2=dims[2], L3=dims[3])
    if name:
        c["name"] = name
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: the operator on one spinor of the free-field workload's
        # lattice, as a user's own outer solver or eigensolver calls it (latency)
        _case("apply", (16, 8, 8, 8), "apply_f64_1rhs_8c16", nrhs=1, op="full", dagger=False, eps=0.3, csw=CSW, M=0.5,
              profile="exp", alpha0=0.4),
        # the adjoint operator on a whole propagator at the headline lattice
        _case("apply", (48, 24, 24, 24), "apply_dag_f64_12rhs_24c48", nrhs=12, op="full", dagger=True, eps=0.25,
              csw=CSW, M=0.5, profile="cosh", alpha0=0.4),
        # a new configuration on a ragged lattice (no extent a power of two, partial
        # waves), then the Schur operator on three columns
        _case("newconf", (36, 18, 20, 14), "newconf_schur_3rhs_ragged", nrhs=3, op="schur", dagger=False, eps=0.3,
              csw=CSW, M=0.2, profile="exp_sym", alpha0=0.1),
        # the smallest propagator: launch latency and host round trips of a solve
        _case("solve", (16, 8, 8, 8), "solve_f32_12col_8c16", ncols=12, solver="bicgstab", precision="f32", r=1e-11,
              eps=0.3, csw=0.0, M=0.5, profile="exp", alpha0=0.4),
        # one column of the interacting 16^3x32 workload
        _case("solve", (32, 16, 16, 16), "solve_f32_1col_16c32", ncols=1, solver="bicgstab", precision="f32", r=1e-11,
              eps=0.3, csw=CSW, M=0.5, profile="cosh", alpha0=0.4),
        # the headline propagator, 12 columns at 24^3x48, with each inner precision
        _case("solve", (48, 24, 24, 24), "solve_f32_12col_24c48", ncols=12, solver="bicgstab", precision="f32",
              r=1e-11, eps=0.25, csw=CSW, M=0.5, profile="cosh", alpha0=0.4),
        _case("solve", (48, 24, 24, 24), "solve_f64_12col_24c48", ncols=12, solver="bicgstab", precision="f64",
              r=1e-11, eps=0.25, csw=CSW, M=0.5, profile="cosh", alpha0=0.4),
        _case("solve", (48, 24, 24, 24), "solve_f16_12col_24c48", ncols=12, solver="bicgstab", precision="f16",
              r=1e-11, eps=0.25, csw=CSW, M=0.5, profile="cosh", alpha0=0.4),
        # the light-mass workload: one column at 32^3x64, CG on the normal
        # equations with FP16 storage
        _case("solve", (64, 32, 32, 32), "solve_cgnr_f16_1col_32c64", ncols=1, solver="cgnr", precision="f16",
              r=1e-11, eps=0.2, csw=CSW, M=0.01, profile="exp_sym", alpha0=0.05),
        # the two lattices and blockings of the SAP+GCR iteration study, with the
        # four-direction profile
        _case("sap", (64, 32, 32, 32), "sap_b4_32c64", block=4, r=1e-11, eps=0.2, csw=CSW, M=0.05, profile="beta",
              alpha0=0.05),
        _case("sap", (48, 24, 24, 24), "sap_b6_24c48", block=6, r=1e-11, eps=0.25, csw=CSW, M=0.05, profile="beta",
              alpha0=0.05),
        # a burst of served requests on one resident 16^3x32 field
        _case("serve", (32, 16, 16, 16), "serve_f32_6req_16c32", nreq=6, nslots=24, precision="f32", r=1e-11, eps=0.3,
              csw=CSW),
    ]


def _extents(rng, vmin, vmax):
    """Even extents of a lattice whose volume is spread over the logarithm of
    [vmin, vmax], time about twice the spatial extents, ragged more often than not."""
    while True:
        v = math.exp(rng.uniform(math.log(vmin), math.log(vmax)))
        base = (v / 2.0) ** 0.25
        d = [max(4, 2 * round(f * base * math.exp(rng.uniform(-0.3, 0.3)) / 2)) for f in (2, 1, 1, 1)]
        if 0.7 * vmin <= d[0] * d[1] * d[2] * d[3] <= vmax:
            return tuple(d)


def _volume(d):
    return d[0] * d[1] * d[2] * d[3]


def draw(rng):
    kind = rng.choice(["apply", "apply", "newconf", "solve", "solve", "solve", "solve", "sap", "serve"])
    profile, alpha0 = rng.choice([("cosh", 0.4), ("exp_sym", 0.1), ("exp_sym", 0.05), ("exp", 0.1), ("cosh", 0.0)])
    mild = rng.choice([("exp_sym", 0.05), ("exp_sym", 0.1), ("beta", 0.05)])
    M = rng.choice([0.05, 0.2, 0.5])
    eps = round(rng.uniform(0.2, 0.3), 3)
    com = dict(eps=eps, csw=CSW, profile=profile, alpha0=alpha0)
    if kind in ("apply", "newconf"):
        d = _extents(rng, 8192, 660000)
        n = rng.randint(1, 12) if kind == "apply" else rng.randint(1, 4)
        op = rng.choice(["full", "schur", "hop"]) if _volume(d) < 150000 else rng.choice(["full", "hop"])
        return _case(kind, d, nrhs=n, op=op, dagger=rng.random() < 0.5, M=M, **com)
    if kind == "solve":
        d = _extents(rng, 8192, 660000)
        n = rng.choice([1, 1, 2, 3, 4, 6, 9, 12])
        if rng.random() < 0.25:
            return _case(kind, d, ncols=min(n, 4), solver="cgnr", precision=rng.choice(["f16", "f32"]), r=1e-11,
                         M=rng.choice([0.05, 0.2]), **dict(com, profile="exp_sym", alpha0=rng.choice([0.0, 0.05, 0.1])))
        while n > 1 and _volume(d) * n > 6.0e6:
            n -= 1
        return _case(kind, d, ncols=n, solver="bicgstab", precision=rng.choice(["f32", "f32", "f16", "f64"]), r=1e-11,
                     M=M, **com)
    if kind == "sap":
        b = rng.choice([4, 4, 6])
        ext = (8, 16, 24, 32) if b == 4 else (12, 24)
        d = (rng.choice((16, 24, 32, 48) if b == 4 else (24, 36, 48)),) + tuple(rng.choice(ext) for _ in range(3))
        return _case(kind, d, block=b, r=1e-11, M=rng.choice([0.05, 0.2]),
                     **dict(com, profile=mild[0], alpha0=mild[1]))
    d = _extents(rng, 16384, 131072)
    return _case("serve", d, nreq=rng.randint(3, 6), nslots=24, precision=rng.choice(["f32", "f16", "f64"]), r=1e-11,
                 eps=eps, csw=CSW)


def _dims(case):
    return (case["T"], case["L1"], case["L2"], case["L3"])


# ----------------------------------------------------------------- inputs

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _mm(a, b):
    """Products of 3x3 matrices stored [3, 3, ...]."""
    return torch.stack([torch.stack([a[i, 0] * b[0, j] + a[i, 1] * b[1, j] + a[i, 2] * b[2, j] for j in range(3)])
                        for i in range(3)])


def _links(dims, eps, seed):
    """U = P_SU3[exp(i eps H)] with H Gaussian per link, [T, L1, L2, L3, 4, 3, 3]."""
    dev = _device()
    gen = torch.Generator(device=dev).manual_seed(seed)
    n = 4 * _volume(dims)
    h = torch.randn((8, n), generator=gen, device=dev, dtype=torch.float64)
    H = torch.zeros((3, 3, n), dtype=torch.complex128, device=dev)
    H[0, 0] = 0.5 * h[2] + h[7] / math.sqrt(12.0)
    H[1, 1] = -0.5 * h[2] + h[7] / math.sqrt(12.0)
    H[2, 2] = -h[7] / math.sqrt(3.0)
    for (i, j), (a, b) in {(0, 1): (0, 1), (0, 2): (3, 4), (1, 2): (5, 6)}.items():
        H[i, j] = torch.complex(0.5 * h[a], -0.5 * h[b])
        H[j, i] = torch.complex(0.5 * h[a], 0.5 * h[b])
    H *= 1j * eps / 4.0
    one = torch.eye(3, dtype=torch.complex128, device=dev)[:, :, None]
    E = one + H / 8.0  # exp(H) by its series, squared twice
    for k in range(7, 0, -1):
        E = one + _mm(H, E) / k
    E = _mm(E, E)
    E = _mm(E, E)
    r0 = E[0] / torch.sqrt((E[0].abs() ** 2).sum(0))
    r1 = E[1] - (r0.conj() * E[1]).sum(0) * r0
    r1 = r1 / torch.sqrt((r1.abs() ** 2).sum(0))
    r2 = torch.stack([r0[1] * r1[2] - r0[2] * r1[1], r0[2] * r1[0] - r0[0] * r1[2], r0[0] * r1[1] - r0[1] * r1[0]]).conj()
    U = torch.stack([r0, r1, r2])
    return U.permute(2, 0, 1).contiguous().reshape(tuple(dims) + (4, 3, 3))


def _spinors(dims, n, seed):
    gen = torch.Generator(device=_device()).manual_seed(seed + 77)
    x = torch.randn((n, 12 * _volume(dims), 2), generator=gen, device=_device(), dtype=torch.float64)
    return torch.view_as_complex(x)


def _profile(kind, T, alpha0, x0):
    t = (np.arange(T) - x0) % T
    if kind == "exp":
        return np.exp(alpha0 * t)
    if kind == "exp_sym":
        return np.exp(alpha0 * np.minimum(t, T - t))
    return 1.0 / np.cosh(alpha0 * (t - T / 2.0))


def _site(case, seed):
    rng = random.Random(seed)
    d = _dims(case)
    return tuple(rng.randrange(L) for L in d)


def _requests(case, seed):
    """Requests of the served stream (the recipe of serve.poisson_requests)."""
    rng = random.Random(seed)
    out = []
    for k in range(case["nreq"]):
        x0 = rng.randrange(case["T"])
        out.append(dict(M=rng.choice([0.01, 0.05, 0.2, 0.5]), alpha0=rng.choice([0.0, 0.1, 0.4]), x0=x0,
                        ncols=1 + (5 * k + 3 * case["nreq"]) % 12))
    return out


def _wait():
    """The library works on its own stream and does not wait for torch's default one."""
    if torch.cuda.is_available():
        torch.cuda.synchronize()


def _lattice(case, U):
    L = dp.Lattice(_dims(case))
    if U is not None:
        _wait()
        L.set_gauge(U)
        L.set_clover(case["csw"])
    return L


def prepare(case, seed):
    kind, d = case["kind"], _dims(case)
    U = _links(d, case["eps"], seed)
    if kind in ("apply", "newconf"):
        L = _lattice(case, U if kind == "apply" else None)
        L.set_mass(case["M"])
        L.set_alpha(_profile(case["profile"], d[0], case["alpha0"], 0))
        x = _spinors(d, case["nrhs"], seed)
        _wait()
        return dict(case=case, L=L, U=U if kind == "newconf" else None, x=x, y=torch.empty_like(x))
    L = _lattice(case, U)
    del U
    if kind == "serve":
        reqs = _requests(case, seed)
        eta = [L.point_sources((q["x0"], 0, 0, 0), 0, q["ncols"]) for q in reqs]
        alpha = [_profile("exp_sym", d[0], q["alpha0"], q["x0"]) for q in reqs]
        return dict(case=case, L=L, B=dp.Batch(L, case["nslots"], case["precision"]), reqs=reqs, eta=eta, alpha=alpha)
    L.set_mass(case["M"])
    n = case.get("ncols", 1)
    site = _site(case, seed)
    if kind == "sap":
        site = (0,) + site[1:]
    if case["profile"] == "beta":
        L.set_beta([np.cosh(case["alpha0"] * (np.arange(n_mu) - n_mu / 2.0)) for n_mu in d])
    else:
        L.set_alpha(_profile(case["profile"], d[0], case["alpha0"], site[0]))
    eta = L.point_sources(site, 0, n)
    return dict(case=case, L=L, eta=eta, S=torch.empty_like(eta), x0=site[0])


# -------------------------------------------------------------------- run

def run(state):
    case, L = state["case"], state["L"]
    kind = case["kind"]
    if kind in ("apply", "newconf"):
        if kind == "newconf":
            L.set_gauge(state["U"])
            L.set_clover(case["csw"])
        L.apply_dev(state["x"], state["y"], precond=True, dagger=case["dagger"], schur=case["op"] == "schur",
                    hop_only=case["op"] == "hop")
        return state["y"]
    if kind == "solve":
        cpp, _ = L.solve_dev(state["eta"], state["S"], r=case["r"], solver=case["solver"],
                             precision=case["precision"], x0_src=state["x0"], ncols_group=case["ncols"])
        return {"S": state["S"], "cpp": cpp}
    if kind == "sap":
        b = case["block"]
        cpp, _ = L.solve_sap_dev(state["eta"], state["S"], block=(b, b, b, b), r=case["r"])
        return {"S": state["S"], "cpp": cpp}
    B, reqs = state["B"], state["reqs"]
    waiting = list(range(len(reqs)))
    cpp = np.zeros((len(reqs), L.T))
    left = sum(q["ncols"] for q in reqs)
    while left:
        while waiting and B.status()["free"] >= reqs[waiting[0]]["ncols"]:
            k = waiting.pop(0)
            q = reqs[k]
            B.admit(state["eta"][k], None, M=q["M"], alpha=state["alpha"][k], r=case["r"], max_iter=20000,
                    x0_src=q["x0"], tag=k)
        B.step(4)
        for res in B.harvest():
            cpp[res["tag"]] += res["cpp"]
            left -= 1
    return cpp


# ------------------------------------------------------------------- work

def _operator_work(V, n, real):
    """One operator on n spinors: links (72 reals a site) and clover blocks (72) once,
    each spinor in and out; 1320 flops of hops, 552 of clover and 48 a site and column."""
    return V * (144 + 48 * n) * real, V * n * 1920.0


# inner iterations to r = 1e-11 on these fields, by mass (BiCGStab, CGNR, GCR)
_ITERS = {"bicgstab": {0.01: 140, 0.05: 110, 0.2: 60, 0.5: 33}, "cgnr": {0.01: 380, 0.05: 280, 0.2: 160, 0.5: 90},
          "gcr": {0.05: 16, 0.2: 12}}


def work(case):
    kind, V = case["kind"], _volume(_dims(case))
    if kind in ("apply", "newconf"):
        b, f = _operator_work(V, case["nrhs"], 8)
        if kind == "newconf":  # links in, clover blocks out
            b += V * (72 + 72) * 8
            f += V * 6 * 4 * 3 * 198.0
        return {"bytes": b, "flops": f}
    real = {"f64": 8, "f32": 4, "f16": 2}[case.get("precision", "f32")]
    if kind == "serve":
        # the generic draw: masses uniform over four, 1 to 12 columns a request
        n = sum(1 + (5 * k + 3 * case["nreq"]) % 12 for k in range(case["nreq"]))
        it = sum(_ITERS["bicgstab"].values()) / 4.0
    else:
        n = case.get("ncols", 1)
        it = _ITERS[case["solver"] if kind == "solve" else "gcr"][case["M"]]
    if kind == "sap":  # an operator (FP64), about 20 block operators (FP32) and 12 vector sweeps an iteration
        b1, f1 = _operator_work(V, 1, 8)
        b2, f2 = _operator_work(V, 1, 4)
        return {"bytes": it * (b1 + 10 * b2 + 12 * V * 192.0), "flops": it * (f1 + 25 * f2)}
    # two operators an iteration, and the iteration's vectors (half a lattice each) once
    b, f = _operator_work(V, n, real)
    return {"bytes": it * (2 * b + 9 * V / 2 * n * 24.0 * real) + 2 * V * n * 192.0, "flops": it * 2 * f}


# ------------------------------------------------- the same in plain torch

def _gamma():
    s = [np.array([[0, 1], [1, 0]]), np.array([[0, -1j], [1j, 0]]), np.array([[1, 0], [0, -1]])]
    z = np.zeros((2, 2))
    return [np.block([[z, -np.eye(2)], [-np.eye(2), z]]).astype(complex)] + \
           [np.block([[z, -1j * q], [1j * q, z]]) for q in s]


class _Dirac:
    """D + M in complex128 on spinors [n, 4, 3, T, L1, L2, L3]; M a number or one
    per column; antiperiodic in time."""

    def __init__(self, U, csw, M):
        self.dims = tuple(U.shape[:4])
        self.U = U.permute(4, 5, 6, 0, 1, 2, 3).contiguous()
        self.M = M
        self.C = self._clover(csw) if csw else None

    def _shift(self, a, mu, step, bc=1.0):
        """a(x + step mu) on the last four axes, times bc across the time wrap."""
        k = a.ndim - 4 + mu
        r = torch.roll(a, -step, dims=k)
        if bc != 1.0 and mu == 0:
            r.select(k, a.shape[k] - 1 if step > 0 else 0).mul_(bc)
        return r

    def _clover(self, csw):
        g = _gamma()
        C = torch.zeros((12, 12) + self.dims, dtype=torch.complex128, device=self.U.device)

        def dg(a):
            return a.transpose(0, 1).conj()

        for mu in range(4):
            for nu in range(mu + 1, 4):
                sh = self._shift
                A, B = self.U[mu], self.U[nu]
                Am, Bm = sh(A, mu, -1), sh(B, nu, -1)                    # at x - mu, x - nu
                Q = _mm(_mm(A, sh(B, mu, 1)), _mm(dg(sh(A, nu, 1)), dg(B)))
                Q += _mm(_mm(B, dg(sh(Am, nu, 1))), _mm(dg(sh(B, mu, -1)), Am))
                Bmm = sh(Bm, mu, -1)                                      # U_nu(x - mu - nu)
                Q += _mm(_mm(dg(Am), dg(Bmm)), _mm(sh(Am, nu, -1), Bm))
                Q += _mm(_mm(dg(Bm), sh(A, nu, -1)), _mm(sh(Bm, mu, 1), dg(A)))
                F = (Q - dg(Q)) / 8.0
                sig = 0.5j * (g[mu] @ g[nu] - g[nu] @ g[mu])
                for s in range(4):
                    for t in range(4):
                        if abs(sig[s, t]) > 0:
                            C[3 * s:3 * s + 3, 3 * t:3 * t + 3] += complex(0.5j * csw * sig[s, t]) * F
        return C

    def diag(self, x):
        m = torch.as_tensor(self.M, dtype=torch.float64, device=x.device).reshape(-1, 1, 1, 1, 1, 1, 1)
        y = (4.0 + m) * x
        if self.C is not None:
            n = x.shape[0]
            xv, yv = x.reshape((n, 12) + self.dims), y.view((n, 12) + self.dims)
            for a in range(12):
                for b in range(6 * (a // 6), 6 * (a // 6) + 6):
                    yv[:, a].addcmul_(self.C[a, b].expand_as(xv[:, b]), xv[:, b])
        return y

    def hop(self, x, sign=1.0):
        """sign = -1: the gammas with the other sign (gamma5 hop gamma5)."""
        g = _gamma()
        out = torch.zeros_like(x)
        for mu in range(4):
            for fwd in (True, False):
                sg = (1.0 if fwd else -1.0) * sign
                # (1 - sg gamma_mu): the lower spins follow from the upper ones
                G = -sg * g[mu]
                y = self._shift(x, mu, 1 if fwd else -1, -1.0)
                h = torch.empty_like(y[:, :2])
                for s in range(2):
                    t = 2 + int(np.nonzero(G[s, 2:])[0][0])
                    h[:, s] = y[:, s] + complex(G[s, t]) * y[:, t]
                V = self.U[mu] if fwd else self._shift(self.U[mu], mu, -1).transpose(0, 1).conj().resolve_conj()
                w = torch.zeros_like(h)
                for a in range(3):
                    for b in range(3):
                        w[:, :, a].addcmul_(V[a, b].expand_as(h[:, :, b]), h[:, :, b])
                out[:, :2] -= 0.5 * w
                for s in range(2, 4):
                    t = int(np.nonzero(G[s, :2])[0][0])
                    out[:, s] -= (0.5 * complex(G[s, t])) * w[:, t]
        return out

    def __call__(self, x):
        return self.diag(x) + self.hop(x)


def _to_grid(x, d):
    return x.reshape((x.shape[0],) + d + (4, 3)).permute(0, 5, 6, 1, 2, 3, 4).contiguous()


def _from_grid(x):
    return x.permute(0, 3, 4, 5, 6, 1, 2).reshape(x.shape[0], -1)


def _bicgstab(A, b, tol, cap):
    """One BiCGStab solve from zero, per column, until every column met tol."""
    def dot(p, q):
        return (p.reshape(p.shape[0], -1).conj() * q.reshape(q.shape[0], -1)).sum(1)

    def col(c):
        return c.reshape((-1,) + (1,) * (b.ndim - 1))

    def quot(p, q):
        return torch.where(q.abs() > 0, p / torch.where(q.abs() > 0, q, torch.ones_like(q)), torch.zeros_like(q))

    x = torch.zeros_like(b)
    r, rh, p = b.clone(), b.clone(), b.clone()
    goal = tol * dot(b, b).real.sqrt()
    rho = dot(rh, r)
    for _ in range(cap):
        v = A(p)
        al = quot(rho, dot(rh, v))
        s = r - col(al) * v
        t = A(s)
        om = quot(dot(t, s), dot(t, t))
        x += col(al) * p + col(om) * s
        r = s - col(om) * t
        if bool((dot(r, r).real.sqrt() <= goal).all()):
            break
        new = dot(rh, r)
        p = r + col(quot(new, rho) * quot(al, om)) * (p - col(om) * v)
        rho = new
    return x


def _solve(A, b):
    """A x = b to the rounding of 64 bits: BiCGStab restarted on the true residual."""
    x = torch.zeros_like(b)
    r = b
    for _ in range(4):
        x = x + _bicgstab(A, r, 1e-6, 600)
        r = b - A(x)
        if float(r.abs().max() / b.abs().max()) < 1e-15:
            break
    return x


def _point(d, site, n):
    eta = torch.zeros((n,) + d + (12,), dtype=torch.complex128, device=_device())
    for c in range(n):
        eta[(c,) + site + (c,)] = 1.0
    return eta.reshape(n, -1)


def _cpp(S, d, x0):
    """-sum |S|^2 per timeslice from the source, one row a column ([n, V*12] in)."""
    c = -(S.abs() ** 2).reshape(S.shape[0], d[0], -1).sum(2)
    return torch.roll(c, -x0, dims=1)


def exact(case, seed):
    kind, d = case["kind"], _dims(case)
    U = _links(d, case["eps"], seed)
    if kind in ("apply", "newconf"):
        D = _Dirac(U, case["csw"], case["M"])
        al = torch.as_tensor(_profile(case["profile"], d[0], case["alpha0"], 0), device=U.device)
        al = al.reshape(1, 1, 1, -1, 1, 1, 1)
        g5 = torch.tensor([1.0, 1.0, -1.0, -1.0], dtype=torch.float64, device=U.device).reshape(1, 4, 1, 1, 1, 1, 1)
        x = _to_grid(_spinors(d, case["nrhs"], seed), d)

        def hop(v):  # alpha H alpha^-1, or its adjoint gamma5 (1/alpha H alpha) gamma5
            return g5 * D.hop(g5 * (v * al)) / al if case["dagger"] else D.hop(v / al) * al

        if case["op"] == "hop":
            return _from_grid(hop(x))
        if case["op"] == "full":
            return _from_grid(D.diag(x) + hop(x))
        par = sum(torch.arange(n, device=U.device).reshape([-1 if k == mu else 1 for k in range(4)])
                  for mu, n in enumerate(d)) % 2
        xe = x * (par == 0)
        h = (hop(xe) * (par == 1)).reshape(x.shape[0], 12, -1).permute(2, 1, 0).cpu().numpy()
        A = (4.0 + case["M"]) * np.eye(12)
        if D.C is not None:
            A = A + D.C.reshape(12, 12, -1).permute(2, 0, 1).cpu().numpy()
        t = np.linalg.solve(np.broadcast_to(A, (h.shape[0], 12, 12)), h)
        t = torch.as_tensor(t, device=U.device).permute(2, 1, 0).reshape(x.shape).contiguous()
        return _from_grid((D.diag(xe) - hop(t)) * (par == 0))
    if kind == "serve":
        reqs = _requests(case, seed)
        M = [q["M"] for q in reqs for _ in range(q["ncols"])]
        eta = torch.cat([_point(d, (q["x0"], 0, 0, 0), q["ncols"]) for q in reqs])
        S = _from_grid(_solve(_Dirac(U, case["csw"], M), _to_grid(eta, d)))
        out, at = [], 0
        for q in reqs:
            out.append(_cpp(S[at:at + q["ncols"]], d, q["x0"]).sum(0))
            at += q["ncols"]
        return torch.stack(out).cpu().numpy()
    site = _site(case, seed)
    if kind == "sap":
        site = (0,) + site[1:]
    n = case.get("ncols", 1)
    S = _from_grid(_solve(_Dirac(U, case["csw"], case["M"]), _to_grid(_point(d, site, n), d)))
    cpp = _cpp(S, d, site[0]).sum(0).cpu().numpy()
    return {"S": S, "cpp": cpp[None] if kind == "solve" else cpp}
