"""What a user has this solver do, as cases that can be timed and checked.

``listed()`` names twelve calls of the public front end (``Solver`` and
``autograd``): single operator applications from the smallest mesh to one
whose vectors exceed the Infinity Cache, the preconditioners, and whole
solves (MINRES, batched FGMRES, a differentiable training step).  ``draw``
gives further ones of the same kinds over their ranges of mesh, degree, batch
and options.  A pass is ``run(prepare(case, seed))``; ``exact`` is the same
result from dense univariate matrices in 64 bits, written here independently
of the package.

Kinds ("op"):
  K, A, B, Bt, MV   one operator application (nrhs vectors)
  Kquad             the quadrature-based forward operator
  P0, Pk, PV        base preconditioner, hyper-power preconditioner of order q
                    after k updates, its velocity block alone
  solve             one hp_solve (MINRES or FGMRES, nrhs right-hand sides)
  train             forward solve, loss and adjoint gradients (autograd)
"""
import math

import numpy as np
import torch

from paper_2311_06926_amd import synth
from paper_2311_06926_amd.autograd import cavity_loss
from paper_2311_06926_amd.solver import Solver

NU = 0.9


def listed():
    return [
        # the smallest mesh of the paper's Table 1: launch latency only
        {"name": "K_8_p2", "op": "K", "E": 8, "p": 2, "nrhs": 1},
        # an ordinary ragged mesh at a higher degree
        {"name": "K_45_p4", "op": "K", "E": 45, "p": 4, "nrhs": 1},
        # vectors of 233 MB: the operator on an HBM-sized mesh
        {"name": "K_192_p3", "op": "K", "E": 192, "p": 3, "nrhs": 1},
        # a batch of right-hand sides at Table 1's high degree
        {"name": "K_24_p6_x4", "op": "K", "E": 24, "p": 6, "nrhs": 4},
        # the base preconditioner at the benchmark's headline mesh
        {"name": "P0_32_p3", "op": "P0", "E": 32, "p": 3, "nrhs": 1},
        # one hyper-power update on an odd mesh, both blocks
        {"name": "Pk_61_p3", "op": "Pk", "E": 61, "p": 3, "nrhs": 1, "q": 2, "k": 1,
         "schur": "Pcq1"},
        # the operator study of Sec. 5.1: the velocity block on 256^3 elements
        {"name": "PV_256_p2", "op": "PV", "E": 256, "p": 2, "nrhs": 1, "q": 2, "k": 1},
        # the quadrature-based forward operator (the paper's T_f)
        {"name": "Kquad_32_p3", "op": "Kquad", "E": 32, "p": 3, "nrhs": 1},
        # the headline solve: cavity, MINRES to 1e-8, one update
        {"name": "minres_32_p3", "op": "solve", "E": 32, "p": 3, "nrhs": 1, "krylov": "minres",
         "precision": "fp64", "forward": "kronecker", "q": 2, "k": 1, "tol": 1e-8},
        # a small row of Table 1 with the paper's kind of forward operator
        {"name": "minres_quad_16_p4", "op": "solve", "E": 16, "p": 4, "nrhs": 1,
         "krylov": "minres", "precision": "fp64", "forward": "quadrature", "q": 2, "k": 1,
         "tol": 1e-8},
        # 32 body-force right-hand sides in one FGMRES, FP32 preconditioner
        {"name": "fgmres_48_p2_x32", "op": "solve", "E": 48, "p": 2, "nrhs": 32,
         "krylov": "fgmres", "precision": "fp32", "forward": "kronecker", "q": 2, "k": 1,
         "tol": 1e-8},
        # a training step: loss, forward and adjoint solve, gradients
        {"name": "train_64_p3", "op": "train", "E": 64, "p": 3, "nrhs": 1, "precision": "fp32",
         "q": 2, "k": 1, "tol": 1e-10},
    ]


def _sizes(E, p):
    nN, nM = E + p - 2, E + p - 1
    nV, nQ = 3 * nN * nM * nM, nM ** 3
    return nN, nM, nV, nQ, nV + nQ


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: the kind by how often programs call it, the mesh spread
    over the logarithm of its range, capped at the listed cases' cost."""
    op = rng.choice(["K", "K", "K", "A", "Bt", "B", "MV", "P0", "P0", "Pk", "Pk", "PV", "Kquad",
                     "Kquad", "solve", "solve", "solve", "train"])
    if op in ("K", "A", "B", "Bt", "MV"):
        p = rng.choice([2, 3, 3, 4, 5, 6, 8])
        E = _log_int(rng, 4, 180 if p <= 3 else 110 if p == 4 else 56)
        nrhs = rng.choice([1, 1, 1, 2, 3, 8])
        while _sizes(E, p)[4] * nrhs > 2.0e7:
            nrhs -= 1
        return {"op": op, "E": E, "p": p, "nrhs": max(nrhs, 1)}
    if op == "P0":
        p = rng.choice([2, 3, 3, 4, 5])
        return {"op": op, "E": _log_int(rng, 5, 170), "p": p, "nrhs": 1}
    if op == "Pk":
        p, k = rng.choice([2, 3, 3, 4]), rng.choice([0, 1, 1, 2])
        q = rng.choice([2, 2, 3]) if k else 2
        return {"op": op, "E": _log_int(rng, 6, 120 if k < 2 else 72), "p": p, "nrhs": 1, "q": q,
                "k": k, "schur": rng.choice(["Pcq1", "Pcq1", "Pcq2"])}
    if op == "PV":
        k = rng.choice([0, 1, 2])
        return {"op": op, "E": _log_int(rng, 24, 230 if k < 2 else 150), "p": rng.choice([2, 3]),
                "nrhs": 1, "q": 2, "k": k}
    if op == "Kquad":
        p = rng.choice([2, 3, 3, 4, 5, 6])
        return {"op": op, "E": _log_int(rng, 5, 240 // (p + 1)), "p": p, "nrhs": 1}
    if op == "train":
        return {"op": op, "E": _log_int(rng, 10, 60), "p": rng.choice([2, 3]), "nrhs": 1,
                "precision": rng.choice(["fp32", "fp64"]), "q": 2, "k": 1, "tol": 1e-10}
    krylov = rng.choice(["minres", "minres", "fgmres"])
    if krylov == "minres":
        p = rng.choice([2, 3, 3, 4, 6])
        forward = rng.choice(["kronecker", "kronecker", "kronecker", "quadrature"])
        E = _log_int(rng, 6, 64 if forward == "kronecker" else 128 // (p + 1))
        return {"op": "solve", "E": E, "p": p, "nrhs": 1, "krylov": krylov, "precision": "fp64",
                "forward": forward, "q": 2, "k": rng.choice([0, 1, 1, 2]), "tol": 1e-8}
    p, E = rng.choice([2, 3]), _log_int(rng, 10, 44)
    return {"op": "solve", "E": E, "p": p, "nrhs": rng.choice([1, 2, 5, 12, 24]),
            "krylov": krylov, "precision": rng.choice(["fp32", "fp64"]), "forward": "kronecker",
            "q": 2, "k": 1, "tol": 1e-8}


def _vector(n, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(n, dtype=torch.float64, device="cuda", generator=g)


def _length(case):
    _, _, nV, nQ, N = _sizes(case["E"], case["p"])
    op = case["op"]
    n_in = nV if op in ("A", "Bt", "MV", "PV") else nQ if op == "B" else N
    n_out = nV if op in ("A", "B", "MV", "PV") else nQ if op == "Bt" else N
    return n_in * case["nrhs"], n_out * case["nrhs"]


def prepare(case, seed):
    op, E, p, nrhs = case["op"], case["E"], case["p"], case["nrhs"]
    if op == "solve":
        s = Solver(E, p, NU, krylov=case["krylov"], precision=case["precision"],
                   forward=case["forward"], order=case["q"], iters=case["k"], max_rhs=nrhs)
        # cavity lid speeds and 16 body-force modes per component and right-hand side
        draws = [synth.body_force_modes(1000 * seed + r) for r in range(nrhs)]
        amp, wav = zip(*(synth.modes_to_arrays(m) for m, _ in draws))
        b = s.build_rhs([u for _, u in draws], modes=(np.stack(amp), np.stack(wav)))
        return {"case": case, "solver": s, "b": b, "x": s.empty(s.N, nrhs)}
    if op == "train":
        s = Solver(E, p, NU, krylov="fgmres", precision=case["precision"], order=case["q"],
                   iters=case["k"])
        # the target: the cavity flow at another lid speed, with a perturbation
        target, _ = s.solve(s.build_rhs([1.5]), case["tol"])
        target = target[:s.nV] * (1.0 + 0.05 * torch.tanh(_vector(s.nV, 2 * seed)))
        return {"case": case, "solver": s, "target": target,
                "beta": 0.3 * _vector(s.nV, 2 * seed + 1),
                "nu": torch.tensor(NU, dtype=torch.float64, device="cuda")}
    s = Solver(E, p, NU, max_rhs=nrhs, schur=case.get("schur", "Pcq1"))
    n_in, n_out = _length(case)
    return {"case": case, "solver": s, "x": _vector(n_in, seed), "y": s.empty(n_out)}


def run(state):
    case, s = state["case"], state["solver"]
    op = case["op"]
    if op == "solve":
        x, _ = s.solve(state["b"], case["tol"], x=state["x"])
        return x
    if op == "train":
        beta = state["beta"].requires_grad_(True)
        nu = state["nu"].requires_grad_(True)
        loss = cavity_loss(beta, nu, s, state["target"], tol=case["tol"])
        g_beta, g_nu = torch.autograd.grad(loss, (beta, nu))
        return {"loss": loss.detach(), "beta": g_beta, "nu": g_nu}
    x, y = state["x"], state["y"]
    if op == "Pk":
        return s.apply_hyperpower(case["q"], case["k"], x, y)
    if op == "PV":
        return s.apply_PV(case["q"], case["k"], x, y)
    return {"K": s.apply_K, "A": s.apply_A, "B": s.apply_B, "Bt": s.apply_Bt, "MV": s.apply_MV,
            "Kquad": s.apply_K_quad, "P0": s.apply_P0}[op](x, y)


# ---- work ------------------------------------------------------------------------------
def _flops(case):
    """Flops of one application per right-hand side: banded Kronecker factors
    for the operators; for fast diagonalisation the mode products of the
    univariate matrices split by parity (they are centrosymmetric on a uniform
    mesh), half of the dense ones."""
    E, p = case["E"], case["p"]
    nN, nM, nV, nQ, _ = _sizes(E, p)
    a = 2.0 * nV * 13 * (2 * p - 1) / 3.0 + 2.0 * nQ * 3 * (2 * p - 1)
    bt = 2.0 * nQ * 3 * (2 * p - 1) + 3.0 * nQ
    kk = a + bt
    pv0, pq0 = 2.0 * nV * (nN + 2 * nM), 3.0 * nQ * nM
    return {"K": kk, "A": a, "B": bt, "Bt": bt, "MV": 2.0 * nV * 3 * (2 * p - 1), "pv0": pv0,
            "pq0": pq0}


def _pk_flops(f, q, k, schur):
    def pv(level):
        n = q ** level
        return n * f["pv0"] + (n - 1) * f["A"]

    def pq(level):
        if level == 0:
            return f["pq0"]
        if schur == "Pcq2":
            n = q ** level
            return n * f["pq0"] + (n - 1) * (2 * f["B"] + f["pv0"])
        s = 2 * f["B"] + pv(0 if level == 1 else level)
        return q * pq(level - 1) + (q - 1) * s

    return pv(k), pq(k)


def work(case):
    E, p, op, nrhs = case["E"], case["p"], case["op"], case["nrhs"]
    _, _, nV, nQ, N = _sizes(E, p)
    f = _flops(case)
    if op in ("solve", "train"):
        pv, pq = _pk_flops(f, case["q"], case["k"], "Pcq1")
        # iterations of the cavity (Table 1), and what an iteration reads and
        # writes of the Krylov vectors at least once
        its = {0: 57, 1: 30, 2: 20}[case["k"]] * (2.2 if op == "train" else 1)
        return {"bytes": its * nrhs * 8.0 * 8 * N, "flops": its * nrhs * (f["K"] + pv + pq)}
    n_in, n_out = _length(case)
    if op == "P0":
        fl = f["pv0"] + f["pq0"]
    elif op in ("Pk", "PV"):
        pv, pq = _pk_flops(f, case["q"], case["k"], case.get("schur", "Pcq1"))
        fl = pv + (pq if op == "Pk" else 0.0)
    elif op == "Kquad":
        # per point and field: sum factorisation of 13 values and 10 fluxes
        fl = 2.0 * (E * (p + 1)) ** 3 * 2 * 13 * (p + 1)
    else:
        fl = f[op]
    return {"bytes": 8.0 * (n_in + n_out), "flops": fl * nrhs}


# ---- the same in 64 bits, from dense univariate matrices ---------------------------------
def _splines(t, d, x):
    """Values and derivatives of the degree-d B-splines on knots t at x."""
    m = len(t) - 1
    last = max(i for i in range(m) if t[i + 1] > t[i])
    N = np.array([((x >= t[i]) & (x < t[i + 1])) | ((i == last) & (x == t[-1]))
                  for i in range(m)], dtype=np.float64)
    low = N
    for deg in range(1, d + 1):
        low = N
        N = np.zeros((m - deg, x.size))
        for i in range(m - deg):
            a, b = t[i + deg] - t[i], t[i + deg + 1] - t[i + 1]
            if a > 0:
                N[i] += (x - t[i]) / a * low[i]
            if b > 0:
                N[i] += (t[i + deg + 1] - x) / b * low[i + 1]
    dN = np.zeros_like(N)
    for i in range(N.shape[0]):
        a, b = t[i + d] - t[i], t[i + d + 1] - t[i + 1]
        if a > 0:
            dN[i] += d / a * low[i]
        if b > 0:
            dN[i] -= d / b * low[i + 1]
    return N, dN


class _Dense:
    """K, P_0 and P_k on tensors (n3, n2, n1) with dense univariate matrices."""

    def __init__(self, E, p):
        t = np.concatenate([np.zeros(p), np.arange(E + 1) / E, np.ones(p)])
        tm = t[1:-1]
        scale = (p / (tm[p:] - tm[:-p]))[:, None]  # unit integral
        g, w = np.polynomial.legendre.leggauss(p + 1)
        x = ((np.arange(E)[:, None] + 0.5 + 0.5 * g) / E).reshape(-1)
        W = np.tile(0.5 * w / E, E)
        N, dN = (v[1:-1] for v in _splines(t, p, x))
        M, dM = (v * scale for v in _splines(tm, p - 1, x))
        (m0, d0), (m1, d1) = (tuple(v[:, 0] * scale[:, 0] for v in _splines(tm, p - 1, e))
                              for e in (np.array([0.0]), np.array([1.0])))
        alpha = E * max(12.5, 2.5 * (p + 1))
        bc = np.outer(m1, d1) - np.outer(m0, d0)
        tc = 0.5 * ((dM * W) @ dM.T + 2 * alpha * (np.outer(m1, m1) + np.outer(m0, m0))
                    - bc - bc.T)
        dev = "cuda" if torch.cuda.is_available() else "cpu"

        def up(a):
            return torch.from_numpy(np.ascontiguousarray(a)).to(dev)

        mc, m, k = (M * W) @ M.T, (N * W) @ N.T, (dN * W) @ dN.T
        self.Mc, self.Tc, self.M, self.K = up(mc), up(tc), up(m), up(k)
        self.C, self.Cc = up((N * W) @ dM.T), up((dN * W) @ M.T)
        self.MiMc = up(np.linalg.inv(mc))
        self.eigK, self.eigT = self._eig(k, m, up), self._eig(tc, mc, up)
        nN, nM = E + p - 2, E + p - 1
        self.shapes = [(nM, nM, nN), (nM, nN, nM), (nN, nM, nM), (nM, nM, nM)]

    @staticmethod
    def _eig(a, b, up):
        li = np.linalg.inv(np.linalg.cholesky(b))
        c = li @ a @ li.T
        lam, q = np.linalg.eigh(0.5 * (c + c.T))
        return up(lam), up(li.T @ q)

    @staticmethod
    def _kron(a3, a2, a1, x):
        n3, n2, n1 = x.shape
        x = torch.matmul(x.reshape(-1, n1), a1.t().contiguous()).reshape(n3, n2, -1)
        m1 = x.shape[2]
        x = torch.matmul(a3, x.reshape(n3, -1)).reshape(-1, n2, m1)
        x = x.transpose(0, 1).reshape(n2, -1)
        return torch.matmul(a2, x).reshape(a2.shape[0], -1, m1).transpose(0, 1).contiguous()

    def split(self, v, first, last):
        out = []
        for s in self.shapes[first:last]:
            n = s[0] * s[1] * s[2]
            out.append(v[:n].reshape(s))
            v = v[n:]
        return out

    def A(self, u):
        kr, Mc, Tc, M, K, C = self._kron, self.Mc, self.Tc, self.M, self.K, self.C
        Ct = C.t().contiguous()
        u1, u2, u3 = u
        y1 = 2 * (kr(Mc, Mc, K, u1) + kr(Mc, Tc, M, u1) + kr(Tc, Mc, M, u1))
        y2 = 2 * (kr(Mc, M, Tc, u2) + kr(Mc, K, Mc, u2) + kr(Tc, M, Mc, u2))
        y3 = 2 * (kr(M, Mc, Tc, u3) + kr(M, Tc, Mc, u3) + kr(K, Mc, Mc, u3))
        y1 = y1 + kr(Mc, Ct, C, u2) + kr(Ct, Mc, C, u3)
        y2 = y2 + kr(Mc, C, Ct, u1) + kr(Ct, C, Mc, u3)
        y3 = y3 + kr(C, Mc, Ct, u1) + kr(C, Ct, Mc, u2)
        return [NU * y for y in (y1, y2, y3)]

    def B(self, q):
        kr, Mc, Cc = self._kron, self.Mc, self.Cc
        return [kr(Mc, Mc, Cc, q), kr(Mc, Cc, Mc, q), kr(Cc, Mc, Mc, q)]

    def Bt(self, u):
        kr, Mc, Ct = self._kron, self.Mc, self.Cc.t().contiguous()
        return kr(Mc, Mc, Ct, u[0]) + kr(Mc, Ct, Mc, u[1]) + kr(Ct, Mc, Mc, u[2])

    def MV(self, u):
        kr, Mc, M = self._kron, self.Mc, self.M
        return [kr(Mc, Mc, M, u[0]), kr(Mc, M, Mc, u[1]), kr(M, Mc, Mc, u[2])]

    def PV0(self, u):
        out = []
        for c, x in enumerate(u):
            (l1, q1), (l2, q2), (l3, q3) = (self.eigK if d == c else self.eigT for d in range(3))
            z = self._kron(q3.t().contiguous(), q2.t().contiguous(), q1.t().contiguous(), x)
            z = z / (2 * NU * (l3[:, None, None] + l2[None, :, None] + l1[None, None, :]))
            out.append(self._kron(q3, q2, q1, z))
        return out

    def PQ0(self, q):
        return 2 * NU * self._kron(self.MiMc, self.MiMc, self.MiMc, q)

    def PV(self, q, k, u):
        y = self.PV0(u)
        for _ in range(q ** k - 1):
            d = self.PV0([a - b for a, b in zip(u, self.A(y))])
            y = [a + b for a, b in zip(y, d)]
        return y

    def PQ(self, q, k, x, schur):
        if k == 0:
            return self.PQ0(x)
        if schur == "Pcq2":
            y = self.PQ0(x)
            for _ in range(q ** k - 1):
                y = y + self.PQ0(x - self.Bt(self.PV0(self.B(y))))
            return y
        s = x
        for _ in range(q - 1):
            t = self.PQ(q, k - 1, s, schur)
            s = x + s - self.Bt(self.PV(q, 0 if k == 1 else k, self.B(t)))
        return self.PQ(q, k - 1, s, schur)


def exact(case, seed):
    """The operators and preconditioners from dense univariate matrices; a
    Krylov solve is only good to its own tolerance and has no such value."""
    op, E, p, nrhs = case["op"], case["E"], case["p"], case["nrhs"]
    if op in ("solve", "train"):
        return None
    D = _Dense(E, p)
    n_in, _ = _length(case)
    x = _vector(n_in, seed).to(D.M.device)
    out = []
    for v in x.reshape(nrhs, -1):
        if op in ("A", "MV", "Bt", "PV"):
            u = D.split(v, 0, 3)
            y = (D.A(u) if op == "A" else D.MV(u) if op == "MV" else [D.Bt(u)] if op == "Bt"
                 else D.PV(case["q"], case["k"], u))
        elif op == "B":
            y = D.B(v.reshape(D.shapes[3]))
        else:
            *u, q = D.split(v, 0, 4)
            if op in ("K", "Kquad"):
                y = [a + b for a, b in zip(D.A(u), D.B(q))] + [D.Bt(u)]
            elif op == "P0":
                y = D.PV0(u) + [D.PQ0(q)]
            else:
                y = (D.PV(case["q"], case["k"], u)
                     + [D.PQ(case["q"], case["k"], q, case["schur"])])
        out += [t.reshape(-1) for t in y]
    return torch.cat(out)
