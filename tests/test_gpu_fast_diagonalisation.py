"""P_0 by parity-split fast diagonalisation where its tiles can go wrong: half
lengths just below, at and above a multiple of 16 (and of the tile counts at
which the kernels change), the smallest meshes and the longest passes.

Checked in backward form on the GPU with dense univariate matrices of the
oracle: |A_cc y - x| <= 1e-14 (|A_cc| |y| + |x|), the bound the other P_0
tests use (each of the six contractions and the scaling is backward stable
to a few ulps), FP32 products within 1e-5 and split BF16 within 2e-4 of FP64.
"""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda", 0)


def kron(a3, a2, a1, x):
    """(a3 (x) a2 (x) a1) x for x of shape (n3, n2, n1)."""
    n3, n2, n1 = x.shape
    x = torch.matmul(x.reshape(-1, n1), a1.t().contiguous()).reshape(n3, n2 * n1)
    x = torch.matmul(a3, x).reshape(n3, n2, n1).transpose(0, 1).reshape(n2, n3 * n1)
    return torch.matmul(a2, x).reshape(n2, n3, n1).transpose(0, 1)


def backward_errors(E, p, nu, x, y, dev):
    """Normwise backward errors of y = P_0^{-1} x, one per block."""
    from oracle.assemble import default_c_pen
    from oracle.matrices1d import Matrices1D
    m = Matrices1D(E, p, default_c_pen(p))
    Mc, Tc, M, K = (torch.from_numpy(np.ascontiguousarray(a)).to(dev)
                    for a in (m.Mc, m.Tc, m.M_int, m.K_int))
    nN, nM = m.nN, m.nM
    norm = {id(a): float(a.abs().sum(1).max()) for a in (Mc, Tc, M, K)}
    out, at = [], 0
    for c in range(4):
        shape = tuple(nN if d == c else nM for d in (2, 1, 0))
        n = shape[0] * shape[1] * shape[2]
        xb, yb = x[at:at + n].reshape(shape), y[at:at + n].reshape(shape)
        at += n
        r, a = -xb, 0.0
        if c == 3:
            terms = [(Mc, Mc, Mc, 1.0 / (2 * nu))]
        else:
            terms = [tuple((K if d == e else M) if d == c else (Tc if d == e else Mc)
                           for d in (2, 1, 0)) + (2 * nu,) for e in range(3)]
        for a3, a2, a1, s in terms:
            r = r + s * kron(a3, a2, a1, yb)
            a += s * norm[id(a3)] * norm[id(a2)] * norm[id(a1)]
        out.append(float(r.abs().max() / (a * yb.abs().max() + xb.abs().max())))
    return out


# E, p: E + p - 1 = 2, 16, 17, 33, 34, 49, 64, 65, 97, 128 per direction (all plans)
@pytest.mark.parametrize("E,p", [(1, 2), (14, 3), (15, 3), (31, 3), (33, 2), (48, 2), (62, 3),
                                 (63, 3), (95, 3), (126, 3)])
def test_every_plan_at_tile_edges(dev, E, p):
    from paper_2311_06926_amd.solver import Solver
    nu, R = 0.8, 2
    say(f"[fd] E={E} p={p}")
    x, ref = None, {}
    for plan in (0, 1, 8, 9):
        s = Solver(E, p, nu, autotune=False, fd_plan=plan, max_rhs=R)
        assert s.tuning(1)["fd_plan"][0] == plan
        if x is None:
            x = torch.randn(R * s.N, dtype=torch.float64, device=dev,
                            generator=torch.Generator(device=dev).manual_seed(E))
        y = s.apply_P0(x)
        for r in range(R):
            seg = slice(r * s.N, (r + 1) * s.N)
            eta = backward_errors(E, p, nu, x[seg], y[seg], dev)
            say(f"[fd]   plan {plan} rhs {r}: backward errors {['%.1e' % e for e in eta]}")
            assert max(eta) <= 1e-14
            assert torch.equal(s.apply_P0(x[seg].clone()), y[seg])
        # the plane plans agree bit for bit, and so do the direction passes
        assert torch.equal(ref.setdefault(plan % 2, y), y)
        s.close()
        for prec, tol in (("fp32", 1e-5), ("bf16x3", 2e-4)):
            s = Solver(E, p, nu, autotune=False, fd_plan=plan, precision=prec, krylov="fgmres",
                       max_rhs=R)
            gap = float((s.apply_P0(x) - y).abs().max() / y.abs().max())
            assert gap < tol, (plan, prec, gap)
            s.close()


# 129, 257, 321 (a tile staged in two batches) and 513 (16 waves) per direction
@pytest.mark.parametrize("E,p", [(127, 3), (256, 2), (320, 2), (512, 2)])
def test_direction_passes_beyond_a_plane(dev, E, p):
    from paper_2311_06926_amd.solver import Solver
    nu = 1.2
    say(f"[fd] E={E} p={p}")
    s = Solver(E, p, nu, autotune=False)
    assert s.tuning(1)["fd_plan"][0] == 8
    x = torch.randn(s.N, dtype=torch.float64, device=dev,
                    generator=torch.Generator(device=dev).manual_seed(E))
    y = s.apply_P0(x)
    s.close()
    eta = backward_errors(E, p, nu, x, y, dev)
    say(f"[fd]   backward errors {['%.1e' % e for e in eta]}")
    assert max(eta) <= 1e-14
    if E == 256:
        s = Solver(E, p, nu, autotune=False, precision="fp32", krylov="fgmres")
        assert float((s.apply_P0(x) - y).abs().max() / y.abs().max()) < 1e-5
        s.close()


def test_solve_with_direction_passes(dev):
    """MINRES (its dot partials from k_fd_dot_vel and the mode-3 launch) with the
    direction passes against the plane kernels: P_0 differs by rounding only, so
    the iteration counts are equal and the solutions agree to 1e-10."""
    from paper_2311_06926_amd.solver import Solver
    E, p = 20, 3
    a = Solver(E, p, 1.0, autotune=False, fd_plan=1, max_rhs=2)
    b = Solver(E, p, 1.0, autotune=False, fd_plan=0, max_rhs=2)
    rhs = a.build_rhs([1.0, -0.6])
    xa, ia = a.solve(rhs, 1e-9)
    xb, ib = b.solve(rhs, 1e-9)
    assert ia.iterations == ib.iterations and ib.converged == 1
    assert float((xa - xb).abs().max() / xa.abs().max()) <= 1e-10
    a.close()
    b.close()


@pytest.mark.parametrize("E,p,krylov", [(6, 3, "minres"), (17, 2, "minres"), (31, 4, "minres"),
                                        (40, 3, "minres"), (100, 2, "minres"), (9, 3, "fgmres")])
def test_solve_does_not_depend_on_the_plane_plan(dev, E, p, krylov):
    """The two plane plans (tiles of 32 and of 16 columns in mode 3) give the
    same bits, and so do the dots that their launches leave for MINRES: equal
    solutions and counts, whichever the tuner takes."""
    from paper_2311_06926_amd.solver import Solver
    out = []
    for plan in (1, 9):
        s = Solver(E, p, 1.0, iters=1, krylov=krylov, max_rhs=2, fd_plan=plan, autotune=False)
        x, info = s.solve(s.build_rhs([1.0, 0.7]), 1e-8)
        out.append((x, list(info.iters_per_rhs[:2])))
        s.close()
    assert out[0][1] == out[1][1]
    assert torch.equal(out[0][0], out[1][0])
