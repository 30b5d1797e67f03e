"""The Gram-Schmidt passes of FGMRES at the edges of their kernels' ranges of
basis vectors (8, 16, 24, 32, 64, 128): one cycle of J steps, its residual
against the oracle's FGMRES after J steps.  Both minimise over the same Krylov
space from bases orthogonal to rounding, so the residuals agree to eps times
the condition of the projected problem (bounded by 1e9 here: 1e-6 of the
residual), down to the 1e-12 of |b| that rounding leaves in b - K x.  A batch
takes the same sums as its right-hand sides one at a time: equal bits."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2311_06926_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda", 0)


@pytest.mark.parametrize("E,p,J", [(1, 2, 2), (2, 2, 5)] + [
    (5, 3, J) for J in (1, 4, 8, 9, 16, 17, 24, 25, 32, 33, 64, 65, 100, 128)])
def test_cycle_of_j_steps(dev, E, p, J):
    from oracle.assemble import KronSystem
    from oracle.krylov import fgmres
    from oracle.precond import HyperPower
    from paper_2311_06926_amd.solver import Solver
    print(f"[gs] E={E} p={p} J={J}", file=sys.stderr, flush=True)
    S = KronSystem(E, p, 1.0)
    H = HyperPower(S, 2, 0)
    opts = dict(autotune=False, iters=0, krylov="fgmres", restart=128, maxit=J)
    sol = Solver(E, p, 1.0, max_rhs=3, **opts)
    one = Solver(E, p, 1.0, max_rhs=1, **opts)
    # right-hand sides in the range of K (the pressure is fixed up to a constant)
    b = np.concatenate([S.K @ synth.random_vector(S.N, seed=J + r) for r in range(3)])
    x, _ = sol.solve(torch.from_numpy(b).to(dev), tol=1e-30, raise_on_noconv=False)
    x = x.cpu().numpy()
    for r in range(3):
        seg = slice(r * S.N, (r + 1) * S.N)
        x1, _ = one.solve(torch.from_numpy(b[seg].copy()).to(dev), tol=1e-30,
                          raise_on_noconv=False)
        assert np.array_equal(x1.cpu().numpy(), x[seg])
        ref = fgmres(lambda v: S.K @ v, lambda v, j: H.apply(v), b[seg], tol=1e-30, restart=128,
                     maxit=J)
        nb = np.linalg.norm(b[seg])
        got, want = (np.linalg.norm(b[seg] - S.K @ v) / nb for v in (x[seg], ref.x))
        assert abs(got - want) <= 1e-6 * want + 1e-12
    sol.close()
    one.close()
