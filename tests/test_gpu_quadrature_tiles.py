"""The quadrature-based operator at the edges of its tiles: meshes of one
element, of one tile with both end points, and just below, at and above the
tile sizes in the plane (4x5, 4x3, 3x2, 2x2, 2x1 elements by degree), and more
right-hand sides than one launch takes.  Against the oracle's K with the
operators' tolerance (1e-12 of the largest entry: the same products summed in
another order)."""
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


@pytest.mark.parametrize("E,p,nrhs", [(1, 2, 1), (4, 2, 1), (5, 2, 1), (6, 2, 1), (11, 2, 9),
                                      (1, 3, 1), (3, 3, 1), (4, 3, 2), (7, 3, 1), (10, 3, 1),
                                      (1, 4, 1), (2, 4, 1), (3, 4, 1), (7, 4, 1), (1, 5, 1),
                                      (3, 5, 2), (4, 5, 1), (1, 6, 1), (5, 6, 1), (1, 7, 1),
                                      (3, 7, 1), (1, 8, 1), (4, 8, 2)])
def test_quadrature_tiles(dev, E, p, nrhs):
    from oracle.assemble import KronSystem
    from paper_2311_06926_amd.solver import Solver
    nu = 1.3
    print(f"[quad] E={E} p={p} nrhs={nrhs}", file=sys.stderr, flush=True)
    c_pen = 60.0 if p >= 7 else None   # the default is too small on these few elements
    sol = Solver(E, p, nu, autotune=False, max_rhs=nrhs, c_pen=c_pen or 0.0)
    S = KronSystem(E, p, nu, c_pen=c_pen)
    x = synth.random_vector(nrhs * S.N, seed=E + 10 * p)
    y = sol.apply_K_quad(torch.from_numpy(x).to(dev)).cpu().numpy()
    for r in range(nrhs):
        seg = slice(r * S.N, (r + 1) * S.N)
        ref = S.K @ x[seg]
        assert np.abs(y[seg] - ref).max() <= 1e-12 * np.abs(ref).max()
    sol.close()
