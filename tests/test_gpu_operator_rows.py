"""The operators' tiles are staged in pairs of neighbours, which straddle the
ends of rows of odd length: an infinity or a NaN at the first or last point of
a row may reach the outputs that its column of K couples to and no others.
Against K's sparsity pattern; the other outputs equal, bit for bit, those
without the poison."""
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


@pytest.mark.parametrize("E,p,opts", [(6, 2, {}), (16, 2, {}), (17, 2, {"op_pres_wide": 1}),
                                      (13, 3, {}), (14, 3, {"op_pres_wide": 1}), (12, 4, {}),
                                      (7, 5, {}), (8, 6, {})])
def test_rows_do_not_leak(dev, E, p, opts):
    from oracle.assemble import KronSystem
    from paper_2311_06926_amd.solver import Solver
    print(f"[rows] E={E} p={p} {opts}", file=sys.stderr, flush=True)
    sol = Solver(E, p, 1.0, autotune=False, op_staged=0, op_kchunk=5, **opts)
    K = KronSystem(E, p, 1.0).K.tocsc()
    x = synth.random_vector(sol.N, seed=E + p)
    y = sol.apply_K(torch.from_numpy(x).to(dev)).cpu().numpy()
    for b, (n1, n2, n3) in enumerate(sol.dims):
        for i, j, k, v in [(0, n2 // 2, n3 // 2, np.inf), (n1 - 1, n2 // 2, n3 // 2, np.nan),
                           (0, 0, 1, np.nan), (n1 - 1, n2 - 1, n3 - 2, np.inf)]:
            c = sol.offsets[b] + i + n1 * (j + n2 * k)
            z = x.copy()
            z[c] = v
            got = sol.apply_K(torch.from_numpy(z).to(dev)).cpu().numpy()
            touched = np.zeros(sol.N, bool)
            touched[K.indices[K.indptr[c]:K.indptr[c + 1]]] = True
            assert np.array_equal(got[~touched], y[~touched]), (b, i, j, k)
            # (K has no pressure diagonal: some coupled output, not entry c itself)
            assert not np.isfinite(got[touched]).all()
    sol.close()
