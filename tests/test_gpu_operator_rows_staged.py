"""As test_gpu_operator_rows.py, for the kernels that take all planes of a chunk
at once (their loads come in pairs too) and for the degrees that file leaves out:
an infinity or a NaN at the first or last point of a row reaches the outputs that
its column of K couples to and no others; the other outputs equal, bit for bit,
those without the poison.  K, A, B and B'."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2311_06926_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,p,opts", [(6, 2, {"op_staged": 1, "op_kchunk": 2}),
                                      (16, 2, {"op_staged": 1, "op_kchunk": 4}),
                                      (17, 2, {"op_staged": 1, "op_kchunk": 2}),
                                      (13, 3, {"op_staged": 1, "op_kchunk": 4}),
                                      (14, 3, {"op_staged": 1, "op_kchunk": 2}),
                                      (15, 3, {"op_staged": 1, "op_kchunk": 8}),
                                      (12, 4, {"op_staged": 1, "op_kchunk": 2}),
                                      (13, 4, {"op_staged": 1, "op_kchunk": 4}),
                                      (6, 7, {"op_staged": 0, "op_kchunk": 3}),
                                      (7, 8, {"op_staged": 0, "op_kchunk": 5})])
def test_rows_do_not_leak(E, p, opts):
    from oracle.assemble import KronSystem
    from paper_2311_06926_amd.solver import Solver
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[rows] E={E} p={p} {opts}", file=sys.stderr, flush=True)
    c_pen = 60.0 if p >= 7 else None
    sol = Solver(E, p, 1.0, autotune=False, c_pen=c_pen or 0.0, **opts)
    assert sol.tuning(1)["op_staged"] == opts["op_staged"]
    K = KronSystem(E, p, 1.0, c_pen=c_pen).K.tocsr()
    nV = sol.nV
    x = synth.random_vector(sol.N, seed=E + p)

    def dev(v):
        return torch.from_numpy(np.ascontiguousarray(v)).cuda()

    ops = [(sol.apply_K, K, slice(0, sol.N)), (sol.apply_A, K[:nV, :nV], slice(0, nV)),
           (sol.apply_B, K[:nV, nV:], slice(nV, sol.N)), (sol.apply_Bt, K[nV:, :nV], slice(0, nV))]
    for f, M, cols in ops:
        M = M.tocsc()
        y = f(dev(x[cols])).cpu().numpy()
        for b, (n1, n2, n3) in enumerate(sol.dims):
            if not cols.start <= sol.offsets[b] < cols.stop:
                continue
            for i, j, k, v in [(0, n2 // 2, n3 // 2, np.inf), (n1 - 1, n2 // 2, n3 // 2, np.nan),
                               (0, 0, 1, np.nan), (n1 - 1, n2 - 1, n3 - 2, np.inf)]:
                c = sol.offsets[b] - cols.start + i + n1 * (j + n2 * k)
                z = x[cols].copy()
                z[c] = v
                got = f(dev(z)).cpu().numpy()
                touched = np.zeros(len(y), bool)
                touched[M.indices[M.indptr[c]:M.indptr[c + 1]]] = True
                assert np.array_equal(got[~touched], y[~touched]), (f.__name__, b, i, j, k)
                assert not np.isfinite(got[touched]).all()
    sol.close()
