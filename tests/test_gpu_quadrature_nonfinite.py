"""An infinity or a NaN in one coefficient reaches, through the quadrature
operator, the outputs whose functions share an element with its own and no
others, although a tile's transposed sums run over all its points.  The other
outputs equal, bit for bit, those without the poison."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2311_06926_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu


def elements(i, E, p, interior):
    """First and last element of the support of function i: degree p - 1, or
    the interior functions of degree p."""
    return (max(i + 1 - p, 0), min(i + 1, E - 1)) if interior else (max(i + 1 - p, 0), min(i, E - 1))


def overlap(n_out, interior_out, support, E, p):
    lo, hi = support
    out = np.zeros(n_out, bool)
    for i in range(n_out):
        a, b = elements(i, E, p, interior_out)
        out[i] = a <= hi and lo <= b
    return out


@pytest.mark.parametrize("E,p", [(9, 2), (13, 3), (9, 4), (7, 5), (7, 6), (5, 7), (5, 8)])
def test_poison_stays_in_its_elements(E, p):
    from paper_2311_06926_amd.solver import Solver
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[quad nonfinite] E={E} p={p}", file=sys.stderr, flush=True)
    sol = Solver(E, p, 1.0, autotune=False, max_rhs=2, c_pen=60.0)
    x = synth.random_vector(2 * sol.N, seed=E + p)
    y = sol.apply_K_quad(torch.from_numpy(x).cuda()).cpu().numpy()
    for b, n in enumerate(sol.dims):
        for at, v in [((0, 0, 0), np.nan), (tuple(m // 2 for m in n), np.inf),
                      ((n[0] - 1, n[1] // 2, n[2] - 1), -np.inf)]:
            z = x.copy()
            z[sol.offsets[b] + at[0] + n[0] * (at[1] + n[1] * at[2])] = v
            got = sol.apply_K_quad(torch.from_numpy(z).cuda()).cpu().numpy()
            sup = [elements(at[d], E, p, d == b) for d in range(3)]
            clean = np.ones(2 * sol.N, bool)
            for o, m in enumerate(sol.dims):
                t = [overlap(m[d], d == o, sup[d], E, p) for d in range(3)]
                hit = t[2][:, None, None] & t[1][None, :, None] & t[0][None, None, :]
                clean[sol.offsets[o]:sol.offsets[o + 1]] = ~hit.ravel()
            assert clean[:sol.N].any() or E <= p
            assert np.array_equal(got[clean], y[clean]), (b, at)
            assert not np.isfinite(got[~clean]).all()
    sol.close()
