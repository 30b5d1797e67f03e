"""P_0 at the lengths whose odd half leaves 9 to 12 values in its last tile: the
plane kernel reads four steps of it there.  What lies past the half has to be
written by the workgroup itself, so a right-hand side of NaNs, in the batch or in
the call before, changes nothing in another one's result.

Backward errors as in test_gpu_fast_diagonalisation.py (the bound and its
derivation are given there); everything else bit for bit."""
import sys

import pytest

torch = pytest.importorskip("torch")

from test_gpu_fast_diagonalisation import backward_errors  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda", 0)


# E, p: E + p - 1 = 18, 19, 22, 25, 26, 53, 58, 85, 90, 117, 122 per direction
@pytest.mark.parametrize("E,p", [(17, 2), (16, 4), (20, 3), (23, 3), (25, 2), (51, 3), (57, 2),
                                 (83, 3), (88, 3), (115, 3), (120, 3)])
@pytest.mark.parametrize("plan", [1, 9])
def test_nan_stays_in_its_right_hand_side(dev, E, p, plan):
    from paper_2311_06926_amd.solver import Solver
    nu, R = 0.8, 3
    print(f"[tails] E={E} p={p} plan {plan}", file=sys.stderr, flush=True)
    s = Solver(E, p, nu, autotune=False, fd_plan=plan, max_rhs=R)
    N = s.N
    x = torch.randn(R * N, dtype=torch.float64, device=dev,
                    generator=torch.Generator(device=dev).manual_seed(E))
    y = s.apply_P0(x)
    for r in range(R):
        seg = slice(r * N, (r + 1) * N)
        assert max(backward_errors(E, p, nu, x[seg], y[seg], dev)) <= 1e-14
    s.apply_P0(torch.full_like(x, float("nan")))
    assert torch.equal(s.apply_P0(x), y)
    z = x.clone()
    z[N:2 * N] = float("nan")
    got = s.apply_P0(z)
    assert torch.equal(got[:N], y[:N]) and torch.equal(got[2 * N:], y[2 * N:])
    assert bool(got[N:2 * N].isnan().all())
    s.close()
