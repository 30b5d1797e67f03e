"""The scaling omega / (2 nu (l1 + l2 + l3)) of P_0 over the range of nu: exact in
powers of two, as a correctly rounded division is, and zero, not NaN, where the
eigenvalue sum overflows."""
import math
import sys

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,p,plan", [(9, 3, 1), (9, 3, 9), (9, 3, 8), (127, 3, 8)])
def test_viscosity_range(E, p, plan):
    from paper_2311_06926_amd.solver import Solver
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[scaling] E={E} p={p} plan {plan}", file=sys.stderr, flush=True)
    s = Solver(E, p, 1.0, autotune=False, fd_plan=plan)
    x = torch.randn(s.nV, dtype=torch.float64, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(E))
    y = s.apply_PV(2, 0, x)
    assert bool(y.isfinite().all()) and bool((y != 0).any())
    # 2 nu (l1 + l2 + l3) stays in the normal range: the same digits
    for e in (-900, 900):
        s.set_nu(math.ldexp(1.0, e))
        assert torch.equal(s.apply_PV(2, 0, x), y * math.ldexp(1.0, -e))
    # it overflows for every mode: 1 / inf
    s.set_nu(1.7e308)
    assert bool((s.apply_PV(2, 0, x) == 0).all())
    # and for the larger ones only
    s.set_nu(math.ldexp(1.0, 1023) / 100)
    assert bool(s.apply_PV(2, 0, x).isfinite().all())
    s.close()
