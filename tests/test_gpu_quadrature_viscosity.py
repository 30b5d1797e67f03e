"""The quadrature operator over the range of nu: its pressure and divergence terms
do not depend on nu, and vanishing or denormal viscosity leaves them as they are.
Against B and B' of the Kronecker operators with the operators' tolerance (1e-12
of the largest entry: the same products summed in another order)."""
import sys

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,p", [(6, 2), (7, 3), (4, 4), (3, 6), (12, 3)])
@pytest.mark.parametrize("nu", [1e-310, 1e-100, 3e-308])
def test_coupling_without_viscosity(E, p, nu):
    from paper_2311_06926_amd.solver import Solver
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[quad nu] E={E} p={p} nu={nu}", file=sys.stderr, flush=True)
    s = Solver(E, p, nu, autotune=False)
    x = torch.randn(s.N, dtype=torch.float64, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(E))
    y = s.apply_K_quad(x)
    for got, ref in ((y[:s.nV], s.apply_B(x[s.nV:].clone())),
                     (y[s.nV:], s.apply_Bt(x[:s.nV].clone()))):
        assert float((got - ref).abs().max()) <= 1e-12 * float(ref.abs().max())
    s.close()
