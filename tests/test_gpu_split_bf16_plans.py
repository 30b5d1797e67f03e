"""Split BF16 by plan: the plane plans split each FP32 operand (about 16 bits),
fd_plan 0 and 2 and directions beyond 128 take FP32 products for it, the same
bits as FP32 with one direction per pass."""
import sys

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,p", [(6, 2), (30, 3), (45, 3), (126, 3), (127, 3)])
def test_products_of_split_bf16(E, p):
    from paper_2311_06926_amd.solver import Solver
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[bf16 plans] E={E} p={p}", file=sys.stderr, flush=True)
    x = None
    out, used = {}, {}
    for prec, plan in [("fp32", 0), ("bf16x3", 0), ("bf16x3", 2), ("bf16x3", 1), ("bf16x3", 9),
                       ("bf16x3", 3), ("bf16x3", 8), ("bf16x3", -1)]:
        s = Solver(E, p, 1.0, autotune=False, fd_plan=plan, precision=prec, krylov="fgmres")
        if x is None:
            x = torch.randn(s.N, dtype=torch.float64, device="cuda",
                            generator=torch.Generator(device="cuda").manual_seed(E))
        out[prec, plan] = s.apply_P0(x)
        used[prec, plan] = s.tuning(1)["fd_plan"][1 if prec == "fp32" else 2]
        s.close()
    single = out["fp32", 0]
    long = E + p - 1 > 128
    for plan in (0, 2):
        assert used["bf16x3", plan] == (8 if long else 0)
        assert torch.equal(out["bf16x3", plan], single)
    for plan in (1, 9, 3, 8, -1):
        assert used["bf16x3", plan] == (8 if long else 9 if plan == 9 else 1)
        assert torch.equal(out["bf16x3", plan], single if long else out["bf16x3", 1])
    if not long:
        gap = float((out["bf16x3", 1] - single).abs().max() / single.abs().max())
        assert 1e-7 < gap < 2e-4
