"""P_k at k = 0 and 1, whose V and Q blocks share their launches: against the
same blocks composed of the single operators, over orders, right-hand sides,
fast-diagonalisation plans, precisions and the operator shapes with and without
a common launch of the two pressure chains.  The V block's arithmetic is that
of apply_PV: equal bit for bit.  The Q block composes B P_{Q,0}^{-1} where the
product is 2 nu D^T, in another order: eps times a few tens of operations per
term gives 1e-13 to 1e-12 of the largest entry in FP64 (bound 1e-10) and 1e-5
in FP32 (bound 1e-3)."""
import sys

import pytest

torch = pytest.importorskip("torch")

from paper_2311_06926_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda", 0)


def q_block(sol, q, x):
    """P_{Q,1}^{-1} x of eq. Pcq1 from apply_P0, apply_B, apply_PV and apply_Bt."""
    def p_q0(s):
        z = torch.zeros(sol.N, dtype=torch.float64, device=x.device)
        z[sol.nV:] = s
        return sol.apply_P0(z)[sol.nV:]

    s = x.clone()
    for _ in range(1, q):
        t = sol.apply_Bt(sol.apply_PV(q, 0, sol.apply_B(p_q0(s).contiguous())))
        s = x + s - t
    return p_q0(s)


@pytest.mark.parametrize("E,p,q,nrhs,opts", [
    (1, 2, 2, 1, {}), (15, 2, 2, 1, {}), (16, 3, 3, 2, {}), (17, 4, 4, 1, {}), (33, 2, 3, 3, {}),
    (20, 3, 2, 2, {"fd_plan": 0}), (20, 3, 3, 2, {"fd_plan": 9}), (12, 5, 2, 1, {"fd_plan": 1}),
    (132, 2, 2, 1, {}), (21, 3, 3, 2, {"op_slabs": 2}), (21, 3, 3, 2, {"op_fused": 1}),
    (21, 3, 3, 2, {"op_staged": 1, "op_kchunk": 2}), (21, 3, 2, 1, {"op_pres_wide": 1}),
    (18, 3, 2, 2, {"precision": "fp32"}), (18, 3, 3, 2, {"precision": "bf16x3"}),
])
def test_joint_blocks(dev, E, p, q, nrhs, opts):
    from paper_2311_06926_amd.solver import Solver
    print(f"[pk] E={E} p={p} q={q} nrhs={nrhs} {opts}", file=sys.stderr, flush=True)
    sol = Solver(E, p, 0.7, autotune=False, max_rhs=nrhs, **opts)
    # (the single-pass kernel's A rounds differently; the other shapes agree)
    one = Solver(E, p, 0.7, autotune=False, max_rhs=1,
                 **{k: v for k, v in opts.items() if k == "op_fused" or not k.startswith("op_")})
    N, nV = sol.N, sol.nV
    tol = 1e-10 if opts.get("precision", "fp64") == "fp64" else 1e-3
    x = torch.from_numpy(synth.random_vector(nrhs * N, seed=E + q)).to(dev)
    for k in (0, 1):
        y = sol.apply_hyperpower(q, k, x)
        for r in range(nrhs):
            xr, yr = x[r * N:(r + 1) * N], y[r * N:(r + 1) * N]
            assert torch.equal(yr[:nV], one.apply_PV(q, k, xr[:nV].contiguous()))
            z = q_block(one, q, xr[nV:]) if k else one.apply_P0(xr.contiguous())[nV:]
            assert (yr[nV:] - z).abs().max() <= tol * z.abs().max()
    sol.close()
    one.close()
