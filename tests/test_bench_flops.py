"""The flops that the benchmark divides by the time and by the FP64 peak are
those of the products the fast diagonalisation needs: counted here product by
product, and as the performance cases count them."""
import pytest

pytest.importorskip("torch")


def half_products(shape, d):
    """Flops of one mode product along d, split into even and odd halves."""
    n = shape[d]
    lines = shape[0] * shape[1] * shape[2] // n
    he, ho = (n + 1) // 2, n // 2
    return 2.0 * lines * (he * he + ho * ho)


@pytest.mark.parametrize("E,p", [(6, 2), (32, 3), (61, 3), (256, 2)])
def test_fast_diagonalisation_flops(E, p):
    import bench
    from perf import cases
    nN, nM = E + p - 2, E + p - 1
    vel = sum(2 * half_products([nN if d == c else nM for d in range(3)], e)
              for c in range(3) for e in range(3))
    pres = sum(half_products([nM] * 3, e) for e in range(3))
    # he^2 + ho^2 is n^2 / 2, and half more for odd n
    for got, ref in ((bench.pv0_flops(E, p), vel), (bench.p0_flops(E, p), vel + pres)):
        assert 0 <= ref - got <= ref / nN ** 2
    case = dict(next(c for c in cases.listed() if c["op"] == "P0"), E=E, p=p, nrhs=1)
    assert bench.p0_flops(E, p) == cases.work(case)["flops"]
