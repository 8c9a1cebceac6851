"""Every Gaussian of a block, as the FP64 walk draws them (cosine and sine of
each pair, both pairs of a QUAD24 block, the blocks that follow): with b = c =
0, f(x) = x_k, g = 0, X_0 = 0 and a cap of five steps a path's value is
dt (X_1 + .. + X_4)_k, so it holds the coordinate k of the first four steps."""
import numpy as np
import pytest

from workloads.problem import LinearProblem, box, make_fun, zero_fun

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("layout", ["pair52", "quad24"])
@pytest.mark.parametrize("dim,k", [(1, 0), (2, 0), (2, 1), (3, 0), (3, 1), (3, 2)])
def test_every_gaussian_of_a_block(orc, dim, k, layout):
    """Tolerance, in units of 2^-49 (half the last place of numbers from 16 to
    32; |X| < 4 x 0.5 x 8.7 < 17.5 and |value| < 22 here): a Gaussian is within 2
    ulps of r (the walk) and 6.2 (the oracle, whose angle is rounded) of the
    exact one, r < 8.7, so the two differ by at most 8.2; the four enter the
    value 4, 3, 2 and 1 times with dt sqrt(dt) = 1/8: 10.25.  Rounding on each
    side: two for each step of X, entering 4 + 3 + 2 + 1 times with dt = 1/4:
    5, and one for each of the five sums: 5."""
    import paper_1705_03666_amd as pdd
    linear = [0.0] * (dim + 1)
    linear[1 + k] = 1.0
    P = LinearProblem(box((-100.0,) * dim, (100.0,) * dim), 1.0, [zero_fun()] * dim, zero_fun(),
                      make_fun([], 1, linear), make_fun([(0.0, [])]))
    nodes, paths, dt = np.zeros((2, dim)), np.full(2, 30000, np.int64), 0.25
    kw = dict(max_steps=5, dump=True)
    print(f"gaussians of a block: dim {dim} k {k} {layout}", flush=True)
    g = pdd.mc_interface(P, nodes, paths, dt, 78, precision="fp64", layout=layout, **kw)
    torch.cuda.synchronize()
    o = orc.walk(P, nodes, paths, dt, 78, layout=orc.PAIR52 if layout == "pair52" else orc.QUAD24, **kw)
    v, vo = g["phi"].cpu().numpy(), np.asarray(o["phi"])
    assert np.all(g["path_steps"].cpu().numpy() == 5)
    assert np.max(np.abs(v - vo)) <= (10.25 + 2 * (5 + 5)) * 2.0 ** -49
    # variance (1/8)^2 (16 + 9 + 4 + 1): the four Gaussians are all there, and independent
    assert abs(v.var() / (30.0 / 64.0) - 1.0) < 4.5 * np.sqrt(2.0 / len(v))
