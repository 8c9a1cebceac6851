"""The FP64 Gaussians (Box-Muller on the open lattices) as the walk draws
them, read off two-step paths: with b = c = 0, f(x) = x, g = 0 and a cap of two
steps, a path's value is dt x0 + dt (x0 + sigma sqrt(dt) z), z its first
Gaussian."""
import numpy as np
import pytest

from workloads.problem import LinearProblem, box, make_fun, zero_fun

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("layout", ["pair52", "quad24"])
@pytest.mark.parametrize("dim", [1, 2, 3])
def test_fp64_gaussians_match_the_oracle(orc, dim, layout):
    """Tolerance: z is within 2 ulps of r (here) and 6.2 (the oracle, whose
    angle is rounded) of the exact value, r < 8.7 so an ulp of r is at most
    2^-49, and dividing the value by dt sqrt(dt) = 1/8 with the walk's own four
    roundings of numbers below 3 adds at most 8 x 4 x 2^-52 on each side."""
    import paper_1705_03666_amd as pdd
    poly = [0.0, 1.0] + [0.0] * (dim - 1)
    P = LinearProblem(box((-100.0,) * dim, (100.0,) * dim), 1.0, [zero_fun()] * dim, zero_fun(),
                      make_fun([], 1, poly), make_fun([(0.0, [])]))
    nodes, n, dt = np.zeros((3, dim)), 40000, 0.25
    paths = np.full(3, n, np.int64)
    kw = dict(max_steps=2, dump=True)
    print(f"gaussians: dim {dim} {layout}", flush=True)
    g = pdd.mc_interface(P, nodes, paths, dt, 77, precision="fp64", layout=layout, **kw)
    torch.cuda.synchronize()
    o = orc.walk(P, nodes, paths, dt, 77, layout=orc.PAIR52 if layout == "pair52" else orc.QUAD24, **kw)
    z, zo = g["phi"].cpu().numpy() * 8.0, np.asarray(o["phi"]) * 8.0
    assert np.all(g["path_steps"].cpu().numpy() == 2)
    assert np.max(np.abs(z - zo)) <= 8.2 * 2.0 ** -49 + 2 * 32 * 2.0 ** -52
    # the tails are there: 120000 Gaussians reach 4, and are centred
    assert 3.9 < np.max(np.abs(z)) < 8.7 and abs(z.mean()) < 4.5 / np.sqrt(len(z))
