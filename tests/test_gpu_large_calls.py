"""Calls of more nodes (items) than one turn of the reductions' launches takes
(65536): every node's statistics against the oracle, the last turn a partial
one."""
import numpy as np
import pytest

from workloads.problem import LinearProblem, box, make_fun, zero_fun

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [65536, 65537, 150001])
def test_more_nodes_than_a_turn_of_the_reductions(orc, n):
    """Counts and steps exactly; means to 1e-12 (the tolerance of every FP64
    per-path test here).  One node's items are run in pieces, so the pieces of
    as many items are merged in turns too."""
    import paper_1705_03666_amd as pdd
    P = LinearProblem(box((0.0,), (1.0,)), 1.0, [zero_fun()], zero_fun(), zero_fun(), make_fun([], 1, [0.2, 1.0]))
    rng = np.random.default_rng(n)
    nodes, paths = rng.uniform(0.0, 1.0, (n, 1)), rng.integers(1, 4, n).astype(np.int64)
    paths[7], paths[n - 1], paths[n // 2] = 3000, 700, 0
    print(f"large call: {n} nodes", flush=True)
    kw = dict(layout=orc.QUAD24)
    o = orc.walk(P, nodes, paths, 4e-3, 5, **kw)
    g = pdd.mc_interface(P, nodes, paths, 4e-3, 5, precision="fp64", layout="quad24", chunk_paths=4096)
    torch.cuda.synchronize()
    for k in ("n", "steps", "censored"):
        assert np.array_equal(g[k].cpu().numpy(), o[k]), k
    assert np.allclose(g["mean"].cpu().numpy(), o["mean"], rtol=1e-12, atol=1e-12)
    assert np.allclose(g["m2"].cpu().numpy(), o["m2"], rtol=1e-9, atol=1e-12)
