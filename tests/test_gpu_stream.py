"""The streaming forward walk at the sizes where it can go wrong: fewer paths
than lanes, partial last rows, more tiny items than a wavefront holds open,
paths longer than the value ring, nodes outside, caps reached while draining;
per path against the oracle, and independent of how the call is cut."""
import numpy as np
import pytest

from workloads.problem import LinearProblem, ball, box, make_fun, zero_fun

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _problem(kind, dim, bcf, offset=0.0):
    dom = box((0.0,) * dim, (1.0,) * dim) if kind == "box" else ball(dim, 1.0, (0.1,) * dim)
    lin = lambda c: make_fun([], 1, [c] + [0.3 - 0.1 * k for k in range(dim)])  # noqa: E731
    z = [zero_fun()] * dim
    return LinearProblem(dom, 1.0, [lin(0.2)] * dim if bcf else z, lin(0.7) if bcf else zero_fun(),
                         lin(-0.4) if bcf else zero_fun(), lin(offset))


def _nodes(kind, dim, n):
    x = np.full((n, dim), 0.5) + 0.03 * np.arange(n)[:, None]
    x[-1] = 3.0                                        # outside
    x[0, 0] = 1e-3 if kind == "box" else 0.1 - 0.3     # box: most paths short, a few very long
    return x


# one path; less than, exactly and more than a wavefront; several rows; none; outside the domain
PATHS = np.array([700, 1, 63, 64, 65, 0, 130], np.int64)


@pytest.mark.parametrize("kind", ["box", "ball"])
@pytest.mark.parametrize("dim", [1, 2, 3])
@pytest.mark.parametrize("layout", ["pair52", "quad24"])
@pytest.mark.parametrize("bcf", [False, True])
def test_stream_matches_the_oracle_per_path(orc, kind, dim, layout, bcf):
    """Values to 1e-12 and steps exactly (the tolerance of every FP64 per-path
    test here), whole and capped."""
    import paper_1705_03666_amd as pdd
    P, nodes = _problem(kind, dim, bcf), _nodes(kind, dim, len(PATHS))
    lay = orc.PAIR52 if layout == "pair52" else orc.QUAD24
    for cap, kw in ((0, {}), (0, dict(chunk_paths=5, blocks_per_cu=1)), (37, {}), (150, dict(chunk_paths=64))):
        print(f"stream {kind} {dim} {layout} bcf={bcf} cap={cap} {kw}", flush=True)
        o = orc.walk(P, nodes, PATHS, 4e-3, 5, layout=lay, dump=True, max_steps=cap or None)
        g = pdd.mc_interface(P, nodes, PATHS, 4e-3, 5, precision="fp64", layout=layout, dump=True, max_steps=cap, **kw)
        torch.cuda.synchronize()
        assert np.array_equal(g["path_steps"].cpu().numpy(), o["path_steps"])
        phi = np.asarray(o["phi"])
        assert np.all(np.abs(g["phi"].cpu().numpy() - phi) <= 1e-12 * np.maximum(1.0, np.abs(phi)))
        for k in ("n", "steps", "censored"):
            assert np.array_equal(g[k].cpu().numpy(), o[k]), k
        assert np.allclose(g["mean"].cpu().numpy(), o["mean"], rtol=1e-12, atol=1e-12)
        assert np.allclose(g["m2"].cpu().numpy(), o["m2"], rtol=1e-9, atol=1e-12)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("wos", [False, True])
def test_stream_does_not_depend_on_the_cut(precision, wos):
    """Per-path values and steps bit for bit whatever the items, the grid and
    the refills; the statistics are those of the path values (1e-9 of the sum
    of squares for values of 1e4 and deviations of 0.3: 2^-52 (1e4 / 0.3)^2
    = 2.5e-7 is what a plain sum of squares would lose)."""
    import paper_1705_03666_amd as pdd
    P = _problem("ball", 2, False, offset=1e4)
    nodes = np.array([[0.1, 0.1], [-0.4, 0.3], [1.0, 0.3], [0.1, 1.05]])
    paths = np.array([2100, 1, 513, 1025], np.int64)
    call = (lambda **kw: pdd.wos_interface(P, nodes, paths, 1e-4, 3, precision=precision, dump=True, **kw)) if wos else \
        (lambda **kw: pdd.mc_interface(P, nodes, paths, 2e-3, 3, precision=precision, dump=True, **kw))
    print(f"stream cut {precision} wos={wos}", flush=True)
    ref = call()
    for kw in (dict(chunk_paths=100000, blocks_per_cu=1), dict(chunk_paths=1), dict(refill_groups=1),
               dict(refill_groups=40, chunk_paths=300)):
        g = call(**kw)
        torch.cuda.synchronize()
        assert torch.equal(g["phi"], ref["phi"]) and torch.equal(g["path_steps"], ref["path_steps"]), kw
        phi, off = g["phi"].cpu().numpy(), np.concatenate([[0], np.cumsum(paths)])
        for i in range(len(paths)):
            v = phi[off[i]:off[i + 1]]
            assert g["mean"][i].item() == pytest.approx(v.mean(), rel=1e-13)
            assert g["m2"][i].item() == pytest.approx(np.sum((v - v.mean()) ** 2), rel=1e-9, abs=1e-12)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("trees", [1, 65, 1500])
def test_branching_trees_stream_independent_of_the_cut(precision, trees):
    """Trees with a boundary, handed out across items of one tree to more than
    the ring holds: the same trees bit for bit; the sums are those of the
    dumped values (the tolerances of the FP64 sums above)."""
    import paper_1705_03666_amd as pdd
    from workloads import configs as CF
    B, Bd = CF.kpp_bvp_travelling_wave(-1.0, 1.5, 0.01, (0.0, 0.25, 0.5, 1.0))
    pts = np.array([[-0.6], [0.0], [0.8], [1.3], [2.0]])
    ref = None
    for kw in ({}, dict(chunk_paths=1, blocks_per_cu=1), dict(chunk_paths=7, blocks_per_cu=1), dict(chunk_paths=700)):
        print(f"bvp stream {precision} trees={trees} {kw}", flush=True)
        g = pdd.branching_bvp(B, Bd, pts, trees, 9, precision=precision, dump=True, **kw)
        torch.cuda.synchronize()
        ref = g if ref is None else ref
        assert torch.equal(g["value"], ref["value"]) and torch.equal(g["segments"], ref["segments"])
        assert torch.equal(g["steps"], ref["steps"]) and torch.equal(g["n"], ref["n"])
        v = g["value"].double().cpu().numpy()
        mean = v.mean(axis=1).T
        assert np.allclose(g["mean"].cpu().numpy(), mean, rtol=1e-12, atol=1e-12)
        assert np.allclose(g["m2"].cpu().numpy(), ((v - v.mean(axis=1, keepdims=True)) ** 2).sum(axis=1).T,
                           rtol=1e-9, atol=1e-12)


@pytest.mark.parametrize("dim", [1, 2, 3])
@pytest.mark.parametrize("deg", range(9))
def test_boundary_polynomials_of_every_degree(orc, dim, deg):
    """Rows of 1 to 9 coefficients, alone and in a batch, per path to 1e-12 of
    the oracle and bit for bit the same in both."""
    import paper_1705_03666_amd as pdd
    from math import comb
    rng = np.random.default_rng(10 * dim + deg)
    z = [zero_fun()] * dim
    P = LinearProblem(ball(dim, 1.0, (0.1,) * dim), 1.0, z, zero_fun(), zero_fun(),
                      make_fun([], deg, list(rng.standard_normal(comb(dim + deg, dim)))))
    nodes, paths = np.full((2, dim), 0.2), np.array([65, 30], np.int64)
    print(f"boundary polynomial dim={dim} deg={deg}", flush=True)
    o = orc.walk(P, nodes, paths, 4e-3, 5, layout=orc.QUAD24, dump=True)
    g = pdd.mc_interface(P, nodes, paths, 4e-3, 5, precision="fp64", layout="quad24", dump=True)
    pad = np.concatenate([nodes, np.zeros((2, 3 - dim))], axis=1)
    b = pdd.mc_interface_batch([P], np.zeros(2, np.int32), pad, paths, 4e-3, 5, precision="fp64", layout="quad24",
                               dump=True)
    torch.cuda.synchronize()
    phi = np.asarray(o["phi"])
    assert np.all(np.abs(g["phi"].cpu().numpy() - phi) <= 1e-12 * np.maximum(1.0, np.abs(phi)))
    assert torch.equal(g["phi"], b["phi"])
