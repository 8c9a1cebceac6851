"""Streams that run long: every wavefront of a grid of one block per compute
unit takes several times its ring's places in paths (trees), from items of
many rows and from items of one path, most of them short and a few of them
longer than the ring holds behind them.  So the hand-out stops for room and for
open items and goes on inside an item, items leave the ring row by row, the
ring wraps, and the steps are those of full wavefronts.  Per path (tree)
against the oracle, and independent of how the call is cut."""
import numpy as np
import pytest

from workloads.problem import LinearProblem, ball, box, factor, make_fun, zero_fun

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

WAVES_PER_BLOCK = 4
RING = {"fp64": 512, "fp32": 1024}   # path values a wavefront keeps; trees: 512
OPEN = 8                             # items a wavefront keeps open


def _cus():
    return torch.cuda.get_device_properties(torch.cuda.current_device()).multi_processor_count


def _piece(total, chunk):
    """The forward walks' piece size at one block per compute unit (restated):
    at most 64 paths, or four pieces for every wavefront."""
    piece = chunk
    while piece > 64 and total // piece < 4 * _cus() * WAVES_PER_BLOCK:
        piece //= 2
    return piece


def _problem(kind, dim, bcf):
    dom = box((0.0,) * dim, (1.0,) * dim) if kind == "box" else ball(dim, 1.0, (0.1,) * dim)
    lin = lambda c: make_fun([], 1, [c] + [0.3 - 0.1 * k for k in range(dim)])  # noqa: E731
    z = [zero_fun()] * dim
    return LinearProblem(dom, 1.0, [lin(0.2)] * dim if bcf else z, lin(0.7) if bcf else zero_fun(),
                         lin(-0.4) if bcf else zero_fun(), lin(0.3))


def _calls(kind, dim, per_wave, rows):
    """Nodes and budgets of per_wave paths a wavefront: of a few nodes just
    inside the boundary (many rows an item), or of nodes of one to three paths."""
    total = per_wave * _cus() * WAVES_PER_BLOCK
    x = np.full((7 if rows else total // 2, dim), 0.5 if kind == "box" else 0.1)
    x[:, 0] = (0.0 if kind == "box" else 0.1 - 1.0) + 1e-3 * (1 + np.arange(len(x)) % 5)
    if rows:
        paths = np.full(7, total // 7, np.int64)
        paths[3] += 37
    else:
        paths = np.random.default_rng(3).integers(1, 4, len(x)).astype(np.int64)
        assert len(x) > 10 * OPEN * _cus() * WAVES_PER_BLOCK
    return x, paths


ONE_BLOCK = dict(blocks_per_cu=1, chunk_paths=4096)


@pytest.mark.parametrize("rows", [True, False])
@pytest.mark.parametrize("kind,dim,layout,bcf,cap", [
    ("box", 1, "pair52", False, 0), ("ball", 2, "quad24", False, 0), ("box", 3, "pair52", False, 0),
    ("ball", 3, "quad24", False, 25), ("box", 2, "quad24", True, 0), ("ball", 1, "pair52", True, 40)])
def test_long_streams_match_the_oracle_per_path(orc, kind, dim, layout, bcf, cap, rows):
    """Values to 1e-12 and steps exactly (the tolerance of every FP64 per-path
    test here)."""
    import paper_1705_03666_amd as pdd
    P = _problem(kind, dim, bcf)
    nodes, paths = _calls(kind, dim, 3 * RING["fp64"], rows)
    assert not rows or _piece(int(paths.sum()), 4096) > 2 * 64
    print(f"long stream {kind} {dim} {layout} bcf={bcf} cap={cap} rows={rows}: {paths.sum()} paths", flush=True)
    o = orc.walk(P, nodes, paths, 4e-3, 5, layout=orc.PAIR52 if layout == "pair52" else orc.QUAD24, dump=True,
                 max_steps=cap or None)
    g = pdd.mc_interface(P, nodes, paths, 4e-3, 5, precision="fp64", layout=layout, dump=True, max_steps=cap, **ONE_BLOCK)
    torch.cuda.synchronize()
    steps = np.asarray(o["path_steps"])
    # paths that the ring cannot hold the successors of (64 lanes at the mean length), where no cap cuts them
    assert cap or np.mean(steps > RING["fp64"] / 64 * steps.mean()) > 5e-4
    assert np.array_equal(g["path_steps"].cpu().numpy(), steps)
    phi = np.asarray(o["phi"])
    assert np.all(np.abs(g["phi"].cpu().numpy() - phi) <= 1e-12 * np.maximum(1.0, np.abs(phi)))
    for k in ("n", "steps", "censored"):
        assert np.array_equal(g[k].cpu().numpy(), o[k]), k
    assert np.allclose(g["mean"].cpu().numpy(), o["mean"], rtol=1e-12, atol=1e-12)
    assert np.allclose(g["m2"].cpu().numpy(), o["m2"], rtol=1e-9, atol=1e-12)


def _sums_agree(g, phi, paths):
    """The statistics are those of the dumped values (added in 80 bits)."""
    phi = phi.astype(np.longdouble)
    off = np.concatenate([[0], np.cumsum(paths)])
    s = np.add.reduceat(phi, off[:-1])
    mean = s / paths
    m2 = np.add.reduceat((phi - np.repeat(mean, paths)) ** 2, off[:-1])
    assert np.allclose(g["mean"].cpu().numpy(), mean, rtol=1e-12, atol=1e-12)
    assert np.allclose(g["m2"].cpu().numpy(), m2, rtol=1e-9, atol=1e-12)


@pytest.mark.parametrize("rows", [True, False])
@pytest.mark.parametrize("mode", ["free", "bcf", "terms", "wos"])
def test_long_fp32_streams_do_not_depend_on_the_cut(mode, rows):
    """Per-path values and steps bit for bit at the default schedule, where a
    wavefront gets a few paths, and in long streams."""
    import paper_1705_03666_amd as pdd
    P = _problem("ball", 2, mode == "bcf")
    if mode == "terms":
        P.c = make_fun([(0.4, [factor("sin", 0)]), (0.5, [])])
    nodes, paths = _calls("ball", 2, 3 * RING["fp32"], rows)
    assert not rows or _piece(int(paths.sum()), 4096) > 2 * 64
    print(f"long stream fp32 {mode} rows={rows}: {paths.sum()} paths", flush=True)
    if mode == "wos":
        call = lambda **kw: pdd.wos_interface(P, nodes, paths, 1e-4, 3, precision="fp32", dump=True, **kw)  # noqa: E731
    else:
        call = lambda **kw: pdd.mc_interface(P, nodes, paths, 4e-3, 3, precision="fp32", dump=True, **kw)  # noqa: E731
    ref = call()
    for kw in (ONE_BLOCK, dict(ONE_BLOCK, refill_groups=1), dict(ONE_BLOCK, refill_groups=20)):
        g = call(**kw)
        torch.cuda.synchronize()
        assert torch.equal(g["phi"], ref["phi"]) and torch.equal(g["path_steps"], ref["path_steps"]), kw
        _sums_agree(g, g["phi"].cpu().numpy(), paths)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_a_batch_streams_its_problems_one_after_the_other(precision):
    """Long streams of four problems of different dimension and domain, two of
    them with drift, killing and source: the paths are those of a call each."""
    import paper_1705_03666_amd as pdd
    probs = [_problem("box", 1, False), _problem("ball", 2, True), _problem("box", 3, False), _problem("ball", 3, True)]
    kinds = ["box", "ball", "box", "ball"]
    parts = [_calls(k, P.domain.ndim, RING[precision], i % 2 == 0) for i, (P, k) in enumerate(zip(probs, kinds))]
    nodes = np.concatenate([np.pad(x, ((0, 0), (0, 3 - x.shape[1]))) for x, _ in parts])
    paths = np.concatenate([p for _, p in parts])
    which = np.concatenate([np.full(len(p), i, np.int32) for i, (_, p) in enumerate(parts)])
    assert _piece(int(paths.sum()), 4096) > 2 * 64
    print(f"long stream batch {precision}: {paths.sum()} paths", flush=True)
    kw = dict(precision=precision, dump=True)
    g = pdd.mc_interface_batch(probs, which, nodes, paths, 4e-3, 5, **kw, **ONE_BLOCK)
    ref = pdd.mc_interface_batch(probs, which, nodes, paths, 4e-3, 5, **kw)
    torch.cuda.synchronize()
    assert torch.equal(g["phi"], ref["phi"]) and torch.equal(g["path_steps"], ref["path_steps"])
    _sums_agree(g, g["phi"].cpu().numpy(), paths)
    # the first problem's paths (its nodes have the same numbers alone) are the single call's
    n0 = int(parts[0][1].sum())
    one = pdd.mc_interface(probs[0], parts[0][0], parts[0][1], 4e-3, 5, **kw)
    torch.cuda.synchronize()
    assert torch.equal(g["phi"][:n0], one["phi"]) and torch.equal(g["path_steps"][:n0], one["path_steps"])


@pytest.mark.parametrize("chunk", [700, 1])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_long_tree_streams(orc, precision, chunk):
    """Trees with a boundary, from items of 700 (more than the ring of 512) and
    of one tree: FP64 against the oracle per tree, FP32 bit for bit the trees of
    the default schedule."""
    import paper_1705_03666_amd as pdd
    from workloads import configs as CF
    B, Bd = CF.kpp_bvp_travelling_wave(-1.0, 1.5, 0.02, (0.0, 0.25, 0.5))
    pts = np.array([[-0.97], [-0.9], [0.3], [1.45], [1.49], [1.48], [2.0]])
    trees = 3 * 512 * _cus() * WAVES_PER_BLOCK // len(pts)
    print(f"long tree stream {precision} chunk={chunk}: {len(pts)} x {trees} trees", flush=True)
    kw = dict(precision=precision, dump=True)
    if precision == "fp64":
        kw["layout"] = "pair52"
    g = pdd.branching_bvp(B, Bd, pts, trees, 9, blocks_per_cu=1, chunk_paths=chunk, **kw)
    torch.cuda.synchronize()
    v = g["value"].double().cpu().numpy()
    if precision == "fp64":
        o = orc.branching_bvp(B, Bd, pts, trees, 9, layout=orc.PAIR52, dump=True)
        assert np.array_equal(g["segments"].cpu().numpy(), o["segments"])
        ov = np.asarray(o["value"])
        assert np.all(np.abs(v - ov) <= 1e-12 * np.maximum(1.0, np.abs(ov)))
        for k in ("n", "steps"):
            assert np.array_equal(g[k].cpu().numpy(), o[k]), k
    else:
        ref = pdd.branching_bvp(B, Bd, pts, trees, 9, **kw)
        torch.cuda.synchronize()
        assert torch.equal(g["value"], ref["value"]) and torch.equal(g["segments"], ref["segments"])
        assert torch.equal(g["steps"], ref["steps"]) and torch.equal(g["n"], ref["n"])
    # (80-bit sums: numpy adds 224694 values along this axis one by one, which costs 64 bits 1e-11)
    v = v.astype(np.longdouble)
    assert np.allclose(g["mean"].cpu().numpy(), v.mean(axis=1).T, rtol=1e-12, atol=1e-12)
    assert np.allclose(g["m2"].cpu().numpy(), ((v - v.mean(axis=1, keepdims=True)) ** 2).sum(axis=1).T,
                       rtol=1e-9, atol=1e-12)
