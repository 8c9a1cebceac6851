"""pdd_mc_interface_noalloc at the end of its fixed scratch area: a call that
fits with its items whole is taken, whatever running them in pieces would
need, and to the last byte."""
import ctypes as C

import numpy as np
import pytest

from workloads.problem import LinearProblem, box, make_fun, zero_fun

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

def _call(pdd, entry, P, nodes, paths, out):
    keep = []
    p = pdd._linear(P, keep)
    o = pdd._options("fp32", None, 0, "persistent", 0, 0, 0)
    fn = getattr(pdd.library(), entry)
    return fn(C.byref(p), nodes.data_ptr(), nodes.shape[0], paths.ctypes.data_as(C.POINTER(C.c_int64)), 4e-3, 9,
              C.byref(o), out.data_ptr(), torch.cuda.current_stream().cuda_stream)


# Scratch of a 1-D call with whole items, in parts of 256 bytes: node
# coordinates, first items and path offsets (8 bytes a node each, the last two
# one more), 64 bytes an item, and six small parts.
# 680000 nodes and 2551 items: 16.5 MB, 18.4 MB in pieces of 64 paths.
# 698944 nodes and one item of one path: 248 bytes below the limit; 8 nodes
# more: 72 bytes above it.
@pytest.mark.parametrize("n,many,fits", [(680000, 1_900_000, True), (698944, 1, True), (698952, 1, False)])
def test_calls_that_fit_with_whole_items_are_taken(n, many, fits):
    import paper_1705_03666_amd as pdd
    P = LinearProblem(box((0.0,), (1.0,)), 1.0, [zero_fun()], zero_fun(), zero_fun(), make_fun([], 1, [0.2, 1.0]))
    paths = np.zeros(n, np.int64)
    paths[n // 3] = many
    nodes = torch.full((n, 1), 0.02, dtype=torch.float64, device="cuda")
    a = torch.full((n, 5), float("nan"), dtype=torch.float64, device="cuda")
    b = torch.full((n, 5), float("nan"), dtype=torch.float64, device="cuda")
    print(f"noalloc limit: {n} nodes, {many} paths", flush=True)
    st = _call(pdd, "pdd_mc_interface_noalloc", P, nodes, paths, a)
    if not fits:
        torch.cuda.synchronize()
        assert st == -2 and "fixed scratch area" in pdd.library().pdd_last_error().decode()
        assert torch.isnan(a).all()
        return
    assert st == 0, pdd.library().pdd_last_error()
    assert _call(pdd, "pdd_mc_interface", P, nodes, paths, b) == 0
    torch.cuda.synchronize()
    a, b = a.cpu().numpy(), b.cpu().numpy()
    assert np.array_equal(a[:, 2:].view(np.int64), b[:, 2:].view(np.int64))
    assert a[n // 3, 2].view(np.int64) == many
    # FP64 sums of the same path values, in another order
    assert np.allclose(a[:, 0], b[:, 0], rtol=1e-12, atol=0) and np.allclose(a[:, 1], b[:, 1], rtol=1e-9, atol=0)
