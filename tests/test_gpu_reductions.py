"""J^T w at the edges of its tiles: rows around the 64 row groups and the 512
rows in flight, columns around the 16 of a block."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("rows", [1, 63, 64, 65, 511, 512, 513, 4099])
@pytest.mark.parametrize("cols", [1, 15, 16, 17, 160])
def test_jacobian_apply_tiles(rows, cols):
    """A sum of `rows` products in any order is within rows 2^-53 of the sum of
    their magnitudes (and numpy's within the same), a leading dimension above
    the columns; twice the same bits."""
    import paper_1705_03666_amd as pdd
    rng = np.random.default_rng(rows * 1000 + cols)
    J, w = rng.standard_normal((rows, cols + 3)), rng.standard_normal(rows)
    Jd = torch.tensor(J, device="cuda")[:, :cols]
    print(f"jacobian_apply {rows} x {cols}", flush=True)
    a, b = pdd.jacobian_apply(Jd, w), pdd.jacobian_apply(Jd, w)
    torch.cuda.synchronize()
    bound = 2 * (rows + 2) * 2.0 ** -53 * (np.abs(w) @ np.abs(J[:, :cols]))
    assert torch.equal(a, b)
    assert np.all(np.abs(a.cpu().numpy() - w @ J[:, :cols]) <= bound)
