"""The cell list at the edges of its scan: a tile of cells, one more and one
less, several tiles, and grids past the line where one block scans them all."""
import numpy as np
import pytest

from oracle import learned as OL

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.fail("GPU tests need a visible GPU")
    return t


@pytest.mark.parametrize("cells", [
    (3, 3, 227), (8, 16, 16), (3, 683, 3), (64, 64, 32), (52, 52, 52), (64, 64, 64),
    (256, 256, 128),   # 2^23 cells: the largest grid of the several-block scan
    (204, 204, 204),   # more: the one-block scan
])
def test_descriptor_over_cell_grids(torch, cells):
    from paper_2504_15508_amd import learned as L
    rng = np.random.default_rng(sum(cells))
    box = 4.0 * np.array(cells) + 0.5
    n, k = 400, 300
    # pairs and clumps all over the box, its first and last cells among them; 8
    # binary places: the FP32 differences of the coordinates are exact
    at = rng.random((40, 3)) * box
    at[0], at[1] = 0.0, box - 0.01
    pos = at[rng.integers(0, 40, n)] + rng.normal(0.0, 1.2, (n, 3))
    pos = np.mod(np.round(np.mod(pos, box) * 256.0) / 256.0, box)
    q = rng.choice([6.0, 1.0, -8.0], n)
    t = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float32, device="cuda")
    x = (t(pos[:k]), t(q[:k]), t(pos[k:]), t(q[k:]))
    T0, _ = OL.descriptor(pos, q, box)
    m = L.Mlp(n)
    for _ in range(2):  # the counts are cleared for the second call
        T, order = m.descriptor(box, *x)
        got = np.zeros((n, 32, 4))
        got[order.cpu().numpy()] = T.double().cpu().numpy()
        assert sorted(order.cpu().numpy().tolist()) == list(range(n))
        assert np.abs(got - T0).max() <= 2e-5 * np.abs(T0).max()  # the parity test's bar
