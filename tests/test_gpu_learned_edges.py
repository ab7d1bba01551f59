"""The descriptor and the correction where their blocks, lists and cell rows
end: particle counts around a wave's 16 and a block's 32, more neighbours than
one list holds, particles with none, boxes of three cells on an axis, and
neighbours across every face."""
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


def _system(n, box, seed, clump):
    rng = np.random.default_rng(seed)
    pos = rng.random((n, 3)) * box
    if clump:  # half of the particles in two balls, one of them around the box corner
        k = n // 2
        pos[:k] = (rng.normal(0.0, 1.2, (k, 3)) + np.where(rng.random((k, 1)) < 0.5, 0.0, 0.5 * box)) % box
    if box[0] > 200.0:
        # coordinates of 10 binary places: their FP32 differences are exact (a
        # coordinate rounding of 1e-5 A is 5e-5 of such a dense descriptor)
        pos = np.round(pos * 1024.0) / 1024.0 % box
    pos = np.minimum(pos.astype(np.float32), np.nextafter(np.float32(box), np.float32(0))).astype(np.float64)
    q = rng.choice([6.0, 1.0, -8.0], n)
    return pos, q


def _neighbours(pos, box, rc):
    lo, hi = 10 ** 9, 0
    for i in range(len(pos)):
        d = pos - pos[i]
        d -= box * np.rint(d / box)
        c = int(((d ** 2).sum(1) < rc * rc).sum()) - 1
        lo, hi = min(lo, c), max(hi, c)
    return lo, hi


@pytest.mark.parametrize("n,box,clump", [
    (1, (12.0, 12.0, 12.0), False), (5, (40.0, 13.0, 12.5), False), (16, (12.5, 12.5, 12.5), False),
    (31, (12.5, 12.5, 12.5), False), (33, (12.5, 21.0, 16.5), False), (257, (17.0, 12.5, 30.0), False),
    (1000, (12.5, 12.5, 12.5), False),      # about 137 neighbours: three lists
    (900, (20.0, 16.5, 24.5), True),        # lists of very different lengths in one wave
    (700, (64.0, 52.0, 40.0), True),        # 2,080 cells: two tiles of the cell scan
    (300, (256.0, 256.0, 256.0), True),     # 262,144 cells: the one-block scan
])
def test_descriptor_and_correction_match_oracle(torch, n, box, clump):
    from paper_2504_15508_amd import learned as L
    box = np.array(box)
    pos, q = _system(n, box, 11 * n, clump)
    k = (2 * n) // 3
    t = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float32, device="cuda")
    x = (t(pos[:k]), t(q[:k]), t(pos[k:]), t(q[k:]))
    T0, D0 = OL.descriptor(pos, q, box)
    m = L.Mlp(n)
    T, order = m.descriptor(box, *x)
    got = np.zeros((n, 32, 4))
    got[order.cpu().numpy()] = T.double().cpu().numpy()
    scale = max(np.abs(T0).max(), 1e-3)
    assert np.abs(got - T0).max() <= 2e-5 * scale  # the parity test's bar

    p = OL.init_params(4)
    mu, isd = D0.mean(0), 1.0 / (D0.std(0) + 1e-2 * (np.abs(D0).max() + 1))
    m.set_params(L.pack({**p, "mu": mu, "inv_sigma": isd}))
    ref, _ = OL.forward(p, T0, D0, q, mu, isd, 0.01, emulate_bf16=True)
    base = np.random.default_rng(1).normal(0.0, 0.3, (n, 3)).astype(np.float32)
    fi, fw = t(base[:k]), t(base[k:])
    m.forward(box, *x, fi, fw, accumulate=True)
    dF, dw = m.forward(box, *x)
    dF = np.concatenate([dF.double().cpu().numpy(), dw.double().cpu().numpy()])
    norm = np.linalg.norm(ref)
    assert np.linalg.norm(dF - ref) <= 2e-3 * norm + 1e-12  # bf16 rounding decisions that flip, as in the parity test
    both = np.concatenate([fi.double().cpu().numpy(), fw.double().cpu().numpy()])
    assert np.abs(both - (base + dF)).max() <= 1e-6 * max(1.0, np.abs(both).max())  # one FP32 addition
    st = m.read_stats()
    lo, hi = _neighbours(pos, box, 4.0)
    assert (st["min_neighbours"], st["max_neighbours"]) == (lo, hi)
    # |dF| is formed in FP32 from the FP32 components
    assert abs(st["max_correction"] - np.linalg.norm(dF, axis=1).max()) <= 1e-6 * max(st["max_correction"], 1e-30)
