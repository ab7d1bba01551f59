"""Many neighbours: a scan that stops when a list is full and goes on where it
stopped lists every neighbour once, for one particle of a wave with thousands
and others with none."""
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


# a list stops past 62 entries and ends at 78, a chunk has 16 candidates: counts at
# and around these, two lists and many; the centre particle's neighbours lie within the cutoff, the others in
# a shell around them so that only it has them all
@pytest.mark.parametrize("k", [15, 16, 17, 47, 48, 49, 63, 64, 65, 80, 127, 128, 129, 193, 1500])
@pytest.mark.parametrize("corner", [False, True])
def test_neighbour_counts_around_the_list(torch, k, corner):
    from paper_2504_15508_amd import learned as L
    rng = np.random.default_rng(k)
    box = np.array([16.0, 13.0, 24.0])
    centre = np.array([0.01, 12.99, 0.02]) if corner else np.array([7.7, 6.1, 12.3])
    u = rng.normal(size=(k, 3))
    near = centre + u / np.linalg.norm(u, axis=1)[:, None] * (1.0 + 2.9 * rng.random((k, 1)))
    pos = np.concatenate([centre[None], near, rng.random((30, 3)) * box])
    # coordinates of 16 binary places: their FP32 differences are exact
    pos = np.mod(np.round(np.mod(pos, box) * 65536.0) / 65536.0, box)
    q = rng.choice([6.0, 1.0, -8.0], len(pos))
    n = len(pos)
    i, j, d = OL.neighbours(pos, box)
    count = np.bincount(i, minlength=n)
    assert count[0] >= k
    T0, _ = OL.descriptor(pos, q, box, pairs=(i, j, d))
    t = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float32, device="cuda")
    x = (t(pos), t(q), t(pos[:0]), t(q[:0]))
    m = L.Mlp(n)
    T, order = m.descriptor(box, *x)
    got = np.zeros((n, 32, 4))
    got[order.cpu().numpy()] = T.double().cpu().numpy()
    # FP32 sums of up to k terms; a neighbour lost or taken twice is a whole term.
    # Per particle, against the terms' size: k rounding errors of 2^-24 each and
    # those of the recurrence (argument error 2^-22, slope at most 31^2); the switch's
    # fast cosine is off by 2^-20 of a charge, however small the switch is
    size, charge = np.zeros(n), np.zeros(n)
    np.add.at(charge, i, np.abs(q[j]))
    np.add.at(size, i, np.abs(q[j]) * 0.5 * (1 + np.cos(np.pi * np.linalg.norm(d, axis=1) / 4.0)))
    bar = (count * 2.0 ** -24 + 961 * 2.0 ** -22) * size + 2.0 ** -20 * charge
    assert (np.abs(got - T0).max(axis=(1, 2)) <= bar).all()
    m.set_params(L.init_params(1))
    m.forward(box, *x)
    st = m.read_stats()
    assert (st["min_neighbours"], st["max_neighbours"]) == (count.min(), count.max())
