"""The correction network where its tiles end: gradients for last tiles that are
not full and for blocks that take several tiles, and the correction particle by
particle (one norm over all particles lets dense ones hide the others).  The
oracle takes the library's own descriptor, which other tests compare, so that
only the network is judged."""
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


def _lattice(n, seed):
    """n particles at water's density, jittered from a lattice."""
    rng = np.random.default_rng(seed)
    m = int(np.ceil(n ** (1 / 3)))
    box = np.full(3, max(12.5, 1.96 * m))
    g = (np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3) + 0.5) * 1.96
    pos = g[np.sort(rng.permutation(m ** 3)[:n])] + rng.normal(0.0, 0.3, (n, 3))
    return np.mod(pos, box), rng.choice([6.0, 1.0, -8.0], n), box


def _clump(n, seed):
    rng = np.random.default_rng(seed)
    box = np.array([20.0, 16.5, 24.5])
    pos = rng.random((n, 3)) * box
    pos[: n // 2] = np.mod(rng.normal(0.0, 1.2, (n // 2, 3)), box)
    return pos, rng.choice([6.0, 1.0, -8.0], n), box


def _inputs(torch, pos, q):
    k = (2 * len(q)) // 3
    t = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float32, device="cuda")
    return (t(pos[:k]), t(q[:k]), t(pos[k:]), t(q[k:])), k, t


def _descriptor(m, box, x, n):
    T, order = m.descriptor(box, *x)
    got = np.zeros((n, 32, 4))
    got[order.cpu().numpy()] = T.double().cpu().numpy()
    return got, np.einsum("nka,nla->nkl", got, got[:, :4, :]).reshape(n, -1)


def _network(m, D, like, seed):
    """Random parameters, normalised by the particles `like`."""
    from paper_2504_15508_amd import learned as L
    p = OL.init_params(seed)
    rng = np.random.default_rng(seed + 1)
    for k in ("b1", "b2", "b3", "b4"):
        p[k] = rng.normal(0.0, 0.1, p[k].shape)
    mu = D[like].mean(0).astype(np.float32)
    isd = (1.0 / (D[like].std(0) + 1e-6 * (np.abs(D[like]).max() + 1))).astype(np.float32)
    m.set_params(L.pack({**p, "mu": mu, "inv_sigma": isd}))
    return {k: v.astype(np.float32).astype(np.float64) for k, v in p.items()}, mu.astype(float), isd.astype(float)


# tiles of 64 particles, 256 blocks: part of a tile, a tile and one, several and
# one, and more tiles than blocks (16,449 = 257 * 64 + 1: one block takes two)
@pytest.mark.parametrize("n", [1, 3, 63, 65, 257, 16449])
def test_gradients_of_partial_and_repeated_tiles(torch, n):
    from paper_2504_15508_amd import learned as L
    pos, q, box = _lattice(n, n)
    x, k, t = _inputs(torch, pos, q)
    m = L.Mlp(n)
    T, D = _descriptor(m, box, x, n)
    p, mu, isd = _network(m, D, slice(None), 5)
    target = np.random.default_rng(n + 7).normal(0.0, 0.05, (n, 3)).astype(np.float32).astype(float)
    loss, g = m.train_step(box, *x, t(target[:k]), t(target[k:]), lr=0.0, want_grad=True)
    dF, cache = OL.forward(p, T, D, q, mu, isd, 0.01, emulate_bf16=True)
    loss0, g0 = OL.loss_and_grad(p, cache, dF, target, emulate_bf16=True)
    assert abs(float(loss) - loss0) <= 1e-3 * loss0
    gd = L.unpack(np.concatenate([g.cpu().numpy(), np.zeros(256, np.float32)]))
    # a rounding to bf16 that the two sides take differently moves one of at
    # least 32 values by up to 2^-7 of it: that much for a few particles, and the
    # full-tile test's bar where many average
    bar = 2.0 ** -7 if n < 257 else 1e-3
    for name in g0:
        norm = np.linalg.norm(g0[name])
        assert np.linalg.norm(gd[name] - g0[name]) <= bar * norm, name  # n = 1: no neighbours, all zero


@pytest.mark.parametrize("make,n", [(_lattice, 31), (_lattice, 33), (_lattice, 257), (_lattice, 1000), (_clump, 900)])
def test_correction_of_every_particle(torch, make, n):
    from paper_2504_15508_amd import learned as L
    pos, q, box = make(n, 3 * n)
    x, k, t = _inputs(torch, pos, q)
    m = L.Mlp(n)
    T, D = _descriptor(m, box, x, n)
    # the inputs of the sparser half are of order one, so errors in them count
    size = np.abs(D).max(1)
    p, mu, isd = _network(m, D, size <= np.median(size), 9)
    ref, cache = OL.forward(p, T, D, q, mu, isd, 0.01, emulate_bf16=True)
    dF = np.concatenate([a.double().cpu().numpy() for a in m.forward(box, *x)])
    # four roundings to bf16 taken differently on one particle's way through the
    # network, 2^-7 each (one in a thousand of its 320 is that close to a tie),
    # of the product of the norms that the head's sum is made of
    scale = 0.01 * np.abs(q) * np.linalg.norm(T[:, :, 1:], axis=(1, 2)) * np.linalg.norm(cache["c"], axis=1)
    worst = (np.linalg.norm(dF - ref, axis=1) / np.maximum(scale, 1e-30)).max()
    print(f"largest particle error {worst:.2e} of its scale")
    assert worst <= 2.0 ** -5
