"""The forms that a plan picks by precision and mesh, where their edges lie:
field spectra kept as three components or as two (FP64, pencil meshes), field
rows padded for stencils that run past the last column, and the shared scratch
layout of the no-allocation step on rows of 16."""
import numpy as np
import pytest

import systems
from oracle import pppm

pytestmark = pytest.mark.gpu

KE, BETA = systems.COULOMB_K, systems.BETA


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.fail("GPU tests need a visible GPU")
    return t


def _gas(n, box, seed):
    """Charges all over the box, the last columns of every axis included."""
    rng = np.random.default_rng(seed)
    pos = rng.random((n, 3)) * box
    pos[: n // 4] = box * (1 - 0.02 * rng.random((n // 4, 3)))
    q = rng.normal(size=n)
    return pos.astype(np.float32).astype(np.float64), (q - q.mean()).astype(np.float32).astype(np.float64)


def _run(torch, plan, pos, q):
    t = lambda a: torch.tensor(a, dtype=plan.dtype, device="cuda")
    k = len(q) // 3
    E, fi, fw, W = plan.compute(t(pos[:k]), t(q[:k]), t(pos[k:]), t(q[k:]))
    torch.cuda.synchronize()
    return float(E), np.concatenate([fi.double().cpu().numpy(), fw.double().cpu().numpy()]), W.cpu().numpy()


# bars: the FP64 mesh is 2^-40 fixed point (1e-10 relative after the transforms),
# FP32 transforms round at ~4e-7 per pass (1e-5), as in the parity tests
BAR = {"fp64": 1e-10, "fp32": 1e-5}


@pytest.mark.parametrize("mesh,order,precision", [
    ((16, 32, 64), 5, "fp64"), ((32, 16, 16), 5, "fp32"),   # planes in LDS
    ((256, 128, 16), 4, "fp64"), ((256, 128, 16), 4, "fp32"),  # pencils: separate inverse y and x passes
])
def test_field_spectra_are_the_products(torch, mesh, order, precision):
    import paper_2504_15508_amd as dl
    box = np.array([11.0, 13.0, 12.0]) * np.array(mesh) / 32
    pos, q = _gas(600, box, 5)
    plan = dl.Plan(mesh, order=order, beta=BETA, coulomb_k=KE, precision=precision, capacity=len(q))
    plan.set_box(box)
    _run(torch, plan, pos, q)
    got = plan.debug_buffer(dl._lib.BUF_FIELD_SPECTRA).cpu().numpy()  # [a][kx][z][ky]
    parts = pppm.pppm(pos, q, box, mesh, order, BETA, KE, return_parts=True)[3]
    n, k = pppm.wavevectors(box, mesh)
    plane = mesh[0] * mesh[1] <= 16384
    for a in range(3):
        kd = np.where(n[a] == -mesh[a] // 2, 0.0, k[a]).reshape([-1 if b == a else 1 for b in range(3)])
        E = np.fft.ifft(-1j * kd * parts["G"] * parts["Qhat"], axis=2) * mesh[2]
        if not plane:
            E = np.fft.ifft(E, axis=1) * mesh[1]  # the inverse y transform is applied as well
        ref = E[: mesh[0] // 2 + 1].transpose(0, 2, 1)
        assert np.abs(got[a] - ref).max() <= BAR[precision] * np.abs(ref).max(), a


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("mesh", [(16, 16, 16), (16, 64, 32), (256, 128, 16)])
@pytest.mark.parametrize("order", [2, 3, 4, 5, 6, 7, 8])
def test_stencils_past_the_last_column(torch, mesh, order, precision):
    import paper_2504_15508_amd as dl
    box = np.array([9.0, 10.0, 9.5]) * np.array(mesh) / 16
    pos, q = _gas(257, box, 7 * order)
    plan = dl.Plan(mesh, order=order, beta=BETA, coulomb_k=KE, precision=precision, capacity=len(q))
    plan.set_box(box)
    E, F, W = _run(torch, plan, pos, q)
    E0, F0, W0 = pppm.pppm(pos, q, box, mesh, order, BETA, KE)
    assert np.linalg.norm(F - F0) <= BAR[precision] * np.linalg.norm(F0)
    assert abs(E - E0) <= BAR[precision] * abs(E0)
    assert np.abs(W - W0).max() <= BAR[precision] * abs(E0)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("mesh,order", [((16, 16, 16), 8), ((16, 512, 256), 8), ((256, 128, 16), 8)])
def test_noalloc_shares_its_scratch(torch, mesh, order, precision):
    import paper_2504_15508_amd as dl
    if precision == "fp64" and mesh == (16, 512, 256):
        mesh = (16, 512, 128)  # FP64 at 16 x 512 x 256 needs more scratch than there is
    box = np.array([9.0, 10.0, 9.5]) * np.array(mesh) / 16
    pos, q = _gas(1001, box, 3)
    plan = dl.Plan(mesh, order=order, beta=BETA, coulomb_k=KE, precision=precision, capacity=len(q))
    plan.set_box(box)
    t = lambda a: torch.tensor(a, dtype=plan.dtype, device="cuda")
    x = (t(pos[:333]), t(q[:333]), t(pos[333:]), t(q[333:]))
    want = plan.compute(*x)
    for _ in range(2):  # the second call finds the first one's contents in the scratch array
        got = dl.plan.compute_noalloc(mesh, box, *x, order=order, beta=BETA, coulomb_k=KE)
        for a, b in zip(got, want):
            assert torch.equal(a, b)


@pytest.mark.parametrize("mesh,order,precision", [((32, 16, 32), 5, "fp32"), ((16, 32, 16), 4, "fp64"),
                                                  ((12, 18, 20), 3, "fp32")])
@pytest.mark.parametrize("n", [2, 1024, 1025, 4096, 4097, 5121, 16384, 16385])
def test_sort_forms(torch, mesh, order, precision, n):
    """The one-block sort up to 4,096 particles, the placement that adds up the
    chunk histograms up to 16 chunks of 1,024, the column scan beyond; the
    spread's block sizes and (FP64) particle splits change along the way."""
    import paper_2504_15508_amd as dl
    box = np.array([9.0, 10.0, 9.5]) * np.array(mesh) / 16
    pos, q = _gas(n, box, n)
    plan = dl.Plan(mesh, order=order, beta=BETA, coulomb_k=KE, precision=precision, capacity=n)
    plan.set_box(box)
    E, F, W = _run(torch, plan, pos, q)
    E0, F0, W0 = pppm.pppm(pos, q, box, mesh, order, BETA, KE)
    assert np.linalg.norm(F - F0) <= BAR[precision] * np.linalg.norm(F0)
    assert abs(E - E0) <= BAR[precision] * abs(E0)
    assert np.abs(W - W0).max() <= BAR[precision] * abs(E0)
    again = _run(torch, plan, pos, q)
    assert again[0] == E and np.array_equal(again[1], F) and np.array_equal(again[2], W)
    # fewer particles through the same buffers
    k = max(1, n // 3)
    Ek = _run(torch, plan, pos[:k], q[:k])[0]
    E1 = pppm.pppm(pos[:k], q[:k], box, mesh, order, BETA, KE)[0]
    assert abs(Ek - E1) <= BAR[precision] * abs(E1)


@pytest.mark.parametrize("mesh,precision", [
    ((5, 6, 5), "fp32"), ((50, 50, 6), "fp32"), ((54, 50, 6), "fp32"), ((25, 15, 400), "fp32"),
    ((90, 90, 10), "fp32"), ((125, 125, 10), "fp32"), ((128, 125, 20), "fp32"),
    ((5, 6, 5), "fp64"), ((50, 54, 6), "fp64"), ((75, 75, 15), "fp64"), ((90, 90, 10), "fp64"), ((25, 10, 500), "fp64")])
def test_block_sizes_of_the_fused_planes(torch, mesh, precision):
    """Mixed meshes from the smallest blocks of the plane and z kernels to the
    largest (planes of 30 to 16,000 points, z rows of 5 to 500)."""
    import paper_2504_15508_amd as dl
    box = np.array([9.0, 10.0, 9.5]) * np.array(mesh) / 16
    pos, q = _gas(900, box, mesh[0] + mesh[2])
    plan = dl.Plan(mesh, order=5, beta=BETA, coulomb_k=KE, precision=precision, capacity=len(q))
    plan.set_box(box)
    E, F, W = _run(torch, plan, pos, q)
    E0, F0, W0 = pppm.pppm(pos, q, box, mesh, 5, BETA, KE)
    assert np.linalg.norm(F - F0) <= BAR[precision] * np.linalg.norm(F0)
    assert abs(E - E0) <= BAR[precision] * abs(E0)
    assert np.abs(W - W0).max() <= BAR[precision] * abs(E0)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_sort_with_many_bins(torch, precision):
    """More bins than the placement adds up by itself (4,096): their totals are staged."""
    import paper_2504_15508_amd as dl
    mesh = (128, 256, 128)
    box = np.array([9.0, 10.0, 9.5]) * np.array(mesh) / 16
    pos, q = _gas(6000, box, 77)
    plan = dl.Plan(mesh, order=4, beta=BETA, coulomb_k=KE, precision=precision, capacity=len(q))
    plan.set_box(box)
    E, F, W = _run(torch, plan, pos, q)
    E0, F0, W0 = pppm.pppm(pos, q, box, mesh, 4, BETA, KE)
    assert np.linalg.norm(F - F0) <= BAR[precision] * np.linalg.norm(F0)
    assert abs(E - E0) <= BAR[precision] * abs(E0)
    assert np.abs(W - W0).max() <= BAR[precision] * abs(E0)
