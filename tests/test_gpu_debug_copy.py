"""The inspection copies report the last compute, whatever was called since, and
take the same sizes whatever form the last compute chose."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.fail("GPU tests need a visible GPU")
    return t


def _plan(torch, mesh, precision, n, box):
    import paper_2504_15508_amd as dl
    plan = dl.Plan(mesh, precision=precision, capacity=n)
    plan.set_box(box)
    rng = np.random.default_rng(n)
    t = lambda a: torch.tensor(a, dtype=plan.dtype, device="cuda")
    plan.compute(t(rng.random((n, 3)) * box), t(rng.normal(size=n)))
    return plan


@pytest.mark.parametrize("mesh,precision", [((32, 32, 32), "fp32"), ((32, 32, 32), "fp64"),
                                            ((256, 128, 16), "fp32"), ((256, 128, 16), "fp64")])
def test_field_spectra_keep_the_box_of_their_compute(torch, mesh, precision):
    import paper_2504_15508_amd as dl
    plan = _plan(torch, mesh, precision, 300, (12.0, 13.0, 14.0))
    before = plan.debug_buffer(dl._lib.BUF_FIELD_SPECTRA)
    plan.set_box((24.0, 11.0, 17.0))
    assert torch.equal(plan.debug_buffer(dl._lib.BUF_FIELD_SPECTRA), before)


@pytest.mark.parametrize("n", [20, 20000])  # one particle split and several
def test_spectrum_copy_refuses_part_of_a_value(torch, n):
    import ctypes
    import paper_2504_15508_amd as dl
    plan = _plan(torch, (32, 32, 32), "fp64", n, (12.0, 13.0, 14.0))
    full = plan.debug_buffer(dl._lib.BUF_SPECTRUM).view(torch.uint8).reshape(-1)
    out = torch.zeros(64, dtype=torch.uint8, device="cuda")
    lib = dl._lib.load()
    copy = lambda size: lib.dplr_lr_debug_copy(plan._h, dl._lib.BUF_SPECTRUM, ctypes.c_void_p(out.data_ptr()), size)
    assert copy(33) == dl._lib.E_INVALID
    assert copy(48) == dl._lib.OK
    torch.cuda.synchronize()
    assert torch.equal(out[:48], full[:48]) and not out[48:].any()
