"""The grid of a persistent batch launch leaves room on the chip: its barrier
needs every workgroup resident, so it stays a workgroup a CU (or a CU per XCD)
below what the kernel's registers allow, and no larger than the batch's work."""
import pytest

from kernel_resources import find, kernels, wavefronts
from paper_1608_04118_amd import inputs as I

pytestmark = pytest.mark.gpu

CUS, XCDS = 256, 8
FORMS = {"f64": (I.FP64, "dd"), "f32sr": (I.FP32SR, "fd"), "f16s": (I.FP16S, "DF16_f"), "f32": (I.FP32, None)}


@pytest.fixture(scope="module")
def B():
    torch = pytest.importorskip("torch")
    assert torch.cuda.is_available()
    from paper_1608_04118_amd import binding
    return binding


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("fields", [0, 1, 2, 3])
def test_grid_leaves_room(B, form, fields):
    import numpy as np
    precision, args = FORMS[form]
    table = kernels(B.LIB_PATH)
    if form == "f32":  # pairs of steps, workgroups of eight wavefronts
        per_cu = wavefronts(find(table, "batch2p_kernel", "Li%dE" % fields)) // 2
    else:  # of four
        per_cu = wavefronts(find(table, "batch_kernel", args + "Li%dE" % fields))
    most = (per_cu - 1) * CUS if per_cu > 1 else CUS - XCDS
    ps = [I.cavity_small(nx=512, ny=512, precision=precision) for _ in range(9)]
    f = np.full((512, 512), 0.5)
    b = B.Batch(ps, phi_fields=[f if fields & 1 else None] * 9, Hv_fields=[f if fields & 2 else None] * 9)
    info = b.info()
    b.close()
    assert info["tiles"] > per_cu * CUS
    assert info["grid"] == most


@pytest.mark.parametrize("form", FORMS)
def test_grid_no_larger_than_the_work(B, form):
    b = B.Batch([I.cavity_small(nx=66, ny=67, precision=FORMS[form][0])])
    info = b.info()
    b.close()
    assert info["tiles"] <= info["grid"] < info["tiles"] + XCDS
