"""One-row layers with a pool whose filters are too wide (or too tall) for the pooled
epilogue's halo: around the last width that fits, far past it, and with filters of
several rows.  Dense against the oracle and against the dilated evaluation, which
never pools in the epilogue."""
import numpy as np
import pytest

import oracle
from paper_1508_06904_amd import dss, workloads as wl
from tests.gpu_helpers import assert_close, log, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    dss.lib()
    yield
    torch.cuda.synchronize()


# filter rows and columns, whether the pool runs in the epilogue (255 + fw halo samples a row, at most 498)
@pytest.mark.parametrize("fh,fw,pooled", [(1, 243, True), (1, 244, False), (1, 245, False), (1, 500, False), (1, 564, False),
                                          (2, 9, False), (3, 5, False)])
def test_wide_row_filter_before_a_pool(fh, fw, pooled):
    import torch
    nd = 1 if fh == 1 else 2
    arch = [("conv", 16, 32, fh, fw, "relu"), ("pool", 1, 2), ("conv", 32, 2, 1, 3, "none")]
    w = wl.custom(arch, 16, fh, 20 * 255 + fw - 1, seed=90 + fw, ndim=nd, value_kind="normal")
    plan = dss.Plan(w.layers, nd, 16)
    x = to_device(w.x, "f32")
    plan.set_timing(True)
    got = plan.eval_dense(x)
    names = [r["kernel"] for r in plan.timings()]
    plan.set_timing(False)
    log("%dx%d: %s" % (fh, fw, names))
    assert any(n.endswith("_pool") for n in names) == pooled
    dil = plan.eval_dilate(x)
    torch.cuda.synchronize()
    assert torch.equal(got, dil)
    assert_close(got.cpu().numpy().astype(np.float64), oracle.eval_stride(w.layers, w.x), 1e-4, "%dx%d" % (fh, fw))
