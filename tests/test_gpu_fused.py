"""The dense evaluation of a small network in one launch: every output against the
oracle and bit for bit against the dilated evaluation (separate launches of the
same sums), on grids around the edges of its tiles and on networks that reach
each form of its loops."""
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


# (arch, channels, ndim): 1, 2, 4, 8 and 16 output channels a thread, input channels in fours and not, pools of 2 and
# 3 rows or columns, a pool first, two pools, a layer without a pool, the last layer pooled; 1-D, which stays on its launches
NETS = {
    "tanh_small": (wl.arch_c1(), 1, 2),
    "sixteen": ([("conv", 3, 16, 3, 3, "relu"), ("pool", 2, 3), ("conv", 16, 12, 1, 1, "none")], 3, 2),   # 16 inputs: not the plain direct kernel
    "cob16": ([("conv", 3, 16, 3, 3, "relu"), ("pool", 2, 3)], 3, 2),
    "pool_first": ([("pool", 2, 2), ("conv", 2, 5, 3, 2, "relu"), ("pool", 3, 1), ("pool", 1, 2),
                    ("conv", 5, 2, 2, 2, "tanh")], 2, 2),
    "last_pooled": ([("conv", 4, 8, 2, 2, "relu"), ("conv", 8, 3, 3, 3, "relu"), ("pool", 2, 2)], 4, 2),
    "one_row": ([("conv", 1, 8, 1, 9, "relu"), ("pool", 1, 2), ("conv", 8, 1, 1, 5, "none")], 1, 1),
}
OUT = [(1, 1), (3, 4), (4, 5), (8, 9), (16, 17), (33, 31), (70, 65)]


@pytest.mark.parametrize("out", OUT, ids=["%dx%d" % o for o in OUT])
@pytest.mark.parametrize("net", list(NETS))
def test_fused_chain(net, out):
    import torch
    arch, C, nd = NETS[net]
    B = oracle.receptive_field(wl.custom(arch, C, 1, 1, seed=1, ndim=nd).layers)
    H, W = (1, B[1] + 16 * out[1] - 1) if nd == 1 else (B[0] + out[0] - 1, B[1] + out[1] - 1)
    w = wl.custom(arch, C, H, W, seed=81, ndim=nd, value_kind="normal")
    plan = dss.Plan(w.layers, nd, C)
    x = to_device(w.x, "f32")
    plan.set_timing(True)
    got = plan.eval_dense(x)
    names = [r["kernel"] for r in plan.timings()]
    plan.set_timing(False)
    log("%s %dx%d: %s" % (net, H, W, names))
    assert (names == ["dense_fused"]) == (net not in ("sixteen", "one_row"))
    dil = plan.eval_dilate(x)
    torch.cuda.synchronize()
    assert torch.equal(got, dil)
    assert_close(got.cpu().numpy().astype(np.float64), oracle.eval_stride(w.layers, w.x), 1e-4, net)


@pytest.mark.parametrize("size", [(64, 64), (150, 300), (400, 400), (900, 700)])
def test_fused_chain_tile_choice(size):
    """Each tile size of the small-image network, and the separate launches past them: the same bits."""
    import torch
    w = wl.make("c1_64x64", H=size[0], W=size[1])
    plan = dss.Plan.from_workload(w)
    x = to_device(w.x, "f32")
    got, dil = plan.eval_dense(x), plan.eval_dilate(x)
    torch.cuda.synchronize()
    assert torch.equal(got, dil)


# calls on either side of the rule (both ways measured: one launch / separate launches in us)
@pytest.mark.parametrize("arch,C,H,W,fused", [
    ([("conv", 12, 3, 3, "relu")] + [("conv", 12, 3, 3, "relu")] * 2 + [("pool", 2, 2), ("conv", 2, 3, 3, "none")], 1, 150, 150,
     True),      # 35 / 48
    ([("conv", 12, 3, 3, "relu")] + [("conv", 12, 3, 3, "relu")] * 2 + [("pool", 2, 2), ("conv", 2, 3, 3, "none")], 1, 200, 320,
     False),     # 68 / 58
    ([("conv", 14, 11, 11, "relu"), ("conv", 1, 5, 5, "none")], 3, 200, 320, True),      # 70 (tiles of 16; 138 of 8) / 92
    ([("conv", 8, 5, 5, "relu")] * 3, 4, 600, 800, False),                               # 172 / 113
])
def test_fused_chain_is_taken_where_it_is_faster(arch, C, H, W, fused):
    import torch
    layers, cin = [], C
    for s in arch:
        layers.append(("conv", cin) + s[1:] if s[0] == "conv" else s)
        cin = s[1] if s[0] == "conv" else cin
    w = wl.custom(layers, C, H, W, seed=82, value_kind="normal")
    plan = dss.Plan(w.layers, 2, C)
    x = to_device(w.x, "f32")
    plan.set_timing(True)
    got = plan.eval_dense(x)
    names = [r["kernel"] for r in plan.timings()]
    plan.set_timing(False)
    dil = plan.eval_dilate(x)
    torch.cuda.synchronize()
    assert (names == ["dense_fused"]) == fused
    assert torch.equal(got, dil)
