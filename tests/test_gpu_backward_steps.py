"""GPU parity of two backward kernels at their edges, on integer data that every summation order computes exactly
(all partial sums below 2^23, ties in the maxima decided by the shared first-maximum rule): the strip walk of the
2 x 2 pool's gradient (one to several strips of 16 rows, with remainders), and the one-pass backward of a 1x1 layer
to 1..4 outputs (channel counts of 1, 3, 9 and 33 quads of lanes, with and without the previous layer's ReLU)."""
import numpy as np
import pytest

import oracle
from oracle import backward as ob
from paper_1508_06904_amd import dss, workloads as wl
from tests.gpu_helpers import to_device
from tests.test_gpu_split import _weight_gradient, check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mid,cout,H,W,act", [(4, 1, 12, 30, "relu"), (12, 2, 18, 47, "none"), (36, 3, 35, 28, "relu"),
                                              (132, 4, 52, 23, "relu")])
def test_pool_and_narrow_backward(mid, cout, H, W, act):
    import torch
    arch = [("conv", 4, 8, 3, 3, "relu"), ("pool", 2, 2), ("conv", 8, mid, 2, 2, act), ("conv", mid, cout, 1, 1, "none")]
    w = wl.custom(arch, 4, H, W, seed=40 + mid, weight_kind="int", value_kind="int")
    B = oracle.receptive_field(w.layers)
    G = np.random.default_rng(41).integers(-1, 2, size=(cout, H - B[0] + 1, W - B[1] + 1)).astype(np.float64)
    ref = ob.dense_backward(w.layers, w.x, G)
    plan = dss.Plan(w.layers, 2, 4)
    gw, gb, gx = plan.backward(to_device(w.x, "f32"), to_device(G, "f32"))
    torch.cuda.synchronize()
    ws, bs = plan.split_grads(gw, gb)
    for a, b in zip(list(ws) + list(bs) + [gx], ref[0] + ref[1] + [ref[2]]):
        assert np.abs(b).max() < 2 ** 23
        np.testing.assert_array_equal(a.cpu().numpy().astype(np.float64), b)


# 20 and 32 input channels: half a tile of the weight gradient's bfloat16-part kernel, 1 to 7 taps a group
@pytest.mark.parametrize("cin", [20, 32])
@pytest.mark.parametrize("fw", [1, 2, 3, 4, 5, 6, 7])
def test_weight_gradient_half_tile(cin, fw):
    import torch
    w = wl.custom([("conv", cin, 68, 2, fw, "none")], cin, 45, 61, seed=50 + fw, value_kind="normal")
    G = np.random.default_rng(51).standard_normal((68, 44, 62 - fw)).astype(np.float32)
    plan = dss.Plan(w.layers, 2, cin)
    gw, gb, _ = plan.backward(torch.from_numpy(w.x).cuda(), torch.from_numpy(G).cuda(), with_signal_grad=False)
    torch.cuda.synchronize()
    got = plan.split_grads(gw, gb)[0][0].cpu().numpy().astype(np.float64)
    check(got, _weight_gradient(w.x, G, 2, fw), "dW %d channels fw %d" % (cin, fw))
