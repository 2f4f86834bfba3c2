"""binary32 layers whose channels differ in magnitude by up to 2^98: every output channel is held to the rounding of
its own sum, |error| <= bound * sum |w| |x| of that output, against 64 bits.  The bound is that of the arithmetic:
operands of 22 bits and a dropped product of two low parts (3 2^-22), what an uncertified sum may lack (sqrt(K) 2^-24), and
roundings of K binary32 additions as a random walk (2 sqrt(K) 2^-24)."""
import numpy as np
import pytest

from paper_1508_06904_amd import dss, workloads as wl
from tests.gpu_helpers import log, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    dss.lib()
    yield
    torch.cuda.synchronize()


def bound(K):
    return 3 * 2.0 ** -22 + 3 * K ** 0.5 * 2.0 ** -24


def evaluate(layers, x):
    """The dense output in 64 bits, and the same sums over magnitudes (stride 1; pools as sliding maxima, whose error
    is at most the largest of their inputs')."""
    import torch
    import torch.nn.functional as F
    t = torch.from_numpy(x).double()[None]
    m, dil, K = t.abs(), (1, 1), 0
    for l in layers:
        if l["kind"] == "maxpool":
            def pool(v):
                h, w = v.shape[2] - dil[0] * (l["kh"] - 1), v.shape[3] - dil[1] * (l["kw"] - 1)
                return torch.stack([v[:, :, a * dil[0]:a * dil[0] + h, b * dil[1]:b * dil[1] + w]
                                    for a in range(l["kh"]) for b in range(l["kw"])]).amax(0)
            t, m, dil = pool(t), pool(m), (dil[0] * l["kh"], dil[1] * l["kw"])
            continue
        w = torch.from_numpy(l["weight"]).double()
        t = F.conv2d(t, w, torch.from_numpy(l["bias"]).double(), dilation=dil)
        m = F.conv2d(m, w.abs(), torch.from_numpy(l["bias"]).double().abs(), dilation=dil)
        K += l["cin"] * l["fh"] * l["fw"]
        if l["act"] == "relu":
            t = t.clamp(min=0)
    return t[0].numpy(), m[0].numpy(), K


def check(got, ref, mag, K, what):
    assert got.shape == ref.shape
    assert np.isfinite(got).all(), what
    err = np.abs(got - ref) / np.maximum(mag, 1e-300)
    log("  %s: %.2e of the sum of magnitudes, bound %.2e" % (what, err.max(), bound(K)))
    assert err.max() <= bound(K), what


# (arch, channels, H, W, ndim): 128-, 64- and 32-channel tiles, folded projection, 1-D pool, flat launch
CASES = {
    "n128": ([("conv", 36, 144, 3, 3, "none")], 36, 24, 40, 2),
    "n64": ([("conv", 32, 72, 5, 5, "none")], 32, 21, 37, 2),
    "n32": ([("conv", 20, 36, 1, 1, "none")], 20, 20, 33, 2),
    "proj": ([("conv", 32, 72, 3, 2, "relu"), ("conv", 72, 3, 1, 1, "none")], 32, 21, 27, 2),
    "pool_1d": ([("conv", 16, 40, 1, 5, "relu"), ("pool", 1, 2)], 16, 1, 700, 1),
    "flat": ([("conv", 16, 32, 3, 3, "relu"), ("pool", 3, 3), ("conv", 32, 32, 3, 3, "none")], 16, 41, 44, 2),
}


def make(case, seed):
    arch, C, H, W, nd = CASES[case]
    w = wl.custom(arch, C, H, W, seed=seed, ndim=nd, value_kind="normal")
    for l in w.layers:
        if l["kind"] == "conv":
            l["bias"][:] = 0
    return w, nd


def fashions(w, nd):
    """The dense and the dilated evaluation, whose bits agree."""
    import torch
    plan = dss.Plan(w.layers, nd, w.x.shape[0])
    x = to_device(w.x, "f32")
    dense, dil = plan.eval_dense(x), plan.eval_dilate(x)
    torch.cuda.synchronize()
    assert torch.equal(dense, dil)
    return dense.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("case", list(CASES))
def test_output_channels_of_different_magnitude(case):
    """Filters of 1, 2^-14, ... 2^-98; a following projection weighs them the other way."""
    w, nd = make(case, 80)
    e = 2.0 ** (-14.0 * (np.arange(w.layers[-1]["cout"] if case == "flat" else w.layers[0]["cout"]) % 8))
    if case == "proj":
        w.layers[1]["weight"] /= e[None, :, None, None].astype(np.float32)
    l = w.layers[-1] if case == "flat" else w.layers[0]
    l["weight"] *= e[:, None, None, None].astype(np.float32)
    check(fashions(w, nd), *evaluate(w.layers, w.x), case)


def test_zero_and_small_filters_beside_huge_ones():
    """Samples of 2^110 under filters of 2^60 overflow; those of 0 and 2^-60 in the same layer do not."""
    w, nd = make("n64", 81)
    w.x *= np.float32(2.0 ** 110)
    w.layers[0]["weight"][0] *= np.float32(2.0 ** 60)
    w.layers[0]["weight"][1] = 0
    w.layers[0]["weight"][2:] *= np.float32(2.0 ** -60)
    import torch
    plan = dss.Plan(w.layers, nd, w.x.shape[0])
    got = plan.eval_dense(to_device(w.x, "f32")).cpu().numpy().astype(np.float64)
    torch.cuda.synchronize()
    ref, mag, K = evaluate(w.layers, w.x)
    assert (got[1] == 0).all()
    check(got[2:], ref[2:], mag[2:], K, "2^-60")


def test_input_gradient_of_different_channels():
    """The signal's gradient where the filters' input channels differ."""
    import torch
    w, nd = make("n64", 82)
    e = 2.0 ** (-14.0 * (np.arange(32) % 8))
    w.layers[0]["weight"] *= e[None, :, None, None].astype(np.float32)
    G = np.random.default_rng(83).standard_normal((72, 17, 33)).astype(np.float32)
    plan = dss.Plan(w.layers, nd, 32)
    _, _, gx = plan.backward(to_device(w.x, "f32"), to_device(G, "f32"))
    torch.cuda.synchronize()
    flipped = [{"kind": "conv", "cin": 72, "cout": 32, "fh": 5, "fw": 5, "act": "none", "bias": np.zeros(32, np.float32),
                "weight": np.ascontiguousarray(w.layers[0]["weight"].transpose(1, 0, 2, 3)[:, :, ::-1, ::-1])}]
    check(gx.cpu().numpy().astype(np.float64), *evaluate(flipped, np.pad(G, ((0, 0), (4, 4), (4, 4)))), "signal gradient")


# one channel 2^r times the others under weights 2^-r; channels in two groups that no filter sees together; a signal of
# magnitudes 2^-130 .. 2^-90 (subnormal numbers among them) under weights of 2^100; channels of random magnitude; the
# two groups 2^170 apart (products with the scale underflow); a silent channel with weights of 2^40 in a signal of 2^-90
@pytest.mark.parametrize("data", ["r12", "r16", "r20", "r24", "r30", "r36", "r41", "r60", "groups", "tiny", "mixed", "far", "unused"])
@pytest.mark.parametrize("case", list(CASES))
def test_input_channels_of_different_magnitude(case, data):
    w, nd = make(case, 84)
    rng = np.random.default_rng(85)
    conv = w.layers[0]
    if data[0] == "r":
        r = int(data[1:])
        ch = rng.integers(0, conv["cin"])
        w.x[ch] *= np.float32(2.0 ** r)
        conv["weight"][:, ch] *= np.float32(2.0 ** -r)
    elif data == "groups":
        a = np.arange(conv["cin"]) % 2 == 0
        w.x[a] *= np.float32(2.0 ** 34)
        for n in range(conv["cout"]):
            conv["weight"][n, a == (n % 2 == 0)] = 0
    elif data == "far":
        a = np.arange(conv["cin"]) % 2 == 0
        w.x[a] *= np.float32(2.0 ** 110)
        w.x[~a] *= np.float32(2.0 ** -60)
        for n in range(conv["cout"]):
            conv["weight"][n, a == (n % 2 == 0)] = 0
    elif data == "unused":
        ch = rng.integers(0, conv["cin"])
        w.x *= np.float32(2.0 ** -90)
        w.x[ch] = 0
        conv["weight"][:, ch] *= np.float32(2.0 ** 40)
    elif data == "tiny":
        w.x *= (2.0 ** rng.uniform(-130, -90, size=w.x.shape)).astype(np.float32)
        conv["weight"] *= np.float32(2.0 ** 100)
    else:
        e = 2.0 ** rng.integers(-30, 31, size=conv["cin"])
        w.x *= e[:, None, None].astype(np.float32)
        conv["weight"] /= e[None, :, None, None].astype(np.float32)
    check(fashions(w, nd), *evaluate(w.layers, w.x), "%s %s" % (case, data))


def test_signal_gradient_of_different_output_channels():
    """The input gradient's operand is the upstream gradient: its channels differ, the filters the other way."""
    import torch
    w, nd = make("n64", 86)
    e = 2.0 ** np.random.default_rng(87).integers(-30, 31, size=72)
    w.layers[0]["weight"] /= e[:, None, None, None].astype(np.float32)
    G = np.random.default_rng(88).standard_normal((72, 17, 33)).astype(np.float32) * e[:, None, None].astype(np.float32)
    plan = dss.Plan(w.layers, nd, 32)
    _, _, gx = plan.backward(to_device(w.x, "f32"), to_device(G, "f32"))
    torch.cuda.synchronize()
    flipped = [{"kind": "conv", "cin": 72, "cout": 32, "fh": 5, "fw": 5, "act": "none", "bias": np.zeros(32, np.float32),
                "weight": np.ascontiguousarray(w.layers[0]["weight"].transpose(1, 0, 2, 3)[:, :, ::-1, ::-1])}]
    check(gx.cpu().numpy().astype(np.float64), *evaluate(flipped, np.pad(G, ((0, 0), (4, 4), (4, 4)))), "signal gradient")


# what the weight gradient's operands are made of: channels of x, of dy or of both 2^-30 .. 2^30 apart; single samples
# of 2^40; dead channels beside live ones; magnitudes whose scales overflow one after the other; a signal that starts
# 2^-75 of what it becomes in some of its channels
@pytest.mark.parametrize("data", ["x", "dy", "both", "hot", "dead", "far", "start"])
@pytest.mark.parametrize("fw", [1, 3, 4, 7])
def test_weight_gradient_of_different_channels(fw, data):
    import torch
    from tests.test_gpu_split import _weight_gradient
    cin, cout, fh, H, W = (68, 72, 2, 50, 61) if fw % 2 else (36, 64, 1, 70, 83)
    w = wl.custom([("conv", cin, cout, fh, fw, "none")], cin, H, W, seed=90 + fw, value_kind="normal")
    rng = np.random.default_rng(91)
    x, G = w.x, rng.standard_normal((cout, H - fh + 1, W - fw + 1)).astype(np.float32)
    if data in ("x", "both"):
        x *= (2.0 ** rng.integers(-30, 31, size=cin))[:, None, None].astype(np.float32)
    if data in ("dy", "both"):
        G *= (2.0 ** rng.integers(-30, 31, size=cout))[:, None, None].astype(np.float32)
    if data == "hot":
        x[3, H // 2, W // 3] *= np.float32(2.0 ** 40)
        G[5, H // 3, W // 2] *= np.float32(2.0 ** 40)
    if data == "dead":
        x[rng.integers(0, cin, 8)] = 0
        G[rng.integers(0, cout, 8)] = 0
        G *= rng.integers(0, 2, size=G.shape)
    if data == "far":
        x *= np.float32(2.0 ** -100)
        G *= np.float32(2.0 ** 120)
    if data == "start":
        x[:, :H // 2] *= np.float32(2.0 ** -75)
        x[::2, H // 2:] = 0
    plan = dss.Plan(w.layers, 2, cin)
    gw, gb, _ = plan.backward(to_device(x, "f32"), to_device(G, "f32"), with_signal_grad=False)
    torch.cuda.synchronize()
    got = plan.split_grads(gw, gb)[0][0].cpu().numpy().astype(np.float64)
    mag = _weight_gradient(np.abs(x), np.abs(G), fh, fw)
    check(got, _weight_gradient(x, G, fh, fw), mag, G[0].size, "dW fw %d %s" % (fw, data))
    if data == "dead":
        assert (got[mag == 0] == 0).all()
