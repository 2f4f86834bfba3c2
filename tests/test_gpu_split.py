"""The binary32 MFMA convolution's operands are split into two binary16 parts under
a power-of-two scale per sample and 32-channel chunk; these tests hold it to what
binary32 arithmetic gives where the split could go wrong: infinities and NaN (in
the signal and in the weights, through every epilogue), magnitudes far outside
binary16's range, neighbouring regions of very different magnitude, and the bits
of one window whatever lies around it."""
import numpy as np
import pytest

import oracle
from paper_1508_06904_amd import dss, workloads as wl
from tests.gpu_helpers import gpu_dense, log

pytestmark = pytest.mark.gpu

F32_TOL = 1e-4      # of max|oracle|, the bound of every binary32 comparison here

# (arch, channels, H, W, ndim): store epilogue (64- and 32-channel tiles), folded projection, 1-D pool,
# and a flat launch (many small fragments)
CASES = {
    "store_n64": ([("conv", 20, 64, 3, 3, "none"), ("conv", 64, 12, 1, 1, "none")], 20, 24, 30, 2),
    "store_tanh": ([("conv", 16, 36, 2, 3, "tanh")], 16, 20, 33, 2),
    "proj": ([("conv", 32, 72, 3, 2, "relu"), ("conv", 72, 3, 1, 1, "none")], 32, 21, 27, 2),
    "pool_1d": ([("conv", 16, 40, 1, 5, "relu"), ("pool", 1, 2), ("conv", 40, 2, 1, 3, "none")], 16, 1, 700, 1),
    "flat": ([("conv", 16, 32, 3, 3, "relu"), ("pool", 3, 3), ("conv", 32, 32, 3, 3, "none")], 16, 41, 44, 2),
}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    dss.lib()
    yield
    torch.cuda.synchronize()


def reference(w):
    """The dense output of the layers in binary32 torch on the CPU, which keeps infinities, NaN and ReLU(NaN) apart
    as a chain of binary32 sums does (relu here is fmax(x, 0): NaN gives 0, as on the GPU)."""
    import torch
    t = torch.from_numpy(w.x)
    dil = (1, 1)
    for l in w.layers:
        if l["kind"] == "maxpool":
            h, wd = t.shape[1] - dil[0] * (l["kh"] - 1), t.shape[2] - dil[1] * (l["kw"] - 1)
            m = None
            for a in range(l["kh"]):
                for b in range(l["kw"]):
                    v = t[:, a * dil[0]:a * dil[0] + h, b * dil[1]:b * dil[1] + wd]
                    m = v if m is None else torch.fmax(m, v)
            t, dil = m, (dil[0] * l["kh"], dil[1] * l["kw"])
            continue
        h, wd = t.shape[1] - dil[0] * (l["fh"] - 1), t.shape[2] - dil[1] * (l["fw"] - 1)
        wt = torch.from_numpy(l["weight"])
        out = torch.zeros((l["cout"], h, wd))
        for c in range(l["cin"]):          # products one by one: a product of 0 and an infinity is NaN
            for a in range(l["fh"]):
                for b in range(l["fw"]):
                    out = out + wt[:, c, a, b][:, None, None] * t[c, a * dil[0]:a * dil[0] + h, b * dil[1]:b * dil[1] + wd]
        out = out + torch.from_numpy(l["bias"])[:, None, None]
        t = torch.fmax(out, torch.zeros(())) if l["act"] == "relu" else torch.tanh(out) if l["act"] == "tanh" else out
    return t.numpy().astype(np.float64)


def check(got, ref, what):
    for name, f in (("nan", np.isnan), ("+inf", np.isposinf), ("-inf", np.isneginf)):
        np.testing.assert_array_equal(f(got), f(ref), err_msg="%s: %s" % (what, name))
    fin = np.isfinite(ref)
    if fin.any():
        err, scale = np.abs(got[fin] - ref[fin]).max(), np.abs(ref[fin]).max()
        log("  %s: %d of %d finite, ratio %.2e" % (what, fin.sum(), fin.size, err / max(scale, 1e-300)))
        assert err <= F32_TOL * scale, what


@pytest.mark.parametrize("where", ["signal", "weights"])
@pytest.mark.parametrize("case", list(CASES))
def test_non_finite_values(case, where):
    """Infinities of both signs and a NaN at scattered samples (or an infinite weight): the same outputs are NaN,
    +inf, -inf and finite as in binary32, and the finite ones are right."""
    arch, C, H, W, nd = CASES[case]
    w = wl.custom(arch, C, H, W, seed=61, ndim=nd, value_kind="normal")
    if where == "signal":
        rng = np.random.default_rng(7)
        for v in (np.inf, -np.inf, np.nan):
            w.x[rng.integers(0, C), rng.integers(0, H), rng.integers(0, W)] = v
    else:
        conv = w.layers[0]
        conv["weight"][3, 1, 0, 0] = np.inf
        conv["weight"][5, 0, -1, -1] = -np.inf
    out, _ = gpu_dense(w.layers, w.x, nd)
    check(out, reference(w), "%s %s" % (case, where))


@pytest.mark.parametrize("scale", [1e-30, 1e-12, 3e5, 1e18])
def test_magnitudes(scale):
    """A whole signal far outside binary16's range, and its weights the other way."""
    arch = [("conv", 32, 64, 3, 3, "none"), ("conv", 64, 16, 2, 2, "none")]
    w = wl.custom(arch, 32, 20, 40, seed=62, value_kind="normal")
    w.x *= np.float32(scale)
    for l in w.layers:
        l["bias"][:] = 0
    w.layers[0]["weight"] *= np.float32(min(1e12, max(1e-12, 1 / scale)))
    out, _ = gpu_dense(w.layers, w.x, 2)
    check(out, oracle.eval_stride(w.layers, w.x), "scale %g" % scale)


def test_neighbouring_magnitudes():
    """Columns of magnitude 1e10, 1 and 1e-10 side by side within one tile: windows inside one band are as precise as
    that band alone (a sample's scale is its own)."""
    arch = [("conv", 32, 64, 3, 3, "none"), ("conv", 64, 16, 1, 1, "none")]
    w = wl.custom(arch, 32, 20, 48, seed=63, value_kind="normal")
    for l in w.layers:
        l["bias"][:] = 0
    for k, s in enumerate((1e10, 1.0, 1e-10)):
        w.x[:, :, 16 * k:16 * k + 16] *= np.float32(s)
    out, _ = gpu_dense(w.layers, w.x, 2)
    ref = oracle.eval_stride(w.layers, w.x)
    for k in range(3):
        check(out[:, :, 16 * k:16 * k + 14], ref[:, :, 16 * k:16 * k + 14], "band %d" % k)


def test_bits_do_not_depend_on_the_surroundings():
    """A window's output bits are those of the window evaluated alone, with samples of 2^20 times its magnitude next
    to it in the same tile."""
    arch = [("conv", 32, 64, 5, 5, "relu"), ("conv", 64, 16, 2, 2, "none")]
    w = wl.custom(arch, 32, 26, 30, seed=64, value_kind="normal")
    inner = w.x[:, 4:20, 6:25].copy()
    w.x *= np.float32(2.0 ** 20)
    w.x[:, 4:20, 6:25] = inner
    out, _ = gpu_dense(w.layers, w.x, 2)
    alone, _ = gpu_dense(w.layers, np.ascontiguousarray(inner), 2)
    np.testing.assert_array_equal(out[:, 4:4 + alone.shape[1], 6:6 + alone.shape[2]], alone)


def _weight_gradient(x, G, fh, fw):
    """dW[o][i][a][b] = sum_p G[o][p] x[i][p + (a, b)] in 64 bits."""
    eh, ew = G.shape[1:]
    g = G.astype(np.float64).reshape(G.shape[0], -1)
    out = np.empty((G.shape[0], x.shape[0], fh, fw))
    for a in range(fh):
        for b in range(fw):
            out[:, :, a, b] = g @ x[:, a:a + eh, b:b + ew].astype(np.float64).reshape(x.shape[0], -1).T
    return out


# taps per group 1..7 (the kernel's instantiations, 8 in two groups of 4), channels past one 64-wide tile, several
# splits; "rising": magnitudes that grow by 1e8 along the signal after a zero start; "inf" / "nan": one such sample
@pytest.mark.parametrize("fw", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("data", ["plain", "rising", "inf", "nan"])
def test_weight_gradient_parts(fw, data):
    import torch
    cin, cout, fh, H, W = (68, 72, 2, 50, 61) if fw % 2 else (36, 64, 1, 70, 83)
    w = wl.custom([("conv", cin, cout, fh, fw, "none")], cin, H, W, seed=70 + fw, value_kind="normal")
    rng = np.random.default_rng(71)
    G = rng.standard_normal((cout, H - fh + 1, W - fw + 1)).astype(np.float32)
    if data == "rising":
        w.x *= np.geomspace(1e-4, 1e4, H, dtype=np.float32)[None, :, None]
        G *= np.geomspace(1e-5, 1e3, G.shape[1], dtype=np.float32)[None, :, None]
        w.x[:, :4] = 0
        G[:, :3] = 0
    if data in ("inf", "nan"):
        w.x[5, H // 2, W // 2] = np.inf if data == "inf" else np.nan
    plan = dss.Plan(w.layers, 2, cin)
    gw, gb, _ = plan.backward(torch.from_numpy(w.x).cuda(), torch.from_numpy(G).cuda(), with_signal_grad=False)
    torch.cuda.synchronize()
    got = plan.split_grads(gw, gb)[0][0].cpu().numpy().astype(np.float64)
    ref = _weight_gradient(w.x, G, fh, fw)
    check(got, ref, "dW fw %d %s" % (fw, data))
    db = G.astype(np.float64).sum((1, 2))
    assert np.abs(gb.cpu().numpy() - db).max() <= F32_TOL * max(np.abs(db).max(), np.abs(G).max())
