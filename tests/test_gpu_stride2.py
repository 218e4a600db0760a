"""Input gradients of strided blocks by classes of input pixels (fp32, and bf16
of whole 64-channel blocks) and by the gradient spread to the input grid (other
bf16 channel counts), against the oracle; and their sums that are not finite."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from gcpsl_inputs import get_config  # noqa: E402
from paper_2609_29395_amd import driver, gcpsl  # noqa: E402
from test_gpu_parity import check_run, matched_run  # noqa: E402

pytestmark = pytest.mark.gpu


# one output pixel per image, one row, one column; tiles that end inside an
# image; channel blocks 64, 128, 192 (tap loops of one to three blocks) and 8,
# 72, 136 (stages that span two taps in fp32); 8 to 136 inputs (few workgroups)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("H,W,B,C,w1,w2", [(2, 2, 5, 1, 8, 64), (2, 10, 7, 2, 64, 64), (6, 2, 9, 2, 72, 128), (12, 12, 5, 3, 136, 72),
                                           (10, 6, 11, 2, 24, 192), (8, 8, 9, 2, 128, 8)])
def test_round_against_the_oracle(dtype, H, W, B, C, w1, w2):
    layers = [("conv", 3, w1, False), ("gnorm", w1, w1 // 8), ("block", w1, w2, 2, w2 // 8), ("avgpool",),
              ("linear", w2, 4)]
    cfg = get_config("tiny", H=H, W=W, B=B, C=C, K=8 * C, N_ex=4 * max(C * B, 16), layers=layers, cut=2, momentum=0.9,
                     F=0, T=1, dtype=dtype)
    ctx, o, theta0, losses, _ = matched_run(cfg, 1)
    check_run(ctx, o, theta0, losses, cfg)


# fp32 tiles of many replicas: 129 output pixels end inside every tile, 72 and 40
# inputs inside the channel tiles, at the replica counts that just reach the 256
# workgroups of each tile's rule; one-tap weight gradients of 40 to 64 inputs
# (projections)
@pytest.mark.parametrize("C,w1,w2,dgrad,wgrad", [
    (128, 72, 24, "128x128,w8", "32x128,w4"), (128, 40, 24, "128x64,w4", "32x64,w4"), (2, 56, 136, "64x64,w4", "128x64,w4"),
    (2, 24, 40, "32x32,w4", "64x32,w4"), (3, 64, 64, "64x64,w4", "64x64,w4"),
])
def test_fp32_tiles_against_the_oracle(C, w1, w2, dgrad, wgrad):
    layers = [("conv", 3, w1, False), ("gnorm", w1, w1 // 8), ("block", w1, w2, 2, w2 // 8), ("avgpool",),
              ("linear", w2, 4)]
    cfg = get_config("tiny", H=6, W=86, B=1, C=C, K=8 * C, N_ex=32 * C, layers=layers, cut=2, momentum=0.9, F=0, T=1,
                     rule="size")
    ctx, o, theta0, losses, _ = matched_run(cfg, 1)
    check_run(ctx, o, theta0, losses, cfg)
    ctx, _ = driver.setup(cfg, max_steps=1)
    ctx.timing(True)
    ctx.sample(0)
    ctx.step(0)
    ran = set(ctx.timing_read())
    assert {f"conv_dgrad<f32,{dgrad},stride2,split>", f"conv_wgrad<f32,{wgrad},split>"} <= ran, ran


def test_products_that_overflow_pass_as_in_fp32():
    """Weights of 1e38 from one input channel of a strided block (and of its
    projection) to one output channel: the products of the input gradient
    overflow one by one, and of a class of several taps the first to do so decides
    (a chain of FMAs stays at its first infinity; the split's terms of both signs
    would meet as NaN).  Checked against such chains in float64 from the GPU's own
    output gradients, shortcut gradient and mask."""
    side, w1, w2, B = 10, 24, 40, 3
    layers = [("conv", 3, w1, False), ("gnorm", w1, 3), ("block", w1, w2, 2, 5), ("avgpool",), ("linear", w2, 4)]
    rng = np.random.default_rng(6)
    sizes = [(w1, 3, 3, 3), (w1,), (w1,), (w1,), (w2, 3, 3, w1), (w2,), (w2,), (w2,), (w2, 3, 3, w2), (w2,), (w2,), (w2,),
             (w2, w1), (w2,), (w2,), (w2,), (4, w2), (4,)]
    th = [rng.uniform(-0.3, 0.3, s).astype(np.float32) for s in sizes]
    for i in (2, 6, 10, 14):  # norms
        th[i][:], th[i + 1][:] = 1, 0
    k, co, kp, cop = 4, 7, 17, 9
    for ch in (k, kp):  # the input channels of the huge weights are tiny, but pass the ReLU
        th[2][ch], th[3][ch] = 1e-31, 3e-31
    th[4][..., k], th[12][:, kp] = 0, 0
    th[4][co, :, :, k], th[12][cop, kp] = 1e38, 1e38
    th[16] *= np.float32(1e13)  # large gradients
    images = rng.standard_normal((B, side, side, 3)).astype(np.float32)
    cfg = dict(K=1, C=1, B=B, L=4, H=side, W=side, Cin=3, N_ex=B, layers=layers, cut=2, dtype="f32", lr=0.0, momentum=0.0,
               seed=0)
    ctx = gcpsl.Context(cfg, images, np.zeros(B, np.int32), np.zeros(B, np.int32), np.zeros(1, np.int32),
                        np.concatenate([t.reshape(-1) for t in th]), max_steps=1)
    ctx.sample(0)
    ctx.step(0)
    torch.cuda.synchronize()
    h = side // 2

    def get(name, hw, ch):
        return ctx.tensor(name).cpu().numpy().reshape(B, hw, hw, ch).astype(np.float64)

    act, dz1, dzp = get("act1", side, w1), get("dz2.1", h, w2), get("dz2.p", h, w2)
    gsc, got = get("gsc2", side, w1), get("gpre1", side, w1)
    top = float(np.finfo(np.float32).max)

    def add(acc, g, w):  # one tap (of the huge channels, one product)
        v = acc + (g[..., None] * w.astype(np.float64)).sum(3)
        return np.where(np.isinf(acc), acc, np.where(np.abs(v) > top, np.sign(v) * np.inf, v))

    proj, conv = np.zeros((B, side, side, w1)), np.zeros((B, side + 2, side + 2, w1))
    proj[:, ::2, ::2] = add(proj[:, ::2, ::2], dzp, th[12])
    for r in (2, 1, 0):  # output pixel i takes input rows 2 i + r - 1: taps by ascending output pixel
        for s in (2, 1, 0):
            conv[:, r:r + side:2, s:s + side:2] = add(conv[:, r:r + side:2, s:s + side:2], dz1, th[4][:, r, s])
    want = np.where(act > 0, conv[:, 1:-1, 1:-1] + gsc, 0.0)
    # (a sum near the end of the fp32 range, which its order could decide, is not to be here)
    for got_, want_ in ((gsc, proj), (got, want)):
        assert not ((np.abs(want_) > top / 100) & np.isfinite(want_)).any()
        assert not np.isnan(got_).any() and np.array_equal(np.isposinf(got_), np.isposinf(want_))
        assert np.array_equal(np.isneginf(got_), np.isneginf(want_))
        fin = np.isfinite(want_)
        assert np.abs(got_[fin] - want_[fin]).max() <= 1e-5 * np.abs(want_[fin]).max()
    assert np.isinf(gsc[..., kp]).any() and np.isinf(got[:, 1::2, 1::2, k]).any()
