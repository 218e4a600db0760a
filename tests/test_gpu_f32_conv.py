"""The fp32 convolutions on the bf16 matrix cores (k_conv_f32.hip): every tile
and both stagings at the sizes where they can go wrong, against the oracle,
and sums with operands that have no finite three-way split, in every pass."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from gcpsl_inputs import get_config  # noqa: E402
from paper_2609_29395_amd import driver, gcpsl  # noqa: E402
from test_gpu_parity import check_run, matched_run  # noqa: E402

pytestmark = pytest.mark.gpu


def _net(w1, w2, w3, classes=4):
    return [("conv", 3, w1, False), ("conv", w1, w2, False), ("conv", w2, w3, False), ("conv", w3, w3, True),
            ("avgpool",), ("linear", w3, classes)]


# image side (W beside the halo kernels' 32-pixel limit), batch and widths:
# 8 and 24 channels (per-tap staging), 32 and 40 (halo, a ragged second
# block), 64 / 72 / 136 (tile edges in N); M tails of every tile; enough
# workgroups for the 256- and 128-pixel tiles, and too few
@pytest.mark.parametrize("side,B,C,widths", [
    (4, 3, 2, (8, 32, 40)), (4, 24, 2, (32, 136, 72)), (5, 7, 3, (24, 40, 64)), (7, 5, 1, (40, 72, 136)),
    (16, 9, 2, (32, 64, 136)), (32, 3, 1, (32, 64, 32)), (33, 2, 2, (32, 40, 8)), (16, 64, 4, (8, 32, 128)),
])
def test_round_against_the_oracle(side, B, C, widths):
    cfg = get_config("tiny", H=side, W=side, B=B, C=C, K=8 * C, N_ex=4 * max(C * B, 16), layers=_net(*widths), cut=2,
                     momentum=0.9, F=0, T=1)
    ctx, o, theta0, losses, _ = matched_run(cfg, 1)
    check_run(ctx, o, theta0, losses, cfg)


# Tiles of many replicas: 288 pixels end inside every tile, 72, 40 and 24 channels
# inside the channel tiles and (flat: per-tap staging) the k stages, at the replica
# counts that just reach the 256 workgroups of each tile's rule
@pytest.mark.parametrize("C,widths,fwd,dgrad,wgrad", [
    (128, (32, 72, 32), ["256x128,w8,halo", "256x32,w8,halo"], ["256x128,w8,halo", "256x32,w8,halo"], ["64x288,w4,halo"]),
    (64, (32, 72, 32), ["128x64,w8,halo", "64x32,w4,halo"], ["128x64,w8,halo", "64x32,w4,halo"], ["64x288,w4,halo"]),
    (32, (32, 72, 32), ["64x64,w4,halo"], ["64x64,w4,halo"], ["32x32,w4"]),
    (86, (24, 72, 24), ["128x128,w8", "128x32,w4"], ["128x128,w8", "128x32,w4"], ["32x128,w4"]),
    (86, (24, 40, 24), ["128x64,w4"], ["128x64,w4"], ["32x32,w4"]),
    (2, (136, 8, 136), ["64x64,w4", "64x32,w4,halo"], ["32x64,w4,halo", "64x64,w4"], ["128x32,w4", "128x128,w4"]),
    (2, (40, 24, 8), ["32x32,w4"], ["32x32,w4", "64x64,w4"], ["64x32,w4", "32x128,w4"]),
])
def test_every_tile_against_the_oracle(C, widths, fwd, dgrad, wgrad):
    cfg = get_config("tiny", H=6, W=6, B=8, C=C, K=8 * C, N_ex=128 * C, layers=_net(*widths), cut=2, momentum=0.9,
                     F=0, T=1, rule="size")
    ctx, o, theta0, losses, _ = matched_run(cfg, 1)
    check_run(ctx, o, theta0, losses, cfg)
    # the tiles the rows are for
    ctx, _ = driver.setup(cfg, max_steps=1)
    ctx.timing(True)
    ctx.sample(0)
    ctx.step(0)
    ran = set(ctx.timing_read())
    want = {f"conv_{k}<f32,{t},split>" for k, ts in (("fwd", fwd), ("dgrad", dgrad), ("wgrad", wgrad)) for t in ts}
    assert want <= ran, (want - ran, ran)


def _round(images, layers, side, change=None, labels=None):
    """One round of one cluster on `images` (all of them, one batch): the convs'
    outputs, grad, the batch's example order, labels, parameters and the
    gradients at the convs' sums."""
    B = len(images)
    rng = np.random.default_rng(3)
    labels = rng.integers(0, 4, B).astype(np.int32) if labels is None else labels
    shapes = []
    for s in layers:
        if s[0] == "conv":
            shapes += [(s[2], 3, 3, s[1]), (s[2],)]
        elif s[0] == "linear":
            shapes += [(s[2], s[1]), (s[2],)]
    theta = [rng.uniform(-0.3, 0.3, s).astype(np.float32) for s in shapes]
    if change:
        change(theta)
    cfg = dict(K=1, C=1, B=B, L=4, H=side, W=side, Cin=3, N_ex=B, layers=layers, cut=1, dtype="f32", lr=0.0,
               momentum=0.0, seed=0)
    ctx = gcpsl.Context(cfg, images, labels, np.zeros(B, np.int32), np.zeros(1, np.int32),
                        np.concatenate([t.reshape(-1) for t in theta]), max_steps=1)
    ctx.sample(0)
    ctx.step(0)
    torch.cuda.synchronize()
    idx = ctx.tensor("idx").cpu().numpy()
    convs = [i for i, s in enumerate(layers) if s[0] == "conv"]
    acts, gpre = ([ctx.tensor(f"{n}{i}").cpu().numpy().reshape(B, side, side, -1) for i in convs]
                  for n in ("act", "gpre"))
    return acts, ctx.tensor("grad").cpu().numpy(), idx, labels, theta, gpre


def _conv(x, w, b):
    """ReLU(conv) in float64 (a product of an infinity and a padding zero is
    NaN, as on the GPU, and ReLU turns NaN into 0)."""
    n, h, ww, c = x.shape
    p = np.zeros((n, h + 2, ww + 2, c))
    p[:, 1:-1, 1:-1] = x
    with np.errstate(invalid="ignore", over="ignore"):
        z = sum(p[:, r:r + h, s:s + ww, None, :] * w[:, r, s].astype(np.float64) for r in range(3) for s in range(3))
        z = z.sum(-1) + b
    return np.where(z > 0, z, 0.0)


LAYERS = [("conv", 3, 40, False), ("conv", 40, 40, False), ("avgpool",), ("linear", 40, 4)]


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_infinities_and_nan_pass_as_in_fp32(value):
    """An infinity has no finite split: the tiles that hold one are summed in
    plain fp32 (image layer: per-tap staging; second layer: halo staging)."""
    side = 8
    images = np.random.default_rng(1).standard_normal((6, side, side, 3)).astype(np.float32)
    images[2, 3, 4, 1] = value
    (a0, a1), _, idx, _, th, _ = _round(images, LAYERS, side)
    w0 = _conv(images[idx].astype(np.float64), th[0], th[1])
    # the second layer from the GPU's own first one
    w1 = _conv(a0.astype(np.float64), th[2], th[3])
    for got, want in ((a0, w0), (a1, w1)):
        inf = np.isinf(want)
        assert np.array_equal(np.isinf(got), inf) and not np.isnan(got).any()
        assert np.allclose(got[~inf], want[~inf], rtol=1e-5, atol=1e-5)
    assert np.isinf(a0).any() == (not np.isnan(value))


def test_values_that_round_to_infinity_in_bf16():
    """Finite fp32 values above the largest bf16 (their first part rounds to
    infinity) as image, as activation and in the weight gradient: everything
    stays finite and right."""
    side, big = 8, np.float32(3.4e38)
    images = np.random.default_rng(2).standard_normal((6, side, side, 3)).astype(np.float32)
    images[1, 2, 2, 0] = big

    def change(th):  # the pixel passes the first layer nearly unscaled; the second and the head scale it down
        th[0][::2, 1, 1, 0] = 0.9999
        th[2] *= np.float32(1e-30)
        th[4] *= np.float32(1e-7)

    (a0, a1), grad, idx, labels, th, _ = _round(images, LAYERS, side, change)
    assert np.isfinite(a0).all() and np.isfinite(a1).all() and a0.max() > 3.39e38
    assert np.allclose(a0, _conv(images[idx].astype(np.float64), th[0], th[1]), rtol=1e-5, atol=1e-5)
    # (360 products of up to 3.4e8 cancel: an element's bound is 360 x 2^-24 of their magnitude)
    w1 = _conv(a0.astype(np.float64), th[2], th[3])
    assert np.abs(a1 - w1).max() <= 360 * 2.0**-24 * 3.4e8 and np.linalg.norm(a1 - w1) <= 1e-6 * np.linalg.norm(w1)
    # dW of the second conv from the GPU's own activations
    z = a1.astype(np.float64).mean((1, 2)) @ th[4].astype(np.float64).T + th[5]
    p = np.exp(z - z.max(1, keepdims=True))
    p /= p.sum(1, keepdims=True)
    p[np.arange(6), labels[idx]] -= 1
    g = (p / 6 @ th[4])[:, None, None] / side**2 * (a1 > 0)
    pad = np.zeros((6, side + 2, side + 2, 40))
    pad[:, 1:-1, 1:-1] = a0
    want = np.stack([[np.einsum("nhwo,nhwc->oc", g, pad[:, r:r + side, s:s + side]) for s in range(3)]
                     for r in range(3)])  # [r][s][co][ci]
    o = th[0].size + th[1].size
    got = grad[o:o + th[2].size].reshape(40, 3, 3, 40).transpose(1, 2, 0, 3)
    assert np.isfinite(got).all() and np.abs(want).max() > 1e25
    assert np.linalg.norm((got - want) / 1e25) <= 1e-4 * np.linalg.norm(want / 1e25)


def test_sums_of_large_terms_that_cancel():
    """Operands just below 2^60: the second layer's positive terms (its first 32
    input channels, 288 products near 2^120) pass 2^128 when a block of channels
    is summed over the taps first, while in the order of k, a tap's channels
    together, the sum stays below: finite, as in plain fp32.  Every term is a
    power of two times 255, so the sums are exact in either order but for fp32's
    rounding, 576 x 2^-24 of the terms' magnitude."""
    side, top = 5, np.float32(255 * 2.0**52)
    layers = [("conv", 3, 64, False), ("conv", 64, 64, False), ("avgpool",), ("linear", 64, 4)]

    def change(th):
        th[0][:] = 0
        th[0][:, 1, 1, 0] = top  # every activation of the first layer: top
        th[1][:] = 0
        th[2][:] = top
        th[2][..., 32:] *= np.float32(-0.5)
        th[3][:] = 0

    images = np.ones((3, side, side, 3), np.float32)
    (a0, a1), _, _, _, th, _ = _round(images, layers, side, change)
    assert (a0 == top).all()
    want = _conv(a0.astype(np.float64), th[2], th[3])
    terms = 1.5 * 32 * 9 * float(top)**2
    assert want.max() < float(np.finfo(np.float32).max) < terms
    assert np.isfinite(a1).all() and np.abs(a1 - want).max() <= 576 * 2.0**-24 * terms


def _same(got, want):
    """Infinities and NaN where `want` (float64) has them, the others close."""
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isposinf(got), np.isposinf(want)) and \
        np.array_equal(np.isneginf(got), np.isneginf(want))
    fin = np.isfinite(want)
    if fin.any():
        assert np.abs(got[fin] - want[fin]).max() <= 1e-5 * max(np.abs(want[fin]).max(), 1e-30)


def _grads64(g, x, w):
    """Weight gradient [co][3][3][ci], bias gradient and input gradient of a conv
    in float64 (padding as zeros, as on the GPU: an infinity times one is NaN)."""
    n, h, v, _ = g.shape
    gp, xp = (np.pad(t.astype(np.float64), ((0, 0), (1, 1), (1, 1), (0, 0))) for t in (g, x))
    with np.errstate(invalid="ignore", over="ignore"):
        dw = np.stack([np.stack([(g.astype(np.float64)[..., :, None] * xp[:, r:r + h, s:s + v, None, :]).sum((0, 1, 2))
                                 for s in range(3)], 1) for r in range(3)], 1)
        dx = sum((gp[:, 2 - r:2 - r + h, 2 - s:2 - s + v, :, None] * w[:, r, s].astype(np.float64)).sum(3)
                 for r in range(3) for s in range(3))
        return dw, g.astype(np.float64).sum((0, 1, 2)), dx


# per-tap staging (24 channels) and halo staging (64), input and weight gradients;
# 289 pixels: two splits of the weight gradients.  mixed: the infinite terms of an
# input gradient have both signs and meet as NaN, else it is an infinity
@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("a,b", [(8, 24), (32, 64)])
def test_infinite_gradients_pass_as_in_fp32(a, b, mixed):
    """One channel of the last conv (residual) has an infinite gradient: two
    classes with weights of +-3.4e38 there, one example, the wrong one right.
    The input gradient (residual and ReLU mask included), the weight gradients
    with it and, of what reaches the layer below, all gradients there are checked
    against float64 from the GPU's own inputs of each pass."""
    side, c = 17, 5
    layers = [("conv", 3, a, False), ("conv", a, b, False), ("conv", b, b, True), ("avgpool",), ("linear", b, 4)]

    images = np.random.default_rng(4).standard_normal((1, side, side, 3)).astype(np.float32)

    def change(th):
        th[4][c] *= np.float32(1e-3)  # a small channel (its logits stay finite), on at half the pixels
        th[2][c], th[3][c], th[5][c] = 0, 0, 0
        if not mixed:
            th[4][c] = np.abs(th[4][c])
        x = _conv(_conv(images.astype(np.float64), th[0], th[1]), th[2], th[3])
        th[5][c] = -np.median(_conv(x, th[4][c:c + 1], np.array([1e3])) - 1e3)
        th[6][1, c], th[6][2, c] = np.float32(-3.4e38), np.float32(3.4e38)

    act, grad, _, _, th, gpre = _round(images, layers, side, change, labels=np.array([1], np.int32))
    assert all(np.isfinite(x).all() for x in act)
    live = act[2][..., c] > 0
    assert 0 < live.sum() < live.size
    assert np.isposinf(gpre[2][..., c][live]).all() and (gpre[2][..., c][~live] == 0).all()
    assert np.isfinite(np.delete(gpre[2], c, 3)).all()
    o = 0
    for i in range(3):
        x = images if i == 0 else act[i - 1]
        dw, db, dx = _grads64(gpre[i], x, th[2 * i])
        n = th[2 * i].size
        _same(grad[o:o + n].reshape(th[2 * i].shape), dw)
        _same(grad[o + n:o + n + len(db)], db)
        o += n + len(db)
        if i:
            with np.errstate(invalid="ignore"):
                dx = np.where(act[i - 1] > 0, dx + gpre[i] if i == 2 else dx, 0.0)
            _same(gpre[i - 1], dx)
    inf, nan = np.isinf(gpre[1]).sum(), np.isnan(gpre[1]).sum()
    assert nan > 0 if mixed else inf > 0 and nan == 0
