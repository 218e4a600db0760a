"""bf16 convolutions against the oracle, at the sizes where their kernels can go
wrong: the k loop unrolled over whole 64-channel blocks (k_conv_lds.hip, 128 x
64 tiles) and the weight gradient of images of any width (k_conv.hip)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from gcpsl_inputs import get_config  # noqa: E402
from paper_2609_29395_amd import driver  # noqa: E402
from test_gpu_parity import check_run, matched_run  # noqa: E402

pytestmark = pytest.mark.gpu


# 3 x 3: one, two and three channel blocks; one pixel to several tiles with a
# ragged last one; output channels that end inside a tile (72, 136); a
# residual layer; images of one pixel and a width that is no power of two
@pytest.mark.parametrize("side,B,C,w1,w2,w3", [
    (1, 5, 1, 64, 64, 128), (4, 8, 2, 64, 128, 64), (5, 27, 2, 64, 72, 64), (6, 29, 3, 64, 136, 192), (12, 20, 3, 64, 64, 128),
    (32, 2, 2, 64, 64, 64),
])
def test_three_by_three(side, B, C, w1, w2, w3):
    layers = [("conv", 3, w1, False), ("conv", w1, w2, False), ("conv", w2, w3, False), ("conv", w3, w3, True),
              ("avgpool",), ("linear", w3, 4)]
    cfg = get_config("tiny", H=side, W=side, B=B, C=C, K=8 * C, N_ex=4 * max(C * B, 16), layers=layers, cut=2,
                     momentum=0.9, F=0, T=1, dtype="bf16")
    ctx, o, theta0, losses, _ = matched_run(cfg, 1)
    check_run(ctx, o, theta0, losses, cfg)


# strided blocks: one-tap products of one to four k tiles (projections) and of
# nine and more (the im2col rows of the 3 x 3), with tails of the group of three
@pytest.mark.parametrize("side,B,w1,w2,w3", [(4, 9, 64, 64, 128), (8, 5, 128, 192, 64), (12, 3, 192, 64, 72),
                                             (4, 16, 256, 64, 128)])
def test_strided_blocks(side, B, w1, w2, w3):
    layers = [("conv", 3, w1, False), ("gnorm", w1, w1 // 8), ("block", w1, w2, 2, w2 // 8), ("block", w2, w3, 2, w3 // 8),
              ("avgpool",), ("linear", w3, 4)]
    cfg = get_config("tiny", H=side, W=side, B=B, C=2, K=16, N_ex=128, layers=layers, cut=3, momentum=0.9, F=0, T=1,
                     dtype="bf16")
    ctx, o, theta0, losses, _ = matched_run(cfg, 1)
    check_run(ctx, o, theta0, losses, cfg)


# fewer than 64 output channels on widths that are no multiple of a block's
# eight pixels: blocks across image rows, images and the batch's end; one pixel
# wide; column tiles of 32, 64 and 128
@pytest.mark.parametrize("H,W,B,w1,w2,w3", [(1, 1, 9, 8, 8, 8), (4, 3, 5, 8, 16, 24), (2, 9, 11, 16, 56, 8), (5, 12, 7, 32, 40, 16),
                                            (3, 33, 3, 24, 8, 56)])
def test_weight_gradient_of_any_width(H, W, B, w1, w2, w3):
    layers = [("conv", 3, w1, False), ("conv", w1, w2, False), ("conv", w2, w3, False), ("avgpool",), ("linear", w3, 4)]
    cfg = get_config("tiny", H=H, W=W, B=B, C=2, K=16, N_ex=128, layers=layers, cut=2, momentum=0.9, F=0, T=1,
                     dtype="bf16")
    ctx, o, theta0, losses, _ = matched_run(cfg, 1)
    check_run(ctx, o, theta0, losses, cfg)


# residual layers whose tile depends on the launch's replicas: eight clusters
# take 256 x 128 (or 256 x 256) tiles, one alone 128 x 64
@pytest.mark.parametrize("side,B,w", [(32, 16, 128), (8, 128, 256), (8, 256, 256)])
def test_serial_residual_layers_bit_for_bit(side, B, w):
    layers = [("conv", 3, 64, False), ("conv", 64, w, False), ("conv", w, w, True), ("avgpool",), ("linear", w, 4)]
    cfg = get_config("tiny", H=side, W=side, B=B, C=8, K=64, N_ex=4 * 8 * B, layers=layers, cut=2, momentum=0.9, F=0,
                     T=1, dtype="bf16")
    out = []
    for serial in (False, True):
        ctx, _ = driver.setup(cfg, max_steps=1)
        losses = torch.zeros(1, 8, device="cuda")
        driver.train(ctx, 1, losses=losses, serial=serial)
        torch.cuda.synchronize()
        out.append([t.cpu().numpy() for t in (losses, ctx.theta, ctx.mom)])
        ctx.close()
    for a, b in zip(*out):
        assert np.isfinite(a).all() and np.array_equal(a, b)
