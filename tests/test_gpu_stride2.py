"""Input gradients of strided blocks by classes of input pixels (fp32, and bf16
of whole 64-channel blocks) and by the gradient spread to the input grid (other
bf16 channel counts), against the oracle."""
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from gcpsl_inputs import get_config  # noqa: E402
from test_gpu_parity import check_run, matched_run  # noqa: E402

pytestmark = pytest.mark.gpu


# one output pixel per image, one row, one column; tiles that end inside an
# image; channel blocks 64, 128, 192 (tap loops of one to three blocks) and 8,
# 72, 136 (stages that span two taps in fp32); a tile of 32, 64, 128 inputs
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
