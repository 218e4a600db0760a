"""The SGD pass where the split-K partials of small networks are summed by four
waves (12 splits or more and few elements), beside the one-chain sums."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from gcpsl_inputs import get_config  # noqa: E402
from paper_2609_29395_amd import driver  # noqa: E402

pytestmark = pytest.mark.gpu


# few elements and many splits (one replica, and parameter rows of every
# alignment: 10, 7 and 4 classes); more replicas; a batch too small to split
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("C,B,classes,w", [(1, 48, 10, (8, 32, 64)), (3, 24, 7, (8, 40, 24)), (2, 40, 4, (32, 64, 72)), (2, 3, 10, (8, 16, 8))])
def test_round_against_the_oracle(dtype, C, B, classes, w):
    from test_gpu_parity import check_run, matched_run
    layers = [("conv", 3, w[0], False), ("conv", w[0], w[1], False), ("maxpool",), ("conv", w[1], w[2], False), ("avgpool",),
              ("linear", w[2], classes)]
    cfg = get_config("tiny", H=16, W=16, B=B, C=C, K=8 * C, N_ex=classes * 4 * max(C * B, 16), L=classes, layers=layers,
                     cut=2, momentum=0.9, F=0, T=1, dtype=dtype)
    ctx, o, theta0, losses, _ = matched_run(cfg, 1)
    check_run(ctx, o, theta0, losses, cfg)


def test_serial_and_concurrent_bit_for_bit():
    cfg = get_config("tiny", H=16, W=16, B=40, C=3, K=24, N_ex=960, momentum=0.9, F=0, T=2,
                     layers=[("conv", 3, 32, False), ("conv", 32, 64, False), ("avgpool",), ("linear", 64, 4)], cut=1)
    out = []
    for serial in (False, True):
        ctx, _ = driver.setup(cfg, max_steps=2)
        losses = torch.zeros(2, 3, device="cuda")
        driver.train(ctx, 2, losses=losses, serial=serial)
        torch.cuda.synchronize()
        out.append([t.cpu().numpy() for t in (losses, ctx.theta, ctx.mom)])
        ctx.close()
    for a, b in zip(*out):
        assert np.isfinite(a).all() and np.array_equal(a, b)
