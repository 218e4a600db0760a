"""The classifier head in parts of its batch: parts of equal and unequal size,
one part, heads in registers and in LDS, and labels, losses and gradients that
only the parts' sums hold."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from gcpsl_inputs import get_config  # noqa: E402
from paper_2609_29395_amd import driver  # noqa: E402

pytestmark = pytest.mark.gpu


def _cfg(B, C, ch, classes, dtype, **kw):
    layers = [("conv", 3, 8, False), ("conv", 8, ch, False), ("avgpool",), ("linear", ch, classes)]
    return get_config("tiny", H=4, W=4, B=B, C=C, K=8 * C, N_ex=classes * 4 * max(C * B, 16), L=classes, layers=layers,
                      cut=1, momentum=0.9, F=0, dtype=dtype, **kw)


# batches of one part (8), of a last part of one example (9, 57), of eight
# parts (64, 100); 16 classes or fewer in registers, more or more than 256
# channels in LDS, with eight lanes per logit (up to 128 logits a part) or a
# thread; parts limited by the room (40 classes beside few weights)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,C,ch,classes", [(8, 2, 16, 4), (9, 2, 64, 10), (57, 1, 136, 7), (100, 2, 256, 16), (64, 3, 24, 17),
                                            (33, 2, 512, 10), (40, 1, 8, 40), (8, 1, 72, 16), (16, 2, 264, 16),
                                            (9, 1, 264, 30)])
def test_round_against_the_oracle(dtype, B, C, ch, classes):
    from test_gpu_parity import check_run, matched_run
    cfg = _cfg(B, C, ch, classes, dtype, T=2, label_smoothing=0.1)
    ctx, o, theta0, losses, _ = matched_run(cfg, 2)
    check_run(ctx, o, theta0, losses, cfg)


def test_serial_and_concurrent_bit_for_bit():
    cfg = _cfg(50, 3, 64, 10, "bf16", T=2)
    out = []
    for serial in (False, True):
        ctx, _ = driver.setup(cfg, max_steps=2)
        losses = torch.zeros(2, 3, device="cuda")
        driver.train(ctx, 2, losses=losses, serial=serial)
        torch.cuda.synchronize()
        out.append([t.cpu().numpy() for t in (losses, ctx.theta, ctx.mom, ctx.tensor("grad"))])
        ctx.close()
    for a, b in zip(*out):
        assert np.isfinite(a).all() and np.array_equal(a, b)
