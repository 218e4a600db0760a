"""Normalisation layers on shapes where their launches split the work
differently for one cluster and for all of them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from gcpsl_inputs import get_config  # noqa: E402
from paper_2609_29395_amd import driver  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_serial_clusters_of_large_norm_layers_bit_for_bit(dtype):
    # 16,384 pixels per cluster: the channel reductions' chunks for four
    # clusters are twice those one cluster alone would take
    cfg = get_config("ragged_norm_bf16", C=4, K=32, B=64, H=16, W=16, N_ex=1400, T=2, F=0, dtype=dtype)
    out = []
    for serial in (False, True):
        ctx, _ = driver.setup(cfg, max_steps=2)
        losses = torch.zeros(2, 4, device="cuda")
        driver.train(ctx, 2, losses=losses, serial=serial)
        torch.cuda.synchronize()
        out.append([t.cpu().numpy() for t in (losses, ctx.theta, ctx.mom, ctx.norm_state)])
        ctx.close()
    for a, b in zip(*out):
        assert np.isfinite(a).all() and np.array_equal(a, b)
