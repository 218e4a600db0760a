"""Normalisation layers on shapes where their launches split the work
differently for one cluster and for all of them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from gcpsl_inputs import get_config  # noqa: E402
from paper_2609_29395_amd import driver, gcpsl  # noqa: E402

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


# group norm: examples held with 256 and 512 threads, and read again (32 x 32
# x 72 channels, and 520), by their own workgroup or where they are fewer than 64
# by an elementwise pass; 3 vectors per pixel (idle lanes); two channels per
# group and one group; batch norm: one launch of up to 2 and 8 pixels a thread,
# three launches (more than 8,192 pixels, or 4,096 of wide rows), one and two
# vectors per workgroup
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("side,B,C,w1,g1,w2,g2,w3", [
    (5, 7, 2, 8, 4, 24, 1, 40), (9, 3, 1, 24, 3, 64, 32, 8), (16, 5, 2, 64, 32, 128, 32, 16), (32, 2, 1, 72, 9, 8, 2, 24),
    (16, 33, 2, 8, 2, 16, 4, 136), (32, 9, 1, 8, 4, 8, 1, 8), (3, 5, 16, 8, 2, 16, 4, 256),
    (2, 33, 2, 520, 8, 16, 4, 8), (3, 9, 2, 520, 1, 1016, 127, 8),
    (16, 17, 2, 8, 2, 8, 2, 1024), (16, 17, 1, 8, 2, 8, 2, 40),
])
def test_norm_round_against_the_oracle(dtype, side, B, C, w1, g1, w2, g2, w3):
    from test_gpu_parity import check_run, matched_run
    layers = [("conv", 3, w1, False), ("gnorm", w1, g1), ("conv", w1, w2, False), ("gnorm", w2, g2),
              ("conv", w2, w3, False), ("bnorm", w3), ("avgpool",), ("linear", w3, 4)]
    cfg = get_config("tiny", H=side, W=side, B=B, C=C, K=8 * C, N_ex=4 * max(C * B, 16), layers=layers, cut=4,
                     momentum=0.9, F=0, T=1, dtype=dtype)
    ctx, o, theta0, losses, _ = matched_run(cfg, 1)
    check_run(ctx, o, theta0, losses, cfg)


# 1,024 pixels per cluster (one launch), 512 channels: four clusters take two
# channel vectors per workgroup, one alone would take one.  Sums over the same
# values in another order agree in fp64 to far below an fp32 spacing, so the
# images make the order visible: each batch holds every image and its negative,
# with magnitudes over 2^40, and two small images besides, so a channel's sum
# cancels to the small images' while its partial sums round at 2^-53 of the large.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_serial_clusters_of_small_batch_norms_bit_for_bit(dtype):
    side, B, C, ch = 4, 64, 4, 512
    rng = np.random.default_rng(7)
    images, clients = [], []
    for n in range(C):
        x = rng.standard_normal((31, side, side, 3)) * 2.0 ** rng.uniform(0, 40, (31, side, side, 3))
        images += [x, -x, rng.standard_normal((2, side, side, 3))]
        clients += [n] * B
    w = rng.uniform(-0.2, 0.2, (ch, 27))
    theta = np.concatenate([w.ravel(), np.zeros(ch), np.ones(ch), np.zeros(ch), rng.uniform(-0.05, 0.05, 4 * ch),
                            np.zeros(4)]).astype(np.float32)
    cfg = dict(K=C, C=C, B=B, L=4, H=side, W=side, Cin=3, N_ex=C * B, dtype=dtype, lr=0.01, momentum=0.9, seed=0,
               layers=[("conv", 3, ch, False), ("bnorm", ch), ("avgpool",), ("linear", ch, 4)], cut=2)
    state0 = np.concatenate([np.zeros(ch), np.ones(ch), np.zeros(1)]).astype(np.float32)
    labels = rng.integers(0, 4, C * B).astype(np.int32)
    out = []
    for serial in (False, True):
        ctx = gcpsl.Context(cfg, np.concatenate(images).astype(np.float32), labels, np.array(clients, np.int32),
                            np.arange(C, dtype=np.int32), theta, max_steps=1, norm_state0=state0)
        loss = torch.zeros(C, device="cuda")
        ctx.sample(0)
        if serial:
            for n in range(C):
                ctx.step_replica(0, n, loss)
        else:
            ctx.step(0, loss)
        torch.cuda.synchronize()
        out.append([t.cpu().numpy() for t in (loss, ctx.theta, ctx.mom, ctx.norm_state)])
        ctx.close()
    for a, b in zip(*out):
        assert np.isfinite(a).all() and np.array_equal(a, b)
