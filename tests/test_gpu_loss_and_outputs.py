"""szo_linear_fwd_mse writes the outputs of szo_linear_fwd beside the loss whenever the descriptor names a buffer, on every
kernel that can run the call, and the steps that return losses alone leave that buffer as it was."""
import numpy as np
import pytest
import torch

from paper_2406_02913_amd import szo
from helpers import make_pair

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _auto_tile_config():
    yield
    szo.szo_set_tile_config(0)


# (seed, M, N, K, group, format, tile, configuration): the kernels that share the call -- split (0 and 8), stream (9; with a
# group of 64 and with tables too), tiled (0 with many tokens)
CALLS = [
    (601, 16, 200, 320, 64, "uniform", "bf16", 0),       # bf16 tile, K an odd multiple of 64
    (602, 77, 130, 320, 32, "uniform", "f16", 0),        # fp16 tile, K an odd multiple of 64, five slices
    (603, 77, 200, 256, 128, "uniform", "bf16", 0),
    (604, 16, 256, 512, 128, "uniform", "f16", 0),
    (605, 1, 65, 256, 64, "uniform", "f16", 8),
    (606, 33, 300, 512, 128, "uniform", "f16", 9),       # a ragged third slice
    (607, 16, 100, 384, 64, "uniform", "f16", 9),
    (608, 20, 192, 512, 128, "lut", "f16", 0),
    (609, 20, 192, 512, 128, "lut", "f16", 9),
    (610, 40, 300, 512, 128, "uniform", "f16", 5),       # 48 token rows per pass
    (611, 300, 200, 256, 128, "uniform", "bf16", 0),
]


@pytest.mark.parametrize("call", CALLS)
def test_outputs_are_written_beside_the_loss(call):
    s, M, N, K, G, fmt, tile, cfg = call
    szo.szo_set_tile_config(cfg)
    o, d = make_pair(s, M, N, K, G, 1e-2, nnz_base=8, fmt=fmt)
    dt = szo.TILE_BF16 if tile == "bf16" else szo.TILE_F16
    ws = szo.new_workspace()
    loss = torch.zeros(2, dtype=torch.float64, device="cuda")
    for sign in (+1, -1, 0):
        szo.szo_linear_fwd(d.desc(dt), 5, 2, sign, 1e-3)
        want = d.y.cpu().numpy().copy()
        d.y.fill_(float("nan"))
        loss.zero_()
        szo.szo_linear_fwd_mse(d.desc(dt), 5, 2, sign, 1e-3, 1.0 / (M * N), loss[0:1], ws)
        assert np.array_equal(d.y.cpu().numpy(), want), sign
        szo.szo_linear_fwd_mse(d.desc(dt, with_y=False), 5, 2, sign, 1e-3, 1.0 / (M * N), loss[1:2], ws)
        assert loss[0].item() == loss[1].item() > 0.0                # the loss does not depend on whether y is wanted


@pytest.mark.parametrize("M,K,G,tile,cfg", [(16, 512, 128, "f16", 8), (40, 512, 128, "f16", 9), (16, 320, 64, "bf16", 0)])
def test_steps_with_the_loss_fused_leave_the_outputs_alone(M, K, G, tile, cfg):
    szo.szo_set_tile_config(cfg)
    o, d = make_pair(621, M, 200, K, G, 1e-2)
    desc = d.desc(szo.TILE_BF16 if tile == "bf16" else szo.TILE_F16)
    scal = torch.zeros(3, dtype=torch.float64, device="cuda")
    d.y.fill_(7.0)
    szo.szo_zo_step([desc], 5, 0, 1e-3, 0.0, scal, szo.new_workspace(), szo.STEP_FUSED_LOSS)
    szo.szo_zo_step_noalloc([desc], 5, 0, 1e-3, 0.0, scal)
    assert bool((d.y == 7.0).all())


def test_a_layer_with_more_partials_than_the_workspace_holds_takes_the_tiled_kernel():
    """64 tokens, one 64-column tile and 2^24 + 64 rows: one band more than the split kernel has room for partials."""
    M, N, K = 64, (1 << 24) + 64, 64
    gen = torch.Generator(device="cuda").manual_seed(3)
    q = torch.randint(256, (N // 64, 64, 32), generator=gen, device="cuda", dtype=torch.uint8)      # [band][row][byte]
    scales = torch.full((N,), 0.01, device="cuda", dtype=torch.float16)
    x = torch.randn((M, K), generator=gen, device="cuda", dtype=torch.bfloat16)
    target = torch.randn((M, N), generator=gen, device="cuda", dtype=torch.bfloat16)
    tile_ptr = torch.zeros(N // 64 + 1, device="cuda", dtype=torch.int32)
    desc = szo.make_desc(M, N, K, 64, 0, 0, x, q.view(-1), scales, tile_ptr, None, None, None, target, szo.TILE_BF16)
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    szo.szo_linear_fwd_mse(desc, 1, 0, 0, 0.0, 1.0 / (M * N), loss, szo.new_workspace())
    want = 0.0
    for lo in range(0, N, 1 << 20):
        rows = q.view(N, 32)[lo:lo + (1 << 20)]
        codes = torch.stack([rows & 15, rows >> 4], dim=2).view(-1, K).float() - 8.0
        w = (codes * scales[0].float()).bfloat16().float()
        want += ((x.float() @ w.t()).double() - target[:, lo:lo + (1 << 20)].double()).square_().sum().item() / (M * N)
    # the same bf16 operands, fp32 sums of 64 products
    assert abs(loss.item() - want) <= 1e-6 * want
