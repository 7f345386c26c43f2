"""Infinite and NaN activations: outputs that are infinite by y = x W^T stay so, and only those without a value become NaN,
on the kernels that add the sensitive weights apart from the dense product just as on the tiled kernel, which adds them to
the weight tile first (configuration 1).  Other token rows are not touched."""
import numpy as np
import pytest
import torch

from paper_2406_02913_amd import szo
from helpers import make_pair, rel_fro
from test_gpu_two_activation_sets import _with_x_minus

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _auto_tile_config():
    yield
    szo.szo_set_tile_config(0)


def _step(d, tile, values, cfg, eps, flags):
    """One step from the given sensitive values (g and with it the update are NaN, also for a learning rate of zero)."""
    scal = torch.zeros(3, dtype=torch.float64, device="cuda")
    d.sp_val.copy_(values)
    szo.szo_set_tile_config(cfg)
    szo.szo_zo_step([d.desc(tile, with_y=not flags)], 3, 1, eps, 0.0, scal, szo.new_workspace(), flags)
    return scal.cpu().numpy()[:2].copy()


def _poison(x, o):
    """An infinity at a sensitive column, one elsewhere, two of opposite sign, a NaN, and bf16 values beyond fp16."""
    K = x.shape[1]
    at = int(o.sp_idx[0]) % K
    x[3, at] = float("inf")
    x[5, (at + 1) % K] = float("-inf")
    x[6, 2], x[6, K - 1] = float("inf"), float("-inf")
    x[7, 0] = float("nan")
    x[9, at] = 1e30


def _same_classes(a, b):
    return np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(np.isposinf(a), np.isposinf(b)) and \
        np.array_equal(np.isneginf(a), np.isneginf(b))


def _agree(y, want, tol):
    fine = np.isfinite(want).all(axis=1)
    assert 0 < fine.sum() < y.shape[0] and np.isinf(want).any() and np.isnan(want).any()
    assert _same_classes(y, want) and rel_fro(y[fine], want[fine]) <= tol


# (M, N, K, group, format, tile, configuration): the split kernel, chosen or forced
@pytest.mark.parametrize("M,N,K,G,fmt,tile,cfg", [(20, 100, 320, 64, "uniform", "bf16", 0), (20, 100, 320, 32, "uniform", "f16", 0),
                                                  (16, 70, 256, 128, "uniform", "f16", 8), (16, 70, 512, 128, "lut", "f16", 8)])
def test_forwards(M, N, K, G, fmt, tile, cfg):
    dt = szo.TILE_BF16 if tile == "bf16" else szo.TILE_F16
    o, d = make_pair(701, M, N, K, G, 2e-2, nnz_base=4, fmt=fmt)
    _poison(d.x, o)
    ws, loss = szo.new_workspace(), torch.zeros(1, dtype=torch.float64, device="cuda")
    for sign in (+1, -1, 0):
        ys, losses = [], []
        for c in (2 if fmt == "lut" else 1, cfg):
            szo.szo_set_tile_config(c)
            szo.szo_linear_fwd(d.desc(dt), 3, 1, sign, 1e-3)
            ys.append(d.y.cpu().numpy().copy())
            loss.zero_()
            szo.szo_linear_fwd_mse(d.desc(dt), 3, 1, sign, 1e-3, 1.0 / (M * N), loss, ws)
            losses.append(loss.cpu().numpy().copy())
            assert _same_classes(d.y.cpu().numpy(), ys[-1])
        _agree(ys[1], ys[0], 1e-3)
        assert _same_classes(losses[1], losses[0])


@pytest.mark.parametrize("tile", ["f16", "bf16"])
@pytest.mark.parametrize("M,N,K,G", [(70, 300, 192, 64), (16, 64, 256, 128)])
def test_step_with_outputs_on_the_one_dense_pass_kernel(M, N, K, G, tile):
    dt = szo.TILE_BF16 if tile == "bf16" else szo.TILE_F16
    o, d = make_pair(702, M, N, K, G, 2e-2)
    _poison(d.x, o)
    values, ys, losses = d.sp_val.clone(), [], []
    for cfg in (1, 11):
        losses.append(_step(d, dt, values, cfg, 1e-3, 0))
        ys.append(d.y.cpu().numpy().copy())
        assert _same_classes(_step(d, dt, values, cfg, 1e-3, szo.STEP_FUSED_LOSS), losses[-1])
    _agree(ys[1], ys[0], 1e-3 if tile == "f16" else 5e-3)
    assert _same_classes(losses[1], losses[0])


@pytest.mark.parametrize("what", ["infinite", "overflow"])
@pytest.mark.parametrize("cfg,two_sets,K", [(8, False, 320), (8, True, 320), (11, False, 320)])
def test_losses_are_infinite_where_every_output_has_a_value(cfg, two_sets, K, what):
    """Five rows of W, an infinite activation in a column without a zero weight (or activations whose products overflow
    fp32): both losses are +inf, not NaN, as on the tiled kernel."""
    o, d = make_pair(703, 70, 5, K, 64, 2e-2)
    if two_sets:
        o, d = _with_x_minus(o, d, 704)
    column = int(np.flatnonzero((o.codes != 8).all(axis=0))[0])
    for x in (d.x, d.x_minus) if two_sets else (d.x,):
        if what == "infinite":
            x[11, column] = float("inf")
        else:
            x[11].fill_(0)
            x[11, column] = 3e38
    if what == "overflow":
        d.scales.fill_(100.0)
    values = d.sp_val.clone()
    for eps in (1e-3, 0.0):
        for c in (1, cfg):
            losses = _step(d, szo.TILE_BF16, values, c, eps, szo.STEP_FUSED_LOSS)
            assert np.isposinf(losses).all(), (c, eps, losses)
