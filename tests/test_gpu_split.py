"""GPU parity of the few-token kernel for small launches (K split over the waves of a workgroup), forced by tile
configuration 8, at the edges of its ranges: one half-filled 128-column block, fewer blocks than waves, ragged bands and
slices, windows of sensitive entries that are refilled, every dequantisation and both tile types."""
import numpy as np
import pytest
import torch

from oracle import layer as olayer, philox as ophilox
from paper_2406_02913_amd import szo
from helpers import make_pair, rel_fro
from test_gpu_two_activation_sets import _check_step, _with_x_minus

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _auto_tile_config():
    yield
    szo.szo_set_tile_config(0)


# (seed, M, N, K, group, density, format, tile)
SHAPES = [
    (201, 1, 64, 128, 128, 1e-2, "uniform", "f16"),       # one band, one block: fewer blocks than waves
    (202, 15, 65, 256, 128, 2e-2, "uniform", "f16"),      # a band of one row
    (203, 17, 200, 2176, 128, 1e-3, "uniform", "f16"),    # 17 blocks over the waves, second slice of one token
    (204, 16, 64, 2048, 128, 8e-2, "uniform", "f16"),     # ~650 entries per wave: several windows
    (205, 33, 130, 512, 128, 0.0, "uniform", "f16"),      # no sensitive entries
    (206, 4, 5000, 256, 128, 2e-3, "uniform", "f16"),     # many workgroups: four waves at most have a block
    (207, 16, 100, 384, 32, 1e-2, "uniform", "f16"),      # group 32
    (208, 9, 128, 640, 64, 2e-2, "uniform", "f16"),       # group 64
    (209, 7, 96, 64, 32, 5e-2, "uniform", "f16"),         # K = 64: half a block
    (210, 20, 70, 320, 64, 2e-2, "uniform", "f16"),       # K an odd multiple of 64
    (211, 18, 129, 1088, 64, 1e-2, "uniform", "bf16"),    # the same with the bf16 tile
    (212, 3, 64, 512, 128, 3e-2, "uniform", "bf16"),      # bf16, group 128
    (213, 16, 192, 512, 128, 1e-2, "lut", "f16"),
    (214, 5, 100, 1152, 128, 3e-2, "lut", "f16"),
]


@pytest.mark.parametrize("shape", SHAPES)
def test_forward_matches_oracle(shape):
    s, M, N, K, G, dens, fmt, tile = shape
    szo.szo_set_tile_config(8)
    o, d = make_pair(s, M, N, K, G, dens, nnz_base=12, fmt=fmt)
    seed, step, eps = 77, 5, 1e-3
    z = ophilox.zbar(seed, step, 12, o.sp_idx.size)
    dt = szo.TILE_BF16 if tile == "bf16" else szo.TILE_F16
    for sign in (+1, -1, 0):
        d.y.fill_(float("nan"))
        szo.szo_linear_fwd(d.desc(tile_dtype=dt), seed, step, sign, eps)
        y = d.y.cpu().numpy()
        assert np.isfinite(y).all()
        if tile == "bf16" or K % 128:
            # operands rounded as in the tiled kernel's weight tile: only the fp32 summation order differs
            want = olayer.linear_fwd(o.x_bits, o.codes, o.scales, G, o.sp_idx, o.sp_val, z, sign, eps, "D", tile)
            tol = 2e-5
        else:
            # the bounds of the few-token path: un-centred codes (group 128), fp16 sparse values
            want = olayer.linear_fwd(o.x_bits, o.codes, o.scales, G, o.sp_idx, o.sp_val, z, sign, eps, "E", lut=o.lut)
            tol = 5e-4 if G == 128 else 1e-3
        assert rel_fro(y, want) <= tol, (sign, rel_fro(y, want))


@pytest.mark.parametrize("two_sets", [False, True])
@pytest.mark.parametrize("tile", ["f16", "bf16"])
def test_steps_match_oracle(two_sets, tile):
    """Whole steps: losses, g and updates, layers of several formats in one step (one launch per instantiation)."""
    szo.szo_set_tile_config(8)
    os_, ds_, base = [], [], 0
    for (s, M, N, K, G, dens, fmt) in [(221, 23, 200, 512, 128, 1e-2, "uniform"), (222, 16, 130, 384, 64, 1e-2, "uniform"),
                                       (223, 40, 64, 256, 128, 2e-2, "lut" if tile == "f16" else "uniform"), (224, 5, 100, 192, 32, 2e-2, "uniform")]:
        o, d = make_pair(s, M, N, K, G, dens, nnz_base=base, fmt=fmt)
        base += (o.sp_idx.size + 3) // 4 * 4
        if two_sets:
            o, d = _with_x_minus(o, d, s + 100)
        if tile == "bf16":
            desc = d.desc
            d.desc = lambda with_y=True, desc=desc: desc(tile_dtype=szo.TILE_BF16, with_y=with_y)
        os_.append(o)
        ds_.append(d)
    if tile == "f16" or two_sets:
        # (two sets: g is the difference of two unrelated losses; bf16 weights move each of them by up to 2^-8 / sqrt(outputs))
        _check_step(os_, ds_, szo.STEP_FUSED_LOSS, ltol=1e-4 if tile == "f16" else 5e-4)
    else:
        # the bf16 tile misses the bar on g by construction: compare with the tiled kernel on the same operands instead
        scal, ws, out = torch.zeros(3, dtype=torch.float64, device="cuda"), szo.new_workspace(), []
        for cfg in (8, 1):
            szo.szo_set_tile_config(cfg)
            szo.szo_zo_step([d.desc(with_y=False) for d in ds_], 3, 1, 1e-3, 0.0, scal, ws, szo.STEP_FUSED_LOSS)
            out.append(scal.cpu().numpy().copy())
        # same operands, other summation order: 1e-6 on the losses, and that over 2 eps on their difference
        assert np.allclose(out[0][:2], out[1][:2], rtol=1e-6, atol=0)
        assert abs(out[0][2] - out[1][2]) <= 1e-6 * out[1][0] / 1e-3


def test_stream_kernel_still_matches_oracle_and_the_split_kernel():
    """The stream kernel on a shape that a small launch no longer takes it for, with and without the non-temporal
    stream (the same bits), against the split kernel."""
    o, d = make_pair(231, 16, 520, 1152, 128, 5e-3, nnz_base=4)
    z = ophilox.zbar(9, 3, 4, o.sp_idx.size)
    ys = {}
    for cfg in (8, 9, 10):
        szo.szo_set_tile_config(cfg)
        szo.szo_linear_fwd(d.desc(), 9, 3, +1, 1e-3)
        ys[cfg] = d.y.cpu().numpy().copy()
    want = olayer.linear_fwd(o.x_bits, o.codes, o.scales, 128, o.sp_idx, o.sp_val, z, +1, 1e-3, "E")
    assert np.array_equal(ys[9], ys[10])
    assert rel_fro(ys[9], want) <= 5e-4 and rel_fro(ys[8], ys[9]) <= 2e-6      # same products, other summation order


# (seed, M, N, K, group, density, format, tile): bands x slices of up to 64 / 128 / more are cut into four / two / one workgroups each
@pytest.mark.parametrize("shape", [
    (251, 4, 64 * 64, 128, 128, 5e-3, "uniform", "f16"),      # 64 bands: the last with four parts, x staged for up to four rows
    (252, 5, 64 * 64 + 1, 128, 128, 5e-3, "uniform", "f16"),  # 65: two parts, the last band of one row
    (253, 3, 64 * 129 - 63, 256, 128, 2e-3, "uniform", "f16"),   # 129: whole bands, three rows
    (254, 33, 64 * 43, 256, 128, 2e-3, "uniform", "f16"),     # three slices, the last of one row: 129
    (255, 17, 64 * 40, 384, 64, 3e-3, "uniform", "bf16"),     # two parts, sensitive weights rounded in the tile
    (256, 130, 500, 8192, 128, 1e-3, "uniform", "f16"),       # 72 and a K of 64 blocks
    (257, 144, 1000, 8192, 128, 1e-3, "uniform", "f16"),      # 144: whole bands again
    (258, 16, 100, 640, 128, 8e-2, "lut", "f16"),             # four parts, several windows of entries per wave
], ids=lambda s: str(s[0]))
def test_bands_cut_into_parts_match_oracle(shape):
    s, M, N, K, G, dens, fmt, tile = shape
    szo.szo_set_tile_config(8)
    o, d = make_pair(s, M, N, K, G, dens, nnz_base=8, fmt=fmt)
    dt = szo.TILE_BF16 if tile == "bf16" else szo.TILE_F16
    z = ophilox.zbar(5, 2, 8, o.sp_idx.size)
    rounded = tile == "bf16"                             # the bounds are those of test_forward_matches_oracle
    want = olayer.linear_fwd(o.x_bits, o.codes, o.scales, G, o.sp_idx, o.sp_val, z, +1, 1e-3, "D" if rounded else "E",
                             *((tile,) if rounded else ()), **({} if rounded else {"lut": o.lut}))
    d.y.fill_(float("nan"))
    szo.szo_linear_fwd(d.desc(tile_dtype=dt), 5, 2, +1, 1e-3)
    y = d.y.cpu().numpy()
    assert np.isfinite(y).all() and rel_fro(y, want) <= (2e-5 if rounded else 5e-4 if fmt == "uniform" else 1e-3)
    # one loss partial per workgroup: none of them lost or added twice
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    szo.szo_linear_fwd_mse(d.desc(tile_dtype=dt), 5, 2, +1, 1e-3, 1.0 / (M * N), loss, szo.new_workspace())
    mine = float(((d.y.double() - d.target.double()) ** 2).mean().item())
    assert abs(loss.item() - mine) <= 1e-6 * mine
    scal = torch.zeros(3, dtype=torch.float64, device="cuda")
    szo.szo_zo_step([d.desc(tile_dtype=dt, with_y=False)], 5, 2, 1e-3, 0.0, scal, szo.new_workspace(), szo.STEP_FUSED_LOSS)
    assert abs(scal[0].item() - mine) <= 1e-6 * mine


def test_long_k_beside_many_short_bands_is_cut_in_two():
    """132 bands of K = 128 and 4 of K = 16384 in one step: the latter are cut for the length of their chain alone."""
    os_, ds_, base = [], [], 0
    for sd, M, N, K, dens in ((261, 64, 2100, 128, 5e-3), (262, 64, 64, 16384, 1e-3)):
        o, d = make_pair(sd, M, N, K, 128, dens, nnz_base=base)
        base += (o.sp_idx.size + 3) // 4 * 4
        os_.append(o)
        ds_.append(d)
    szo.szo_set_tile_config(8)
    _check_step(os_, ds_, szo.STEP_FUSED_LOSS, ltol=1e-4)


@pytest.mark.parametrize("M,N,K,G,fmt,tile", [
    (449, 64, 1024, 128, "uniform", "f16"),       # the first size beyond the limit on tokens, K at its lower limit
    (1500, 130, 4096, 128, "uniform", "f16"),     # 94 slices; the split or the stream kernel by their estimates
    (700, 300, 2048, 64, "uniform", "f16"), (500, 100, 1152, 128, "lut", "f16"), (300, 200, 1088, 64, "uniform", "bf16"),
])
def test_many_tokens_of_a_layer_that_the_tiles_would_walk_for_longer(M, N, K, G, fmt, tile):
    """Few workgroups and a long K: any number of tokens runs as slices, one launch for both signs of a step; outputs,
    losses and g to the bounds of the few-token path against the oracle."""
    dt = szo.TILE_BF16 if tile == "bf16" else szo.TILE_F16
    o, d = make_pair(271, M, N, K, G, 2e-3, nnz_base=4, fmt=fmt)
    z = ophilox.zbar(7, 1, 4, o.sp_idx.size)
    args, kw = (("D", tile), {}) if tile == "bf16" else (("E",), {"lut": o.lut})
    want = olayer.linear_fwd(o.x_bits, o.codes, o.scales, G, o.sp_idx, o.sp_val, z, -1, 1e-3, *args, **kw)
    szo.szo_linear_fwd(d.desc(tile_dtype=dt), 7, 1, -1, 1e-3)
    assert rel_fro(d.y.cpu().numpy(), want) <= (2e-5 if tile == "bf16" else 5e-4 if G == 128 and fmt == "uniform" else 1e-3)
    scal = torch.zeros(3, dtype=torch.float64, device="cuda")
    szo.szo_kernel_timing(True)
    szo.szo_zo_step([d.desc(tile_dtype=dt, with_y=False)], 7, 1, 1e-3, 0.0, scal, szo.new_workspace(), szo.STEP_FUSED_LOSS)
    _, launches = szo.szo_kernel_timing_read()
    szo.szo_kernel_timing(False)
    assert launches == 1
    loss = olayer.mse_loss(want, o.target_bits)
    assert abs(scal[1].item() - loss) <= 1e-4 * loss


def test_noalloc_falls_back_to_fewer_partials():
    """A step whose split launches would write more loss partials than the fixed array holds keeps working."""
    szo.szo_set_tile_config(0)
    o, d = make_pair(241, 100, 2048, 128, 128, 1e-3)
    one = d.desc(with_y=False)
    n = 330                                             # 32 bands x 7 slices x 330 = 73 920 > 65 536
    scal, ref = torch.zeros(3, dtype=torch.float64, device="cuda"), torch.zeros(3, dtype=torch.float64, device="cuda")
    szo.szo_zo_step_noalloc([one] * n, 1, 0, 1e-3, 0.0, scal)
    szo.szo_zo_step_noalloc([one], 1, 0, 1e-3, 0.0, ref)
    assert abs(scal[0].item() - n * ref[0].item()) <= 1e-6 * scal[0].item()


@pytest.mark.parametrize("n", [256, 257])               # 64 bands in four parts each: 65 536 partials per sign, as many as fit, and one layer more
def test_noalloc_falls_back_to_whole_bands(n):
    szo.szo_set_tile_config(8)
    o, d = make_pair(242, 13, 4096, 128, 128, 1e-3)
    one = d.desc(with_y=False)
    scal, ref = torch.zeros(3, dtype=torch.float64, device="cuda"), torch.zeros(3, dtype=torch.float64, device="cuda")
    szo.szo_zo_step_noalloc([one], 1, 0, 1e-3, 0.0, ref)
    szo.szo_zo_step_noalloc([one] * n, 1, 0, 1e-3, 0.0, scal)
    # the same outputs either way (one block of K, four waves), their squares added in fp64 in another order: 2^-53 x 65 536 terms
    want = n * ref[:2].cpu().numpy()
    assert np.all(np.abs(scal[:2].cpu().numpy() - want) <= 1e-11 * want)
    want = olayer.mse_loss(olayer.linear_fwd(o.x_bits, o.codes, o.scales, 128, o.sp_idx, o.sp_val, ophilox.zbar(1, 0, 0, o.sp_idx.size), +1, 1e-3, "E"), o.target_bits)
    assert abs(ref[0].item() - want) <= 1e-4 * want
