"""GPU parity of the fused forward against the fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import layer as olayer, philox as ophilox
from oracle.quant import bf16_bits_to_f64
from paper_2406_02913_amd import szo
from helpers import make_pair, rel_fro

pytestmark = pytest.mark.gpu

# (seed, M, N, K, group, density): tiny config, several tiles, ragged M and N, dense-ish masks
SHAPES = [
    (1, 64, 256, 256, 32, 1e-3),        # the tiny single-layer configuration
    (2, 100, 200, 320, 64, 1e-2),       # ragged M and N
    (3, 300, 384, 1024, 128, 1e-3),     # several tiles each way
    (4, 1, 128, 128, 128, 5e-2),        # a single token, dense mask
    (5, 257, 130, 192, 32, 0.0),        # k = 0: plain dequantise-then-matmul
    (6, 129, 513, 512, 128, 2e-2),      # one row past a tile boundary in both
    (7, 70, 192, 4160, 64, 1e-1),       # 65 column tiles (tile_ptr reload) and > 256 entries per tile
]
DTYPES = [(szo.TILE_F16, "f16", 2e-5), (szo.TILE_BF16, "bf16", 2e-5)]


def _run(d, sign, eps, seed, step, dt):
    d.y.fill_(float("nan"))
    szo.szo_linear_fwd(d.desc(dt), seed, step, sign, eps)
    torch.cuda.synchronize()
    return d.y.cpu().numpy()


@pytest.fixture(autouse=True)
def _auto_tile_config():
    yield
    szo.szo_set_tile_config(0)


@pytest.mark.parametrize("tile_cfg", [1, 2])
@pytest.mark.parametrize("dt,dtname,tol_d", DTYPES)
@pytest.mark.parametrize("shape", SHAPES)
def test_forward_matches_oracle(shape, dt, dtname, tol_d, tile_cfg):
    szo.szo_set_tile_config(tile_cfg)
    s, M, N, K, G, dens = shape
    o, d = make_pair(s, M, N, K, G, dens, nnz_base=8)
    seed, step, eps = 1234, 3, 1e-3
    z = ophilox.zbar(seed, step, 8, o.sp_idx.size)
    for sign in (+1, -1, 0):
        y = _run(d, sign, eps, seed, step, dt)
        assert np.isfinite(y).all()
        yD = olayer.linear_fwd(o.x_bits, o.codes, o.scales, G, o.sp_idx, o.sp_val, z, sign, eps, "D", dtname)
        yE = olayer.linear_fwd(o.x_bits, o.codes, o.scales, G, o.sp_idx, o.sp_val, z, sign, eps, "E")
        assert rel_fro(y, yD) <= tol_d, (sign, rel_fro(y, yD))
        assert rel_fro(y, yE) <= 5e-3, (sign, rel_fro(y, yE))
        # element-wise: fp32 accumulation of exact products over K terms
        scale = np.sqrt(K) * 0.02 * 4
        assert np.max(np.abs(y - yD)) <= 1e-4 * scale + 1e-6


# One 64 x 64 tile with none, one, as many entries as the schedule scatters by itself, and one more; then all of them
@pytest.mark.parametrize("tile_cfg", [1, 2])
@pytest.mark.parametrize("nnz", [0, 1, 64, 65, 4096])
def test_entries_of_a_tile(nnz, tile_cfg):
    szo.szo_set_tile_config(tile_cfg)
    for dt, dtname, tol in DTYPES:
        o, d = make_pair(60, 70, 64, 64, 32, nnz=nnz)
        # v - eps z is formed in fp32: where its error crosses a rounding boundary of the tile type the weight is an ulp off.  With
        # eps = 1e-3 that error is the last rounding's, 2^-25 of the weight: a share of at most 2^-16 / 2^-13 of the weights by 2^-8 /
        # 2^-11 (bf16 / fp16), 1.5e-5 / 6e-6 of the result if all are sensitive (with eps = 0.1 the error of z does so more often)
        z = ophilox.zbar(9, 2, 0, o.sp_idx.size)
        y = _run(d, -1, 1e-3, 9, 2, dt)
        want = olayer.linear_fwd(o.x_bits, o.codes, o.scales, 32, o.sp_idx, o.sp_val, z, -1, 1e-3, "D", dtname)
        assert rel_fro(y, want) <= tol


# More than the schedule of 128-row tiles scatters by itself: the rest of a tile stands behind it, in this window of 256 entries or the next
@pytest.mark.parametrize("nnz", [63, 66, 127, 128, 129, 191, 255, 256, 257, 320])
def test_entries_beyond_the_schedule(nnz):
    szo.szo_set_tile_config(1)
    for dt, dtname, tol in DTYPES:
        o, d = make_pair(61, 70, 128, 192, 32, nnz=nnz)         # two bands and three tiles of columns, their entries one after the other
        z = ophilox.zbar(9, 2, 0, o.sp_idx.size)
        y = _run(d, -1, 1e-3, 9, 2, dt)
        want = olayer.linear_fwd(o.x_bits, o.codes, o.scales, 32, o.sp_idx, o.sp_val, z, -1, 1e-3, "D", dtname)
        assert rel_fro(y, want) <= tol
        o, d = make_pair(62, 70, 64, 256, 32, nnz=4 * nnz)      # about that many in each of four tiles
        z = ophilox.zbar(9, 2, 0, o.sp_idx.size)
        y = _run(d, +1, 1e-3, 9, 2, dt)
        want = olayer.linear_fwd(o.x_bits, o.codes, o.scales, 32, o.sp_idx, o.sp_val, z, +1, 1e-3, "D", dtname)
        assert rel_fro(y, want) <= tol


# 128 x 128 tiles with K in two parts: the shortest K and one above it, both tile types, ragged and half-empty tiles, tiles with more
# entries than their schedule; 192 columns (an odd number of K steps) and 128 (one step for each part) stay whole
@pytest.mark.parametrize("M,N,K,G,dens,dt,dtname", [
    (500, 300, 256, 32, 1e-2, szo.TILE_F16, "f16"), (513, 130, 384, 128, 0.0, szo.TILE_F16, "f16"), (600, 60, 512, 64, 0.2, szo.TILE_F16, "f16"),
    (2100, 1000, 256, 64, 2e-3, szo.TILE_BF16, "bf16"), (513, 200, 128, 32, 1e-2, szo.TILE_F16, "f16"),
    (500, 70, 8448, 64, 0.2, szo.TILE_F16, "f16"),                 # 66 tiles of columns per part (tile bounds are loaded 64 at a time)
    (2100, 1000, 192, 32, 1e-2, szo.TILE_F16, "f16")])
def test_tiles_with_k_in_two_parts(M, N, K, G, dens, dt, dtname):
    o, d = make_pair(63, M, N, K, G, dens, nnz_base=4)
    z = ophilox.zbar(9, 2, 4, o.sp_idx.size)
    ws, loss = szo.new_workspace(), torch.zeros(1, dtype=torch.float64, device="cuda")
    for sign in (+1, -1):
        y = _run(d, sign, 1e-3, 9, 2, dt)
        want = olayer.linear_fwd(o.x_bits, o.codes, o.scales, G, o.sp_idx, o.sp_val, z, sign, 1e-3, "D", dtname)
        assert rel_fro(y, want) <= 2e-5                            # the bar of the shapes above: K exact products summed in fp32
        szo.szo_set_tile_config(1)                                 # the same tiles, K whole: other sums exactly where K is cut
        assert np.array_equal(y, _run(d, sign, 1e-3, 9, 2, dt)) == (K % 128 != 0 or K < 256)
        szo.szo_set_tile_config(0)
        loss.zero_()
        d.y.fill_(float("nan"))
        szo.szo_linear_fwd_mse(d.desc(dt), 9, 2, sign, 1e-3, 1.0 / (M * N), loss, ws)
        assert np.array_equal(d.y.cpu().numpy(), y)
        # the loss of these very outputs: squares and the sums of sixteen of them in fp32 (16 x 2^-24), the rest in fp64
        err = y.astype(np.float64) - bf16_bits_to_f64(o.target_bits)
        assert abs(loss.item() / (np.sum(err * err) / (M * N)) - 1.0) <= 18 * 2.0 ** -24


# 128 x 128 tiles with K whole, the library choosing: blocks of 32 x 32 (fp16: up to 320 tiles, 384 with denser masks; bf16), blocks of 16 x
# 16 beyond; ragged tiles, half-empty ones, tiles with more entries than their schedule; targets staged (rows of 16 bytes) and not
@pytest.mark.parametrize("M,N,K,G,dens,dt,dtname", [
    (2100, 2400, 192, 64, 2e-3, szo.TILE_F16, "f16"), (2100, 2608, 192, 32, 2e-3, szo.TILE_F16, "f16"), (2100, 2608, 192, 32, 1e-2, szo.TILE_F16, "f16"),
    (2100, 2608, 192, 32, 2e-3, szo.TILE_BF16, "bf16"), (500, 300, 448, 64, 0.2, szo.TILE_F16, "f16"), (513, 130, 64, 32, 0.2, szo.TILE_BF16, "bf16"),
    (1100, 70, 4160, 64, 0.1, szo.TILE_F16, "f16")])
def test_whole_small_tiles(M, N, K, G, dens, dt, dtname):
    o, d = make_pair(65, M, N, K, G, dens, nnz_base=4)
    z = ophilox.zbar(9, 2, 4, o.sp_idx.size)
    ws, loss = szo.new_workspace(), torch.zeros(2, dtype=torch.float64, device="cuda")
    for sign in (+1, -1):
        y = _run(d, sign, 1e-3, 9, 2, dt)
        want = olayer.linear_fwd(o.x_bits, o.codes, o.scales, G, o.sp_idx, o.sp_val, z, sign, 1e-3, "D", dtname)
        assert rel_fro(y, want) <= 2e-5
        loss.zero_()
        d.y.fill_(float("nan"))
        szo.szo_linear_fwd_mse(d.desc(dt), 9, 2, sign, 1e-3, 1.0 / (M * N), loss[:1], ws)
        szo.szo_linear_fwd_mse(d.desc(dt, with_y=False), 9, 2, sign, 1e-3, 1.0 / (M * N), loss[1:], ws)
        assert np.array_equal(d.y.cpu().numpy(), y) and loss[0].item() == loss[1].item()
        err = y.astype(np.float64) - bf16_bits_to_f64(o.target_bits)     # squares and the sums of sixteen of them in fp32, the rest in fp64
        assert abs(loss[0].item() / (np.sum(err * err) / (M * N)) - 1.0) <= 18 * 2.0 ** -24


# Rows of y at any multiple of four bytes: quads side by side trade rows where they do not begin at multiples of 16.  K in two parts, whole
# with blocks of 16 x 16 and of 32 x 32, 256 x 256 tiles, tables with either block; full and ragged tiles; targets staged (rows of 16 bytes) and not
@pytest.mark.parametrize("cfg,M,N,K,fmt", [(0, 513, 130, 384, "uniform"), (0, 384, 256, 256, "uniform"), (0, 2100, 2608, 192, "uniform"), (0, 2100, 2609, 192, "uniform"),
                                           (0, 2100, 2609, 1088, "uniform"), (0, 700, 513, 192, "lut"), (0, 3500, 3072, 64, "lut"), (2, 300, 520, 128, "uniform"), (2, 512, 513, 128, "uniform"), (2, 300, 520, 128, "lut")])
def test_outputs_at_any_alignment(cfg, M, N, K, fmt):
    szo.szo_set_tile_config(cfg)
    o, d = make_pair(66, M, N, K, 64, 2e-3, nnz_base=4, fmt=fmt)
    y = torch.from_numpy(_run(d, +1, 1e-3, 9, 2, szo.TILE_F16))
    z = ophilox.zbar(9, 2, 4, o.sp_idx.size)
    assert rel_fro(y, olayer.linear_fwd(o.x_bits, o.codes, o.scales, 64, o.sp_idx, o.sp_val, z, +1, 1e-3, "D", "f16", lut=o.lut)) <= 2e-5
    ws, loss = szo.new_workspace(), torch.zeros(1, dtype=torch.float64, device="cuda")
    szo.szo_linear_fwd_mse(d.desc(with_y=False), 9, 2, +1, 1e-3, 1.0 / (M * N), loss, ws)
    want = loss.item()
    for first in (256, 257, 258, 259, 260):
        guarded = torch.full((M * N + 512,), 7.5, device="cuda")
        d.y = guarded[first:first + M * N].view(M, N)
        szo.szo_linear_fwd(d.desc(), 9, 2, +1, 1e-3)
        assert torch.equal(d.y.cpu(), y)
        d.y.fill_(float("nan"))
        loss.zero_()
        szo.szo_linear_fwd_mse(d.desc(), 9, 2, +1, 1e-3, 1.0 / (M * N), loss, ws)
        assert torch.equal(d.y.cpu(), y) and loss.item() == want
        assert bool((guarded[:first] == 7.5).all()) and bool((guarded[first + M * N:] == 7.5).all())


def test_perturbation_difference_is_linear_in_z():
    # y(+) - y(-) = 2 eps x Z^T: checks the sign convention and that only masked entries move
    o, d = make_pair(7, 96, 256, 256, 32, 5e-3)
    seed, step, eps = 5, 1, 1e-2
    z = ophilox.zbar(seed, step, 0, o.sp_idx.size)
    yp = _run(d, +1, eps, seed, step, szo.TILE_F16).astype(np.float64)
    ym = _run(d, -1, eps, seed, step, szo.TILE_F16).astype(np.float64)
    from oracle.quant import bf16_bits_to_f64
    x = bf16_bits_to_f64(o.x_bits)
    Z = np.zeros((256, 256))
    Z.reshape(-1)[o.sp_idx.astype(np.int64)] = z
    want = 2 * float(np.float32(eps)) * x @ Z.T
    assert rel_fro(yp - ym, want) < 2e-2


def test_forward_is_deterministic_and_leaves_inputs_untouched():
    o, d = make_pair(8, 128, 256, 512, 128, 1e-2)
    before = d.sp_val.clone()
    a = _run(d, +1, 1e-3, 1, 0, szo.TILE_F16)
    b = _run(d, +1, 1e-3, 1, 0, szo.TILE_F16)
    assert np.array_equal(a, b)
    assert torch.equal(before, d.sp_val)


@pytest.mark.parametrize("tile_cfg", [1, 2])
def test_fused_loss_equals_separate_loss(tile_cfg):
    szo.szo_set_tile_config(tile_cfg)
    o, d = make_pair(9, 200, 384, 512, 128, 1e-2)
    ws = szo.new_workspace()
    seed, step, eps = 2, 2, 1e-3
    for dt in (szo.TILE_F16, szo.TILE_BF16):
        y = _run(d, -1, eps, seed, step, dt)
        acc = torch.zeros(2, dtype=torch.float64, device="cuda")
        szo.szo_mse_loss(d.y, d.target, d.M * d.N, 1.0 / (d.M * d.N), acc[0:1], ws)
        d.y.fill_(0)
        szo.szo_linear_fwd_mse(d.desc(dt), seed, step, -1, eps, 1.0 / (d.M * d.N), acc[1:2], ws)
        torch.cuda.synchronize()
        assert np.array_equal(d.y.cpu().numpy(), y)                 # y still written when requested
        a = acc.cpu().numpy()
        # the fused epilogue squares in fp32 and adds 16-term fp32 partials in fp64: per-term relative
        # rounding 2^-24, random in sign, so the sum of ~77k terms agrees to far better than 1e-8
        assert abs(a[0] - a[1]) <= 1e-8 * abs(a[0])
        assert abs(a[0] - olayer.mse_loss(y.astype(np.float64), o.target_bits)) <= 1e-12 * abs(a[0])
        acc2 = torch.zeros(1, dtype=torch.float64, device="cuda")
        szo.szo_linear_fwd_mse(d.desc(dt, with_y=False), seed, step, -1, eps, 1.0 / (d.M * d.N), acc2, ws)
        assert acc2.item() == a[1]                                  # no y, same loss, bit for bit
