"""GPU parity of the step with one dense product per layer (forced by tile configuration 11, or chosen), at the edges of
its tiles: ragged token rows, bands and columns, K with half a chunk at the end, more sensitive entries per chunk than one
group of sixteen and per ring than one refill, no entries, every group size, both tile types, and the outputs."""
import numpy as np
import pytest
import torch

from oracle import layer as olayer, zo as ozo
from paper_2406_02913_amd import szo
from helpers import UpdateBound, clone, make_pair, rel_fro, sigma_g

pytestmark = pytest.mark.gpu

LAYERS = {            # (seed, M, N, K, group, density, mask)
    "one_token_one_row": [(401, 1, 1, 64, 32, 5e-2, "uniform")],
    "half_chunk": [(402, 63, 65, 192, 64, 2e-2, "uniform")],
    "tile_exactly": [(403, 64, 256, 128, 128, 1e-2, "uniform")],
    "one_more_each": [(404, 65, 257, 1088, 32, 1e-3, "uniform")],
    "dense_mask": [(405, 70, 100, 2048, 128, 0.3, "uniform")],        # 2400 entries per chunk: ring and refills
    "hot_rows": [(406, 129, 300, 1024, 128, 1e-2, "heavy_tail")],
    "several": [(407, 200, 320, 512, 128, 2e-3, "uniform"), (408, 5, 64, 320, 64, 0.0, "uniform"),
                (409, 130, 513, 384, 128, 2e-2, "uniform")],
}


@pytest.fixture(autouse=True)
def _auto_tile_config():
    yield
    szo.szo_set_tile_config(0)


def _pairs(name):
    os_, ds_, base = [], [], 0
    for sd, M, N, K, G, dens, kind in LAYERS[name]:
        o, d = make_pair(sd, M, N, K, G, dens, kind=kind, nnz_base=base)
        base += (o.sp_idx.size + 3) // 4 * 4
        os_.append(o)
        ds_.append(d)
    return os_, ds_


@pytest.mark.parametrize("tile", ["f16", "bf16"])
@pytest.mark.parametrize("with_y", [False, True])
@pytest.mark.parametrize("name", sorted(LAYERS))
def test_step_matches_oracle(name, with_y, tile):
    dt = szo.TILE_BF16 if tile == "bf16" else szo.TILE_F16
    os_, ds_ = _pairs(name)
    ref = [clone(o) for o in os_]
    sg, seed, eps, lr = sigma_g(os_), 19, 1e-3, 1e-3
    ws = szo.new_workspace()
    scal = torch.zeros(3, dtype=torch.float64, device="cuda")
    for d in ds_:
        d.y.fill_(float("nan"))
    szo.szo_set_tile_config(11)
    szo.szo_kernel_timing(True)
    bound = UpdateBound(sg, lr)
    for step in range(2):
        z = []
        before = [clone(o) for o in ref]
        szo.szo_zo_step([d.desc(dt, with_y=with_y) for d in ds_], seed, step, eps, lr, scal, ws,
                        0 if with_y else szo.STEP_FUSED_LOSS)
        r = ozo.zo_step(ref, seed, step, eps, lr)
        z = r["z"]
        lp, lm, g = scal.cpu().numpy()
        cells = sum(o.x_bits.shape[0] * o.codes.shape[0] for o in os_)
        # as for the dual-sign tiles: an independent rounding error of ~1e-4 per output, averaged over the outputs
        ltol, gtol = (max(1e-5, 2e-3 / np.sqrt(cells)), 1e-2) if tile == "f16" else (5e-3, 1e-1)
        size = max(r["loss_plus"], 1.0)
        assert abs(lp - r["loss_plus"]) <= ltol * size and abs(lm - r["loss_minus"]) <= ltol * size, (lp, lm, r)
        assert abs(g - r["g"]) <= gtol * max(abs(r["g"]), sg), (g, r["g"], sg)
        bound.add(r, extra_dg=(gtol - 1e-2) * max(abs(r["g"]), sg))
        if with_y and step == 0:        # the outputs are those of the -eps forward; 16-bit operands: 2^-11 / 2^-8 relative
            for o, d, zi in zip(before, ds_, z):
                want = olayer.linear_fwd(o.x_bits, o.codes, o.scales, o.group, o.sp_idx, o.sp_val, zi, -1, eps, "E")
                got = d.y.cpu().numpy()
                assert np.isfinite(got).all() and rel_fro(got, want) <= (5e-4 if tile == "f16" else 4e-3)
    _, launches = szo.szo_kernel_timing_read()
    szo.szo_kernel_timing(False)
    assert launches == 2                                     # one launch per step for all layers and both signs
    for i, (o, d, om) in enumerate(zip(os_, ds_, ref)):
        if o.sp_idx.size:
            bound.check(i, d.sp_val.cpu().numpy(), om.sp_val, o.sp_val)


# One chunk of one band with as many entries as fill half a group, a group, and one more; and none
@pytest.mark.parametrize("group", [128, 64])
@pytest.mark.parametrize("nnz", [0, 1, 7, 8, 9, 15, 16, 17, 24, 25, 33])
def test_groups_of_sensitive_entries(nnz, group):
    o, d = make_pair(440 + nnz, 70, 64, 128, group, nnz=nnz)
    ref = clone(o)
    scal = torch.zeros(3, dtype=torch.float64, device="cuda")
    szo.szo_set_tile_config(11)
    eps = 0.1                                                # z weighs as much as the values: one entry is 1 % of the outputs
    szo.szo_zo_step([d.desc()], 7, 0, eps, 0.0, scal, szo.new_workspace(), 0)
    r = ozo.zo_step([ref], 7, 0, eps, 0.0)
    lp, lm, _ = scal.cpu().numpy()
    ltol = 2e-3 / np.sqrt(70 * 64)                           # as above
    assert abs(lp - r["loss_plus"]) <= ltol * r["loss_plus"] and abs(lm - r["loss_minus"]) <= ltol * r["loss_minus"]
    want = olayer.linear_fwd(o.x_bits, o.codes, o.scales, o.group, o.sp_idx, o.sp_val, r["z"][0], -1, eps, "E")
    assert rel_fro(d.y.cpu().numpy(), want) <= 5e-4


@pytest.mark.parametrize("group,tile", [(128, "f16"), (64, "f16"), (64, "bf16")])
@pytest.mark.parametrize("nnz", [1, 8, 9, 16, 17, 33])
def test_groups_of_sensitive_entries_of_a_sparse_step(nnz, group, tile):
    """The same beside a layer without entries: at 0.03 % the kernel gathers half a group where eight entries or fewer are in it."""
    dt = szo.TILE_BF16 if tile == "bf16" else szo.TILE_F16
    (o, d), (o2, d2) = make_pair(440 + nnz, 70, 64, 128, group, nnz=nnz), make_pair(439, 70, 512, 256, group, nnz=0)
    ref = [clone(o), clone(o2)]
    scal = torch.zeros(3, dtype=torch.float64, device="cuda")
    szo.szo_set_tile_config(11)
    eps = 0.1
    szo.szo_zo_step([d.desc(dt), d2.desc(dt)], 7, 0, eps, 0.0, scal, szo.new_workspace(), 0)
    r = ozo.zo_step(ref, 7, 0, eps, 0.0)
    lp, lm, _ = scal.cpu().numpy()
    ltol = 2e-3 / np.sqrt(70 * 576) if tile == "f16" else 5e-3          # as in test_step_matches_oracle
    assert abs(lp - r["loss_plus"]) <= ltol * r["loss_plus"] and abs(lm - r["loss_minus"]) <= ltol * r["loss_minus"]
    want = olayer.linear_fwd(o.x_bits, o.codes, o.scales, o.group, o.sp_idx, o.sp_val, r["z"][0], -1, eps, "E")
    assert rel_fro(d.y.cpu().numpy(), want) <= (5e-4 if tile == "f16" else 4e-3)


def test_layers_that_share_their_output_buffer_run_one_after_the_other():
    """One buffer for the outputs of a stack holds the last layer's afterwards: concurrent workgroups would mix them."""
    (oa, ob), (da, db) = [list(t) for t in zip(*[make_pair(411 + i, 300, 320, 256, 128, 5e-3, nnz_base=8192 * i) for i in range(2)])]
    results = []
    for shared in (False, True):
        ws = szo.new_workspace()
        scal = torch.zeros(3, dtype=torch.float64, device="cuda")
        descs = [da.desc(), db.desc()]
        if shared:
            descs[0].y = descs[1].y
        szo.szo_zo_step(descs, 3, 0, 1e-3, 0.0, scal, ws, 0)
        results.append((scal.cpu().numpy().copy(), db.y.cpu().numpy().copy()))
    (s0, y0), (s1, y1) = results
    sg = sigma_g([oa, ob])
    assert abs(s0[0] - s1[0]) <= 1e-5 * s0[0] and abs(s0[2] - s1[2]) <= 1e-2 * max(abs(s0[2]), sg)
    assert rel_fro(y1, y0) <= 5e-4


def test_chosen_for_a_step_of_some_hundred_tokens_and_bit_reproducible():
    """... and the entry point without a workspace takes the same kernel: only the grouping of the partials differs."""
    outs = []
    for _ in range(2):
        o, d = make_pair(421, 500, 2048, 512, 128, 1e-3)
        ws = szo.new_workspace()
        scal = torch.zeros(3, dtype=torch.float64, device="cuda")
        szo.szo_kernel_timing(True)
        szo.szo_zo_step([d.desc(with_y=False)], 9, 0, 1e-3, 1e-3, scal, ws, szo.STEP_FUSED_LOSS)
        _, launches = szo.szo_kernel_timing_read()
        szo.szo_kernel_timing(False)
        assert launches == 1
        outs.append((scal.cpu().numpy().copy(), d.sp_val.cpu().numpy().copy()))
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])
    r = ozo.zo_step([clone(o)], 9, 0, 1e-3, 1e-3)
    lp, lm, g = outs[0][0]
    assert abs(lp - r["loss_plus"]) <= 1e-5 * r["loss_plus"] and abs(g - r["g"]) <= 1e-2 * max(abs(r["g"]), sigma_g([o]))
    o, d = make_pair(421, 500, 2048, 512, 128, 1e-3)
    szo.szo_zo_step_noalloc([d.desc(with_y=False)], 9, 0, 1e-3, 1e-3, scal)
    assert np.allclose(scal.cpu().numpy()[:2], outs[0][0][:2], rtol=1e-12, atol=0.0)


@pytest.mark.parametrize("flags", [0, szo.STEP_FUSED_LOSS, szo.STEP_FUSED_LOSS | szo.STEP_ONE_DENSE_PASS])
@pytest.mark.parametrize("M,N,K", [(64, 256, 4096), (65, 200, 384), (129, 70, 128)])
def test_groups_of_128_take_their_scale_in_fp32(M, N, K, flags):
    """No rounding of the dense weights: what is left are fp32 sums of K products, 2^-24 sqrt(K) relative at most for the
    outputs (weights rounded to fp16 after scaling: 1.7e-4) and, averaged over the outputs, far less for the losses."""
    o, d = make_pair(431, M, N, K, 128, 0.0)
    scal = torch.zeros(3, dtype=torch.float64, device="cuda")
    szo.szo_set_tile_config(11)
    szo.szo_zo_step([d.desc(with_y=flags == 0)], 9, 0, 1e-3, 0.0, scal, szo.new_workspace(), flags)
    want = olayer.linear_fwd(o.x_bits, o.codes, o.scales, 128, o.sp_idx, o.sp_val)
    if flags == 0:
        assert rel_fro(d.y.cpu().numpy(), want) <= 2.0 ** -24 * np.sqrt(K)
    loss = olayer.mse_loss(want, o.target_bits)
    assert np.all(np.abs(scal.cpu().numpy()[:2] - loss) <= 1e-7 * loss)


@pytest.mark.parametrize("G", [128, 64])
def test_squares_are_added_in_fp64(G):
    """Zero weights: the differences are the bf16 targets, their squares exact, and the loss is their mean to fp64."""
    o, d = make_pair(441, 70, 300, 256, G, 0.0)
    d.qweight.fill_(0x88)
    scal = torch.zeros(3, dtype=torch.float64, device="cuda")
    szo.szo_set_tile_config(11)
    szo.szo_zo_step([d.desc(with_y=False)], 9, 0, 1e-3, 0.0, scal, szo.new_workspace(), szo.STEP_FUSED_LOSS)
    want = float((d.target.double() ** 2).mean().item())
    assert np.all(np.abs(scal.cpu().numpy()[:2] - want) <= 1e-13 * want)      # 21 000 terms, fp64: 2^-53 sqrt(21 000) = 2e-14


@pytest.mark.parametrize("M,N,K,G,tile", [(16, 700, 512, 64, "bf16"), (16, 700, 192, 64, "f16"), (100, 300, 320, 32, "bf16")])
def test_one_dense_pass_on_request_does_not_lose_the_few_token_path(M, N, K, G, tile):
    """Layers that the stream kernel does not take: the flag changes neither the number of launches nor the result."""
    dt = szo.TILE_BF16 if tile == "bf16" else szo.TILE_F16
    o, d = make_pair(451, M, N, K, G, 1e-2)
    ws, out = szo.new_workspace(), []
    for flags in (szo.STEP_FUSED_LOSS, szo.STEP_FUSED_LOSS | szo.STEP_ONE_DENSE_PASS):
        scal = torch.zeros(3, dtype=torch.float64, device="cuda")
        szo.szo_kernel_timing(True)
        szo.szo_zo_step([d.desc(dt, with_y=False)], 9, 0, 1e-3, 0.0, scal, ws, flags)
        _, launches = szo.szo_kernel_timing_read()
        szo.szo_kernel_timing(False)
        out.append((launches, scal.cpu().numpy().tolist()))
    assert out[0] == out[1] and out[0][0] == 1


@pytest.mark.parametrize("density", [3e-4, 2e-3])            # the form for sparse masks and the other
def test_noalloc_step_on_this_kernel_gives_the_same_g_and_values(density):
    results = []
    for entry in ("workspace", "noalloc"):
        for config in (11, 0):                               # this kernel, and the one that is chosen: the same bits
            szo.szo_set_tile_config(config)
            o, d = make_pair(461, 500, 2048, 512, 128, density)
            scal = torch.zeros(3, dtype=torch.float64, device="cuda")
            szo.szo_kernel_timing(True)
            if entry == "workspace":
                szo.szo_zo_step([d.desc(with_y=False)], 9, 0, 1e-3, 1e-3, scal, szo.new_workspace(), szo.STEP_FUSED_LOSS)
            else:
                szo.szo_zo_step_noalloc([d.desc(with_y=False)], 9, 0, 1e-3, 1e-3, scal)
            _, launches = szo.szo_kernel_timing_read()
            szo.szo_kernel_timing(False)
            assert launches == 1
            results.append((scal.cpu().numpy().copy(), d.sp_val.cpu().numpy().copy(), o))
    for forced, chosen in (results[:2], results[2:]):
        assert np.array_equal(forced[0], chosen[0]) and np.array_equal(forced[1], chosen[1])
    (s0, v0, o), (s1, v1, _) = results[1], results[3]
    assert np.allclose(s0[:2], s1[:2], rtol=1e-12, atol=0.0)                 # the order of the partials
    assert abs(s0[2] - s1[2]) <= 1e-12 * s0[0] / 1e-3                        # ... over 2 eps
    r = ozo.zo_step([clone(o)], 9, 0, 1e-3, 1e-3)
    assert abs(s1[2] - r["g"]) <= 1e-2 * max(abs(r["g"]), sigma_g([o]))
    assert np.max(np.abs(v0 - v1)) <= np.max(np.spacing(np.abs(v0)))


def test_a_bf16_stack_differs_between_the_entry_points_by_the_rounding_of_the_sensitive_weights():
    """Eight layers that one grouped launch computes with v and z rounded one by one, and eight launches of the split kernel
    with v +- eps z rounded: the losses agree to the averaged rounding, g to a few percent of sigma_g, both near the oracle."""
    os_, ds_, base = [], [], 0
    for i in range(8):
        o, d = make_pair(471 + i, 64, 16384, 128, 64, 1e-3, nnz_base=base)
        base += (o.sp_idx.size + 3) // 4 * 4
        os_.append(o)
        ds_.append(d)
    descs = [d.desc(szo.TILE_BF16, with_y=False) for d in ds_]
    out = []
    for entry, want in (("workspace", 1), ("noalloc", 8)):
        scal = torch.zeros(3, dtype=torch.float64, device="cuda")
        szo.szo_kernel_timing(True)
        if entry == "workspace":
            szo.szo_zo_step(descs, 9, 0, 1e-3, 0.0, scal, szo.new_workspace(), szo.STEP_FUSED_LOSS)
        else:
            szo.szo_zo_step_noalloc(descs, 9, 0, 1e-3, 0.0, scal)
        _, launches = szo.szo_kernel_timing_read()
        szo.szo_kernel_timing(False)
        assert launches == want
        out.append(scal.cpu().numpy().copy())
    r, sg = ozo.zo_step([clone(o) for o in os_], 9, 0, 1e-3, 0.0), sigma_g(os_)
    for s in out:                # 2^-9 per weight, averaged over 8 x 10^6 outputs; the bar on g with this tile type is 1e-1
        assert abs(s[0] - r["loss_plus"]) <= 1e-4 * r["loss_plus"] and abs(s[1] - r["loss_minus"]) <= 1e-4 * r["loss_minus"]
        assert abs(s[2] - r["g"]) <= 1e-1 * max(abs(r["g"]), sg)
    assert abs(out[0][2] - out[1][2]) <= 1e-1 * max(abs(r["g"]), sg)


@pytest.mark.parametrize("M,N,K,G,density,tile", [
    (513, 2048, 512, 128, 1e-3, "f16"),         # the first size beyond 512 tokens: nine rows of tiles, the last of one token row
    (2048, 300, 512, 128, 2e-3, "f16"), (2049, 256, 256, 128, 3e-3, "f16"),      # either side of the limit on tokens (few tiles)
    (705, 3392, 320, 64, 1e-3, "bf16"),         # the other line: tile type, half a chunk at the end, one token row in the last tiles
])
def test_chosen_beyond_512_tokens_and_equal_to_two_forwards(M, N, K, G, density, tile):
    """Losses, g and the updated values of the step against two perturbed forwards of the same layer on the tiled kernel:
    they differ by the rounding of the weights after scaling (2^-11, 2^-8 with the bf16 tile) averaged over the outputs."""
    dt = szo.TILE_BF16 if tile == "bf16" else szo.TILE_F16
    o, d = make_pair(481, M, N, K, G, density)
    v0 = d.sp_val.cpu().numpy().copy()
    ws, scal, lr = szo.new_workspace(), torch.zeros(3, dtype=torch.float64, device="cuda"), 1e-2
    two = torch.zeros(2, dtype=torch.float64, device="cuda")
    szo.szo_set_tile_config(2)
    for sign in (1, -1):
        szo.szo_linear_fwd_mse(d.desc(dt, with_y=False), 9, 3, sign, 1e-3, 1.0 / (M * N), two[(1 - sign) // 2:(1 - sign) // 2 + 1], ws)
    forced = torch.zeros(3, dtype=torch.float64, device="cuda")
    szo.szo_set_tile_config(11)
    szo.szo_zo_step([d.desc(dt, with_y=False)], 9, 3, 1e-3, 0.0, forced, ws, szo.STEP_FUSED_LOSS)
    szo.szo_set_tile_config(0)
    szo.szo_kernel_timing(True)
    szo.szo_zo_step([d.desc(dt, with_y=False)], 9, 3, 1e-3, lr, scal, ws, szo.STEP_FUSED_LOSS)
    _, launches = szo.szo_kernel_timing_read()
    szo.szo_kernel_timing(False)
    assert launches == 1 and np.array_equal(scal.cpu().numpy(), forced.cpu().numpy())        # the kernel under test is the one that ran
    (lp, lm, g), want, sg = scal.cpu().numpy(), two.cpu().numpy(), sigma_g([o])
    ltol, gtol = (1e-5, 1e-2) if tile == "f16" else (1e-3, 1e-1)          # the bars of the tiled kernel against the oracle
    assert abs(lp - want[0]) <= ltol * want[0] and abs(lm - want[1]) <= ltol * want[1]
    want_g = (want[0] - want[1]) / (2.0 * float(np.float32(1e-3)))
    assert abs(g - want_g) <= 2 * gtol * max(abs(want_g), sg)
    z = ozo.zo_step([clone(o)], 9, 3, 1e-3, lr)["z"][0]
    moved = d.sp_val.cpu().numpy().astype(np.float64) - v0
    assert np.max(np.abs(moved + float(np.float32(lr)) * g * z)) <= 1e-5 * abs(lr * g) * 6 + np.spacing(np.float32(0.2))


def test_a_large_step_and_its_layers_one_by_one_agree_to_the_roundings():
    """Two layers whose tiles are together beyond the line for one dense product and each within it: two full products in one step, one
    in the steps by themselves.  Weights rounded with and without the sensitive part (2^-11) average out over 4 x 10^7 outputs."""
    ds_, os_, base = [], [], 0
    for i in range(2):
        o, d = make_pair(491 + i, 2049, 16384, 128, 128, 1e-3, nnz_base=base)
        base += (o.sp_idx.size + 3) // 4 * 4
        os_.append(o)
        ds_.append(d)
    ws, alone, scal = szo.new_workspace(), [], torch.zeros(3, dtype=torch.float64, device="cuda")
    for d in ds_:
        forced = torch.zeros(3, dtype=torch.float64, device="cuda")
        szo.szo_zo_step([d.desc(with_y=False)], 9, 0, 1e-3, 0.0, scal, ws, szo.STEP_FUSED_LOSS)
        szo.szo_set_tile_config(11)
        szo.szo_zo_step([d.desc(with_y=False)], 9, 0, 1e-3, 0.0, forced, ws, szo.STEP_FUSED_LOSS)
        szo.szo_set_tile_config(0)
        assert np.array_equal(scal.cpu().numpy(), forced.cpu().numpy())
        alone.append(scal.cpu().numpy().copy())
    szo.szo_zo_step([d.desc(with_y=False) for d in ds_], 9, 0, 1e-3, 0.0, scal, ws, szo.STEP_FUSED_LOSS)
    together, want = scal.cpu().numpy().copy(), alone[0] + alone[1]
    szo.szo_set_tile_config(11)
    szo.szo_zo_step([d.desc(with_y=False) for d in ds_], 9, 0, 1e-3, 0.0, scal, ws, szo.STEP_FUSED_LOSS)
    assert not np.array_equal(together, scal.cpu().numpy())                 # another kernel, other roundings
    assert np.all(np.abs(together[:2] - want[:2]) <= 1e-5 * want[:2])      # the bar of the tiled kernel's losses against the oracle
    assert abs(together[2] - want[2]) <= 2e-2 * max(abs(want[2]), sigma_g(os_))          # 1e-2 for either side
