"""GPU parity of the tiled kernel that computes one dense product for both forwards and the sensitive products behind it (forced by
tile configuration 12, or chosen): ragged tiles, bands with no entries, with one more than a group of thirty-two and with more than
are held at once, targets that are not staged, both tile types, infinite activations, and steps that take more than one launch."""
import numpy as np
import pytest
import torch

from oracle import zo as ozo
from paper_2406_02913_amd import szo
from helpers import UpdateBound, clone, make_pair, sigma_g

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _auto_tile_config():
    yield
    szo.szo_set_tile_config(0)


def _step(descs, config, lr=0.0, eps=1e-3, seed=9, step=0):
    scal = torch.zeros(3, dtype=torch.float64, device="cuda")
    szo.szo_set_tile_config(config)
    szo.szo_kernel_timing(True)
    szo.szo_zo_step(descs, seed, step, eps, lr, scal, szo.new_workspace(), szo.STEP_FUSED_LOSS)
    _, launches = szo.szo_kernel_timing_read()
    szo.szo_kernel_timing(False)
    assert launches == 1                                     # one pair of events, around all launches of a step
    return scal.cpu().numpy().copy()


LAYERS = {            # (seed, M, N, K, group, density, mask)
    "one_token_one_row": [(801, 1, 1, 64, 32, 5e-2, "uniform")],
    "tile_exactly": [(802, 256, 256, 128, 128, 1e-2, "uniform")],
    "one_more_each": [(803, 257, 257, 1088, 64, 1e-3, "uniform")],        # targets not staged
    "half_a_tile": [(804, 129, 200, 320, 32, 2e-2, "uniform")],
    "dense_mask": [(805, 70, 128, 2048, 128, 0.1, "uniform")],            # 13 000 entries per band: the window is refilled
    "hot_rows": [(806, 300, 648, 1024, 128, 1e-2, "heavy_tail")],
    "several": [(807, 200, 320, 512, 128, 2e-3, "uniform"), (808, 5, 64, 320, 64, 0.0, "uniform"),
                (809, 330, 513, 384, 128, 2e-2, "uniform")],
}


@pytest.mark.parametrize("tile", ["f16", "bf16"])
@pytest.mark.parametrize("name", sorted(LAYERS))
def test_step_matches_oracle(name, tile):
    dt = szo.TILE_BF16 if tile == "bf16" else szo.TILE_F16
    os_, ds_, base = [], [], 0
    for sd, M, N, K, G, dens, kind in LAYERS[name]:
        o, d = make_pair(sd, M, N, K, G, dens, kind=kind, nnz_base=base)
        base += (o.sp_idx.size + 3) // 4 * 4
        os_.append(o)
        ds_.append(d)
    ref = [clone(o) for o in os_]
    sg, eps, lr = sigma_g(os_), 1e-3, 1e-3
    bound = UpdateBound(sg, lr)
    # as for the dual-sign tiles: an independent rounding error of ~1e-4 per output, averaged over the outputs
    cells = sum(o.x_bits.shape[0] * o.codes.shape[0] for o in os_)
    ltol, gtol = (max(1e-5, 2e-3 / np.sqrt(cells)), 1e-2) if tile == "f16" else (5e-3, 1e-1)
    for step in range(2):
        lp, lm, g = _step([d.desc(dt, with_y=False) for d in ds_], 12, lr, eps, 19, step)
        r = ozo.zo_step(ref, 19, step, eps, lr)
        size = max(r["loss_plus"], 1.0)
        assert abs(lp - r["loss_plus"]) <= ltol * size and abs(lm - r["loss_minus"]) <= ltol * size, (lp, lm, r)
        assert abs(g - r["g"]) <= gtol * max(abs(r["g"]), sg), (g, r["g"], sg)
        bound.add(r, extra_dg=(gtol - 1e-2) * max(abs(r["g"]), sg))
    for i, (o, d, om) in enumerate(zip(os_, ds_, ref)):
        if o.sp_idx.size:
            bound.check(i, d.sp_val.cpu().numpy(), om.sp_val, o.sp_val)


# entries of one band: none, around a group, around what is held at once (480), and the second half of the rows after refills
@pytest.mark.parametrize("nnz", [1, 31, 32, 33, 479, 480, 481, 1000])
def test_groups_of_sensitive_entries(nnz):
    o, d = make_pair(840 + nnz, 130, 64, 128, 128, nnz=nnz)
    eps = 0.1                                                # z weighs as much as the values: one entry is 1 % of the outputs
    lp, lm, g = _step([d.desc(with_y=False)], 12, eps=eps)
    r = ozo.zo_step([clone(o)], 9, 0, eps, 0.0)
    ltol = 2e-3 / np.sqrt(130 * 64)                          # as above
    assert abs(lp - r["loss_plus"]) <= ltol * r["loss_plus"] and abs(lm - r["loss_minus"]) <= ltol * r["loss_minus"]
    assert abs(g - r["g"]) <= 1e-2 * max(abs(r["g"]), sigma_g([o]))


@pytest.mark.parametrize("what", ["infinite", "overflow"])
def test_losses_are_infinite_where_every_output_has_a_value(what):
    """As on the tiled kernel that adds the sensitive weights to the weight tile first (configuration 1)."""
    o, d = make_pair(860, 70, 5, 320, 64, 2e-2)
    column = int(np.flatnonzero((o.codes != 8).all(axis=0))[0])
    if what == "infinite":
        d.x[11, column] = float("inf")
    else:
        d.x[11].fill_(0)
        d.x[11, column] = 3e38
        d.scales.fill_(100.0)
    values = d.sp_val.clone()
    for eps in (1e-3, 0.0):
        for config in (1, 12):
            d.sp_val.copy_(values)
            scal = torch.zeros(3, dtype=torch.float64, device="cuda")
            szo.szo_set_tile_config(config)
            szo.szo_zo_step([d.desc(szo.TILE_BF16, with_y=False)], 3, 1, eps, 0.0, scal, szo.new_workspace(), szo.STEP_FUSED_LOSS)
            assert np.isposinf(scal.cpu().numpy()[:2]).all(), (config, eps, scal)


def test_a_nan_spoils_the_losses():
    _, d = make_pair(861, 300, 70, 320, 64, 2e-2)
    d.x[270, 5] = float("nan")
    assert np.isnan(_step([d.desc(with_y=False)], 12)[:2]).all()


def _stack(seed, n, M, N, K, density, same_x, group=128, tile=szo.TILE_F16):
    """n descriptors of one layer, each with activations of its own (or one set for all)."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    _, d = make_pair(seed, 64, N, K, group, density)
    keep, descs = [d], []
    for i in range(n):
        if i == 0 or not same_x:
            keep.append(torch.randn((M, K), generator=gen, device="cuda", dtype=torch.bfloat16))
        desc = d.desc(tile, with_y=False)
        desc.M, desc.x = M, keep[-1].data_ptr()
        descs.append(desc)
    target = torch.randn((M, N), generator=gen, device="cuda", dtype=torch.bfloat16)
    for desc in descs:
        desc.target = target.data_ptr()
    return descs, keep + [target]


def _gradient(d, desc, x, target):
    """Of the layer's loss with respect to its sensitive values, in fp32 from the unperturbed outputs: g = gradient . z."""
    y = torch.empty(target.shape, dtype=torch.float32, device="cuda")
    plain = type(desc).from_buffer_copy(desc)
    plain.y = y.data_ptr()
    szo.szo_linear_fwd(plain, 0, 0, 0, 0.0)
    r = (y - target.float()) * (2.0 / y.numel())
    return (r.T @ x.float()).reshape(-1)[d.sp_idx.long()].double()


def _sigma_of_stack(descs, keep):
    """As helpers.sigma_g, of layers with the same z (_stack)."""
    xs = {x.data_ptr(): x for x in keep[1:-1]}
    total = sum(_gradient(keep[0], desc, xs[desc.x], keep[-1]) for desc in descs)
    return float(total.norm())


@pytest.mark.parametrize("same_x", [False, True])
def test_a_step_of_several_launches_is_the_sum_of_its_layers(same_x):
    """Five layers whose activations, 256 MiB each, do not all fit the workspace at once (or are one and the same)."""
    descs, keep = _stack(871, 5, 8192, 64, 16384, 1e-4, same_x)
    alone = [_step([d], 12) for d in descs]
    s = _step(descs, 12)
    total = np.sum(alone, axis=0)
    assert np.allclose(s[:2], total[:2], rtol=1e-12, atol=0.0)               # the order of the partials
    assert abs(s[2] - total[2]) <= 1e-12 * s[0] / 1e-3                       # ... over 2 eps
    one_pass = _step(descs, 11)
    assert np.allclose(s[:2], one_pass[:2], rtol=1e-5, atol=0.0)             # the scale rounded once per weight or not at all
    assert abs(s[2] - one_pass[2]) <= 1e-2 * max(abs(one_pass[2]), _sigma_of_stack(descs, keep))


@pytest.mark.parametrize("density,config", [(1e-3, 12), (1e-2, 6)])
def test_chosen_for_large_steps_with_sparse_masks(density, config):
    """One layer short of 4096 tiles of 256 x 256 the products of the single-layer calls, beyond them the dense product once or, with denser
    masks, still twice."""
    descs, keep = _stack(881, 29, 2304, 4096, 1024, density, True)
    assert np.array_equal(_step(descs[:28], 0), _step(descs[:28], 6))        # 4032 tiles
    chosen = _step(descs, 0)
    assert np.array_equal(chosen, _step(descs, 0)) and np.array_equal(chosen, _step(descs, config))
    other = _step(descs, 18 - config)
    assert not np.array_equal(chosen, other) and np.allclose(chosen[:2], other[:2], rtol=1e-5, atol=0.0)
    # the sensitive products, which are 1e-6 of the losses
    assert abs(chosen[2] - other[2]) <= 1e-2 * max(abs(other[2]), _sigma_of_stack(descs, keep))


@pytest.mark.parametrize("group,tile", [(128, "f16"), (64, "f16"), (128, "bf16")])
def test_chosen_from_512_tiles_on_where_both_kernels_round_the_weights(group, tile):
    """The kernel with tiles of 64 token rows has groups of 128 with the fp16 tile, which it does not round, and fewer tiles; asked for
    or not."""
    descs, keep = _stack(891, 11, 768, 4096, 1024, 1e-3, True, group, szo.TILE_BF16 if tile == "bf16" else szo.TILE_F16)
    for n, config in ((10, 11), (11, 11 if (group, tile) == (128, "f16") else 12)):        # 480 and 528 tiles
        chosen, other = _step(descs[:n], 0), _step(descs[:n], 23 - config)
        assert np.array_equal(chosen, _step(descs[:n], config)) and not np.array_equal(chosen, other)
        assert np.allclose(chosen[:2], other[:2], rtol=1e-5, atol=0.0)
        assert abs(chosen[2] - other[2]) <= 1e-2 * max(abs(other[2]), _sigma_of_stack(descs[:n], keep))
        asked = torch.zeros(3, dtype=torch.float64, device="cuda")
        szo.szo_set_tile_config(0)
        szo.szo_zo_step(descs[:n], 9, 0, 1e-3, 0.0, asked, szo.new_workspace(), szo.STEP_FUSED_LOSS | szo.STEP_ONE_DENSE_PASS)
        assert np.array_equal(chosen, asked.cpu().numpy())


@pytest.mark.parametrize("group,tile", [(128, "bf16"), (64, "f16")])
def test_steps_beyond_4096_tiles_keep_the_sums_of_two_products(group, tile):
    """... sixteen at a time in fp32 whatever the layers; forced on such layers, the kernel adds them one by one in fp64."""
    descs, keep = _stack(885, 29, 2304, 4096, 1024, 1e-3, True, group, szo.TILE_BF16 if tile == "bf16" else szo.TILE_F16)
    chosen, forced, two = _step(descs, 0), _step(descs, 12), _step(descs, 6)
    assert not np.array_equal(chosen, forced) and np.allclose(chosen[:2], forced[:2], rtol=1e-8, atol=0.0)
    # 4e-9 of both losses at most, their difference is summed as such; against two products as test_step_matches_oracle
    sigma = _sigma_of_stack(descs, keep)
    assert abs(chosen[2] - forced[2]) <= 1e-3 * sigma
    assert np.allclose(chosen[:2], two[:2], rtol=1e-5 if tile == "f16" else 1e-3, atol=0.0)
    assert abs(chosen[2] - two[2]) <= (1e-2 if tile == "f16" else 1e-1) * max(abs(two[2]), sigma)


@pytest.mark.parametrize("tile", ["f16", "bf16"])
@pytest.mark.parametrize("M,N", [(256, 512), (300, 520), (70, 257)])        # whole tiles, ragged ones, targets that are not staged
def test_losses_are_added_in_fp64(M, N, tile):
    """Zero weights and one sensitive entry of value zero in every row of W: with x in eighths the outputs +- eps x z are exact in fp32, and
    so are their squares in fp64.  What is left is the order of those sums, 2^-53 of the loss per term and far less in the mean (1e-13 is a
    fifth of all M N of the smallest roundings one way); sixteen terms at a time in fp32, as where the weights are rounded by this kernel
    alone (fp16 tile, groups of 128), leave up to 4e-9."""
    dt, as16 = (szo.TILE_BF16, torch.bfloat16) if tile == "bf16" else (szo.TILE_F16, torch.float16)
    K, group, eps, seed, step = 128, 64, 0.5, 7, 3
    gen = torch.Generator(device="cuda").manual_seed(N)
    column = torch.randint(K, (N,), generator=gen, device="cuda")
    tile_ptr, sp_idx, _ = szo.szo_tcsr_build(N, K, (torch.arange(N, device="cuda") * K + column).cpu().numpy().astype(np.uint32))
    q, scales = np.full((N, K // 2), 0x88, dtype=np.uint8), np.full((N, K // group), 0.01, dtype=np.float16)
    q, scales = szo.szo_layout_weights(q, scales, group)
    dev = lambda a, t: torch.from_numpy(a.view(t)).cuda()
    idx, ptr, qd, sd = dev(sp_idx, np.int32), dev(tile_ptr, np.int32), dev(q, np.uint8), dev(scales, np.float16)
    x = (torch.randint(-64, 65, (M, K), generator=gen, device="cuda") / 8.0).bfloat16()
    target, values = torch.randn((M, N), generator=gen, device="cuda").bfloat16(), torch.zeros(N, device="cuda")
    desc = szo.make_desc(M, N, K, group, N, 0, x, qd, sd, ptr, idx, values, None, target, dt)
    lp, lm, _ = _step([desc], 12, eps=eps, seed=seed, step=step)
    z = torch.empty(N, device="cuda")
    szo.szo_debug_zbar(0, N, seed, step, None, z)
    flat = idx.long()
    Z = torch.zeros((M, N), dtype=torch.float64, device="cuda")
    Z[:, flat // K] = x.double()[:, flat % K] * z.to(as16).double()
    for got, sign in ((lp, 1.0), (lm, -1.0)):
        want = float(((sign * eps * Z - target.double()) ** 2).mean())
        assert abs(got - want) <= 1e-13 * want, (got, want)


def _many_launches(n=153, columns=(1920,), M=16384):
    """Layers with activations of their own (views of one tensor, a row apart), 63 MB each as a copy for 1920 columns: 17 of those fit the
    workspace, more than travel in the kernel arguments.  153 make nine launches.  -> descriptors, [(d, desc, x, target)] of each"""
    gen = torch.Generator(device="cuda").manual_seed(907)
    rows = lambda K: torch.randn((M + n, K), generator=gen, device="cuda", dtype=torch.bfloat16)
    kinds = [(make_pair(907 + K, 64, 64, K, 128, 1e-3)[1], rows(K)) for K in columns]
    targets = rows(64)
    layers = []
    for i in range(n):
        d, xs = kinds[i % len(kinds)]
        x, target = xs[i:i + M], targets[i:i + M]
        desc = d.desc(with_y=False)
        desc.M, desc.x, desc.target, desc.nnz_base = M, x.data_ptr(), target.data_ptr(), 65536 * i
        layers.append((d, desc, x, target))
    return szo.desc_array([l[1] for l in layers]), layers


def test_several_launches_of_many_layers():
    """Forty layers with three K in two launches of more entries than the arguments hold and more copies than one copy launch takes: every
    layer is multiplied with its own activations, targets and z."""
    descs, layers = _many_launches(40, (1920, 128, 1408))
    copies = szo.szo_workspace_bytes() - szo.szo_step_workspace_bytes()
    assert copies < sum(M * K * 2 for _, desc, _, _ in layers for M, K in [(desc.M, desc.K)]) < 2 * copies
    s = _step(descs, 12)
    total = np.sum([_step([desc], 12) for _, desc, _, _ in layers], axis=0)
    assert np.allclose(s[:2], total[:2], rtol=1e-12, atol=0.0) and abs(s[2] - total[2]) <= 1e-12 * s[0] / 1e-3      # the order of the partials
    two = _step(descs, 6)
    sigma = float(torch.cat([_gradient(*l) for l in layers]).norm())        # every layer has z of its own
    assert np.allclose(s[:2], two[:2], rtol=1e-5, atol=0.0) and abs(s[2] - two[2]) <= 1e-2 * max(abs(two[2]), sigma)


def test_the_host_runs_four_steps_ahead_of_the_gpu():
    """A step stages two tables, however many launches its layers take, and the eighth before is the first that a call waits for: four
    steps return while work before them on the stream is still running."""
    descs, keep = _many_launches()
    scal, ws = torch.zeros(3, dtype=torch.float64, device="cuda"), szo.new_workspace()
    szo.szo_set_tile_config(12)
    step = lambda: szo.szo_zo_step(descs, 9, 0, 1e-3, 0.0, scal, ws, szo.STEP_FUSED_LOSS)
    for _ in range(8):                                       # every pinned buffer has its size
        step()
    want = scal.cpu().numpy().copy()
    a = torch.randn((8192, 8192), device="cuda", dtype=torch.bfloat16)
    b = a @ a
    torch.cuda.synchronize()
    for _ in range(400):                                     # some 0.3 s
        torch.matmul(a, a, out=b)
    before = torch.cuda.Event()
    before.record()
    for _ in range(4):
        step()
    assert not before.query()
    assert np.array_equal(scal.cpu().numpy(), want)


@pytest.mark.parametrize("tile,instead", [("f16", 6), ("bf16", 11)])
def test_a_step_may_go_without_the_copies(tile, instead):
    """Told that the workspace ends before them, a large step takes the kernel that it took before there were copies, and leaves what is behind
    alone; with the bytes that the query gives it makes them and no more."""
    descs, keep = _stack(911, 29 if tile == "f16" else 11, 2304 if tile == "f16" else 768, 4096, 1024, 1e-3, False, 128, szo.TILE_BF16 if tile == "bf16" else szo.TILE_F16)
    wanted = _step(descs, 12), _step(descs, instead)
    szo.szo_set_tile_config(0)
    sizes = szo.szo_step_workspace_bytes(descs), szo.szo_step_workspace_bytes(descs, szo.STEP_FUSED_LOSS | szo.STEP_SMALL_WORKSPACE)
    assert sizes[1] == szo.szo_step_workspace_bytes() < 17 << 20 and sizes[0] > sizes[1]
    for flags, nbytes, want in zip((0, szo.STEP_SMALL_WORKSPACE), sizes, wanted):
        memory = torch.full((szo.szo_workspace_bytes(),), 0xA5, dtype=torch.uint8, device="cuda")
        szo.szo_workspace_init(memory)
        scal = torch.zeros(3, dtype=torch.float64, device="cuda")
        szo.szo_zo_step(descs, 9, 0, 1e-3, 0.0, scal, memory, szo.STEP_FUSED_LOSS | flags)
        assert np.array_equal(scal.cpu().numpy(), want) and bool((memory[nbytes:] == 0xA5).all())
