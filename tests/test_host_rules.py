"""The rules that choose a kernel and its launch, evaluated on the host by a probe that is compiled here from the library's own
sources (no GPU): waves per workgroup of the split kernel, and who takes a step where several kernels could."""
import os
import shutil
import subprocess

import pytest

from paper_2406_02913_amd import build as szo_build

HIPCC = szo_build.HIPCC if os.path.exists(szo_build.HIPCC) else shutil.which("hipcc")
pytestmark = pytest.mark.skipif(not HIPCC, reason="no hipcc")

PROBE = r"""
#include "szo_smallm.hip"
#include <cstdio>
using namespace szo;
static SplitLaunch g_last;
namespace szo { int split_launch(const SplitLaunch& l, const SmallArgs&, hipStream_t) { g_last = l; return SZO_OK; } }
// a line: layers, token rows, N, K, group, entries, bf16, table format, two sets, one sign (2: unperturbed), separate launches, asked for,
// K of one more layer
// with the argument "parts": tiles, columns -> whether K is computed in two parts
int main(int argc, char**) {
  long long tiles, columns;
  while (argc > 1 && scanf("%lld %lld", &tiles, &columns) == 2) printf("%d\n", tiles_halve_k(tiles, columns));
  long long n, M, N, K, group, nnz, bf16, lut, two, one, separate, asked, tail;
  while (scanf("%lld %lld %lld %lld %lld %lld %lld %lld %lld %lld %lld %lld %lld", &n, &M, &N, &K, &group, &nnz, &bf16, &lut, &two, &one, &separate, &asked, &tail) == 13) {
    szo_linear_desc d{};
    d.M = M; d.N = N; d.K = K; d.group = (int)group; d.nnz = nnz;
    d.tile_dtype = bf16 ? SZO_TILE_BF16 : SZO_TILE_F16;
    d.format = lut ? SZO_FORMAT_LUT : SZO_FORMAT_UNIFORM;
    d.x_minus = two ? &d : nullptr;
    std::vector<szo_linear_desc> descs((size_t)n, d);
    if (tail > 0) {                                         // and one of 4096 rows with a K of its own
      szo_linear_desc e = d;
      e.N = 4096; e.K = tail; e.nnz = nnz * 4096 * tail / (N * K);
      descs.push_back(e);
      ++n;
    }
    LaunchShape shape;
    for (const auto& e : descs) shape.add(&e);
    const FewPlan p = few_plan(&d, shape, two != 0);
    LaunchTotals t;
    for (const auto& e : descs) t.add(p, &e);
    SmallArgs a{};
    g_last = SplitLaunch{};
    if (p.split() && launch_plan(p, t, one != 0, a, nullptr) != SZO_OK) return 1;
    const bool few = one ? small_m_takes_forward(descs.data(), one == 1) : small_m_eligible(descs.data(), (int)n, false, separate != 0, 2);
    printf("%d %d %d %lld\n", few, g_last.waves, g_last.workgroups,
           one ? 0ll : (long long)onepass_partials(descs.data(), (int)n, few, asked != 0, false, separate != 0));
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    """ask(case, ...) -> [(few-token path, waves, workgroups, loss partials of the one-dense-pass kernel or 0), ...]"""
    if not os.path.exists(szo_build.LIB):
        szo_build.build()
    where = tmp_path_factory.mktemp("rules")
    src, exe = str(where / "probe.hip"), str(where / "probe")
    with open(src, "w") as f:
        f.write(PROBE)
    subprocess.check_call([HIPCC, "--cuda-host-only"] + szo_build.COMMON + [src, "-o", exe, "-L" + os.path.dirname(szo_build.LIB), "-l:" + os.path.basename(szo_build.LIB),
                           "-Wl,-rpath," + os.path.dirname(szo_build.LIB), "-Wl,--unresolved-symbols=ignore-all"], stderr=subprocess.DEVNULL)      # (the device code, which nothing here launches)

    def run(*cases):
        keys = ("layers", "M", "N", "K", "group", "nnz", "bf16", "lut", "two_sets", "one_sign", "separate", "asked_for", "tail_k")
        lines = "\n".join(" ".join(str(int(c.get(k, 0))) for k in keys) for c in cases)
        out = subprocess.run([exe], input=lines, capture_output=True, text=True, check=True).stdout.split("\n")
        return [tuple(int(v) for v in line.split()) for line in out[:len(cases)]]
    run.exe = exe
    return run


def _layer(N, K, M, density, layers=1, group=128, **kw):
    return dict(layers=layers, M=M, N=N, K=K, group=group, nnz=int(density * N * K + 0.5), **kw)


@pytest.mark.parametrize("case,waves,workgroups", [
    # sixteen waves: long K, or many entries per band
    (_layer(11008, 4096, 1, 1e-2, one_sign=1), 16, 172), (_layer(11008, 4096, 1, 3e-3, one_sign=1), 8, 172),
    (_layer(16384, 12416, 1, 1e-4, one_sign=1), 16, 256), (_layer(16384, 12288, 1, 1e-4, one_sign=1), 8, 256),
    (_layer(4096, 4096, 16, 1e-2, one_sign=1), 8, 256),               # cut in four: each part works on its own quarter of the entries
    # eight, and four beyond 1024 workgroups unless the mask is dense
    (_layer(16384, 4096, 64, 1e-3), 8, 1024), (_layer(8192, 16384, 48, 1e-4, layers=3), 4, 1152), (_layer(8192, 16384, 48, 1e-3, layers=3), 8, 1152),
    # both signs rounded with the weights: four beyond 256, eight for dense masks where one K is far longer than the others
    (_layer(5000, 4160, 48, 1e-3, group=64, bf16=1), 8, 237), (_layer(5000, 4160, 64, 1e-3, group=64, bf16=1), 4, 316),
    (_layer(5000, 4160, 64, 1e-2, group=64, bf16=1), 4, 316), (_layer(5000, 4160, 64, 1e-3, group=64, bf16=1, one_sign=1), 8, 316),
    (_layer(4096, 4096, 16, 1e-3, layers=6, bf16=1, tail_k=16384), 4, 448), (_layer(4096, 4096, 16, 2e-3, layers=6, bf16=1, tail_k=16384), 8, 448),
    (_layer(4096, 4096, 48, 3e-3, layers=6, bf16=1, tail_k=16384), 4, 1344), (_layer(4096, 4096, 48, 1e-2, layers=6, bf16=1, tail_k=16384), 8, 1344),
    (_layer(4096, 4096, 64, 2e-2, layers=8, bf16=1, tail_k=16384), 8, 2304), (_layer(4096, 4096, 64, 2e-2, layers=9, bf16=1, tail_k=16384), 4, 2560),
    # many slices: eight; tables: four beyond 1024
    (_layer(70, 5120, 1722, 7e-3, group=64), 8, 216), (_layer(8192, 16384, 48, 1e-3, layers=3, lut=1), 4, 1152),
    # two blocks of K: nothing to split
    (_layer(5000, 256, 4, 1e-2), 4, 158),
])
def test_waves_of_the_split_kernel(ask, case, waves, workgroups):
    (_, got, wgs, _), = ask(case)
    assert (got, wgs) == (waves, workgroups)


@pytest.mark.parametrize("case,few,onepass", [
    # only the split kernel can, up to 128 tokens as measured there; beyond, it or the one-dense-pass kernel or the tiles
    (_layer(11008, 4160, 200, 1e-3, group=64), True, True), (_layer(11008, 4160, 200, 1e-3, group=64, separate=1), True, True),
    (_layer(4059, 6848, 473, 3e-3, group=32), True, True), (_layer(1363, 2816, 1114, 3e-3, group=64, bf16=1), True, False), (_layer(402, 2688, 3276, 1e-3, group=64, bf16=1), True, False),
    (_layer(2080, 448, 905, 1e-3, group=32, separate=1), True, True), (_layer(4590, 1024, 491, 1e-3, group=32, bf16=1), True, True),
    (_layer(810, 9280, 2238, 1e-3, group=64, one_sign=1), False, False), (_layer(544, 13952, 2544, 1e-3, group=32, bf16=1, one_sign=1), True, False), (_layer(5344, 3584, 208, 1e-4, group=32, bf16=1), True, False),
    (_layer(3360, 4288, 535, 1e-3, group=64, bf16=1), True, False), (_layer(9196, 6592, 165, 1e-4, group=64, separate=1), True, False),
    (_layer(1653, 896, 419, 1e-4, group=64, bf16=1), True, False), (_layer(1653, 896, 419, 1e-4, group=64, bf16=1, asked_for=1), True, False),
    (_layer(4096, 4160, 128, 1e-3, group=64), True, False), (_layer(4096, 4160, 128, 1e-3, group=64, separate=1), True, False),
    # ... with two sets of activations: it or the tiles
    (_layer(4096, 4160, 200, 1e-2, group=32, bf16=1, two_sets=1), False, False), (_layer(5782, 3264, 394, 1e-4, group=64, two_sets=1), False, False),
    (_layer(3085, 6464, 187, 1e-4, group=64, two_sets=1), True, False), (_layer(2354, 704, 953, 1e-4, group=32, bf16=1, two_sets=1), False, False),
    (_layer(3552, 12416, 329, 1e-3, group=64, bf16=1, two_sets=1), True, False), (_layer(710, 4032, 2009, 1e-3, group=32), True, False),
    (_layer(3638, 8128, 137, 1e-2, group=64, two_sets=1), True, False),
])
def test_who_takes_layers_that_the_stream_kernel_does_not(ask, case, few, onepass):
    (got_few, _, _, partials), = ask(case)
    assert (bool(got_few), partials > 0) == (few, onepass)


@pytest.mark.parametrize("case,few", [
    # layers of few rows: a step at any of these sizes, a single forward up to 1536 bands and slices or well inside the line
    (_layer(258, 5248, 6437, 1e-3, one_sign=1), False), (_layer(258, 5248, 6437, 1e-3), True),
    (_layer(692, 15872, 2253, 1e-3, one_sign=1), False), (_layer(692, 15872, 2253, 1e-3), True), (_layer(2478, 16000, 695, 1e-3, one_sign=1), False),
    (_layer(423, 13184, 2884, 3e-4, one_sign=1), True), (_layer(285, 1152, 5600, 1e-3, one_sign=1), False), (_layer(300, 4096, 1000, 1e-3, one_sign=1), True),
    (_layer(635, 6400, 2409, 1e-4, one_sign=1), True), (_layer(111, 9088, 7496, 3e-3, one_sign=1), True),
    # with tables
    (_layer(300, 4096, 6000, 1e-3, lut=1, one_sign=1), False), (_layer(300, 4096, 6000, 1e-3, lut=1), True),
    (_layer(1231, 15872, 1741, 1e-3, lut=1, one_sign=1), False), (_layer(445, 9984, 3681, 1e-4, lut=1, one_sign=1), True),
    (_layer(4096, 4096, 450, 1e-3, lut=1, one_sign=1), True), (_layer(312, 12160, 4270, 1e-4, lut=1, one_sign=1), False), (_layer(799, 2304, 1037, 1e-4, lut=1, one_sign=1), True),
    # the group of a table layer decides nothing
    (_layer(1803, 2432, 700, 1e-3, lut=1), True), (_layer(1803, 2432, 700, 1e-3, lut=1, group=64), True),
    (_layer(1803, 2432, 700, 1e-3, lut=1, group=32), True),
])
def test_who_takes_many_tokens_of_few_rows(ask, case, few):
    (got, _, _, _), = ask(case)
    assert bool(got) == few


@pytest.mark.parametrize("case,few", [
    # unperturbed forwards against 128 x 128 tiles with K in two parts, either side of the line: groups, tokens, density, tiles (256 at most), columns
    (_layer(4096, 4096, 256, 1e-3, group=32, one_sign=2), True), (_layer(4096, 4096, 440, 1e-3, group=32, one_sign=2), False),
    (_layer(4096, 4096, 440, 1e-3, one_sign=2), True), (_layer(4096, 4096, 440, 1e-3, group=32, lut=1, one_sign=2), True), (_layer(4096, 4096, 440, 1e-3, group=32), True),
    (_layer(4096, 4096, 64, 1e-2, group=64, one_sign=2), True), (_layer(4096, 4096, 128, 1e-2, group=64, one_sign=2), False), (_layer(4096, 4096, 128, 1e-2, group=64, one_sign=2, bf16=1), True),
    (_layer(11008, 4096, 64, 1e-3, group=32, one_sign=2), True), (_layer(11008, 4096, 128, 1e-3, group=32, one_sign=2), False),
    (_layer(16384, 4096, 200, 1e-3, group=64, one_sign=2), False), (_layer(16512, 4096, 200, 1e-3, group=64, one_sign=2), True),
    (_layer(9359, 512, 69, 1e-3, group=64, one_sign=2), True), (_layer(13245, 256, 43, 1e-2, group=32, one_sign=2), False), (_layer(13245, 128, 43, 1e-2, group=32, one_sign=2), True),
    (_layer(2034, 1152, 317, 1e-2, group=64, one_sign=2), False), (_layer(3284, 512, 354, 1e-3, group=32, one_sign=2), False),
    # 256 columns: cut up to 192 tiles, whole beyond, few-token kernels beyond 256
    (_layer(24500, 256, 43, 1e-2, group=64, one_sign=2), False), (_layer(25000, 256, 43, 1e-2, group=64, one_sign=2), False), (_layer(25000, 256, 100, 5e-3, group=64, one_sign=2), True),
    (_layer(32768, 256, 100, 1e-2, group=64, one_sign=2), False), (_layer(32769, 256, 100, 1e-2, group=64, one_sign=2), True),
    # perturbed forwards stay where v and z are rounded one by one
    (_layer(3284, 512, 354, 1e-3, group=32, one_sign=1), True),
    (_layer(4096, 4096, 440, 1e-3, group=32, one_sign=1), True), (_layer(4096, 4096, 128, 1e-2, group=64, one_sign=1), True), (_layer(11008, 4096, 128, 1e-3, group=32, one_sign=1), True),
    (_layer(6140, 10752, 189, 1e-2, group=32, one_sign=1), True), (_layer(2034, 1152, 317, 1e-2, group=64, one_sign=1), True), (_layer(13245, 256, 43, 1e-2, group=32, one_sign=1), True),
])
def test_who_takes_a_single_forward_of_few_tiles(ask, case, few):
    (got, _, _, _), = ask(case)
    assert bool(got) == few


def test_where_tiles_compute_k_in_two_parts(ask):
    cases = {(192, 256): 1, (193, 256): 0, (193, 384): 1, (256, 384): 1, (257, 384): 0, (1, 128): 0, (1, 192): 0, (1, 320): 0, (1, 256): 1, (1, 448): 0, (256, 16384): 1, (257, 16384): 0}
    out = subprocess.run([ask.exe, "parts"], input="\n".join("%d %d" % c for c in cases), capture_output=True, text=True, check=True).stdout
    assert [int(v) for v in out.split()] == list(cases.values())


@pytest.mark.parametrize("case,onepass", [
    # either side of the lines on the mask's density beyond 512 tokens: 1.34 / 4 with the fp16 tile and K a multiple of 128, else 1.22 / 4
    (_layer(2048, 512, 1024, 3.0e-3), True), (_layer(2048, 512, 1024, 3.3e-3), False),
    (_layer(2368, 320, 1024, 1.9e-3, group=64, bf16=1), True), (_layer(2368, 320, 1024, 2.2e-3, group=64, bf16=1), False),
    (_layer(2368, 320, 1024, 1.9e-3, group=64), True), (_layer(2368, 320, 1024, 2.2e-3, group=64), False),
    # 2048 tokens; 2048 tiles of 256 x 128 beyond
    (_layer(29184, 128, 2048, 1e-3), True), (_layer(29184, 128, 2049, 1e-3), False), (_layer(29056, 128, 2049, 1e-3), True),
    (_layer(16384, 128, 2049, 1e-3), True), (_layer(16384, 128, 2049, 1e-3, layers=2), False),
])
def test_who_takes_one_dense_product_beyond_512_tokens(ask, case, onepass):
    (few, _, _, partials), = ask(case)
    assert not few and (partials > 0) == onepass


def _descs(layers, x_of=lambda i: i, **changes):
    """Descriptors that validate; their addresses are never followed."""
    from paper_2406_02913_amd import szo
    at = 1 << 20
    out = []
    for i, (M, N, K, density) in enumerate(layers):
        d = szo.LinearDesc(M, N, K, 128, szo.TILE_F16, int(density * N * K), 0, at + (x_of(i) << 30), at, at, at, at, at, None, at, None, 0, 0, None)
        for name, value in changes.items():
            setattr(d, name, value)
        out.append(d)
    return out


def test_the_workspace_holds_copies_only_for_steps_that_make_them():
    from paper_2406_02913_amd import szo, synth
    at = 1 << 20
    small, whole = szo.szo_step_workspace_bytes(), szo.szo_workspace_bytes()
    assert 64 + 8 * (1 << 21) <= small <= 17 << 20 and small + (1 << 30) <= whole
    block = lambda M, n, density=1e-3: [(M, N, K, density) for _ in range(n) for _, N, K in synth.LLAMA2_7B_BLOCK]
    of = lambda layers, flags=szo.STEP_FUSED_LOSS, **kw: szo.szo_step_workspace_bytes(_descs(layers, **kw), flags)
    copy = lambda M, K: -(-M // 64) * 64 * K * 2
    # the largest steps: the copies of a launch's layers, each x once
    assert 0.9 * (1 << 30) < of(block(4096, 32)) - small <= whole - small
    assert of(block(4096, 2)) == small + 128 + 2 * sum(copy(4096, K) for _, _, K in synth.LLAMA2_7B_BLOCK)
    assert of(block(4096, 2), x_of=lambda i: i % 7 // 6) == small + 128 + copy(4096, 4096) + copy(4096, 11008)
    assert of(block(1000, 1), tile_dtype=szo.TILE_BF16) > small
    # steps that other kernels take, and layers that this one does not
    assert of(block(4096, 1)) == of(block(16, 32)) == of(block(1000, 1)) == of(block(4096, 32, 1e-2)) == of([(64, 256, 256, 1e-3)]) == small
    assert of(block(4096, 32), x_minus=at) == of(block(4096, 32), format=szo.FORMAT_LUT, lut=at) == small
    assert of(block(65536, 1)) == small                      # one copy alone is larger than what there is
    assert of(block(4096, 32), flags=0, y=at) == small
    # ... and those that are told
    assert of(block(4096, 32), szo.STEP_FUSED_LOSS | szo.STEP_SMALL_WORKSPACE) == small
    # what is refused writes nothing; said before its addresses are known the answer is no promise
    assert of(block(4096, 1), x=None) == whole
