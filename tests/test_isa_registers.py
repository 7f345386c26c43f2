"""Generated gfx950 code: register and LDS use that a kernel's speed rests on (no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2406_02913_amd import build as szo_build

HIPCC = szo_build.HIPCC if os.path.exists(szo_build.HIPCC) else shutil.which("hipcc")


@pytest.mark.skipif(not HIPCC, reason="no hipcc")
def test_the_update_of_a_stack_keeps_eight_waves_per_simd(tmp_path):
    """The update without the reduction: no LDS and at most 32 of the 64 registers that eight waves leave each."""
    out = str(tmp_path / "smallm.s")
    subprocess.check_call([HIPCC, "--cuda-device-only", "-S"] + szo_build.COMMON + szo_build.DEVICE +
                          [os.path.join(szo_build.CSRC, "szo_smallm.hip"), "-o", out], stderr=subprocess.DEVNULL)
    kernels = re.findall(r"\.amdhsa_kernel (\S*sparse_update_table_kernel\S*)(.*?)\.end_amdhsa_kernel", open(out).read(), re.S)
    use = {name: (int(re.search(r"amdhsa_group_segment_fixed_size (\d+)", body).group(1)),
                  int(re.search(r"amdhsa_next_free_vgpr (\d+)", body).group(1))) for name, body in kernels}
    assert len([u for u in use.values() if u[0] == 0 and u[1] <= 32]) == 2, use      # table staged, table in the arguments


def _blocks(text, kernel):
    """Straight stretches of a kernel's instructions: between labels and branches."""
    start = text.index("\n" + kernel + ":")
    blocks, cur = [], []
    for line in text[start:text.index(".section", start)].splitlines():
        t = line.split(";")[0].strip()
        if re.match(r"\.LBB\w+:", t) or t.startswith(("s_cbranch", "s_branch")):
            blocks.append(cur)
            cur = []
        elif t and not t.startswith("."):
            cur.append(t.split()[0])
    return blocks + [cur]


@pytest.mark.skipif(not HIPCC, reason="no hipcc")
def test_further_groups_of_sensitive_entries_gather_beside_their_products(tmp_path):
    """One-dense-pass kernel: the loop over a chunk's entries beyond the first sixteen is one stretch of sixteen gathers and
    eight matrix instructions in every form (a branch between them cost dense masks 2 to 6 %), and the forms for denser masks
    have none in the schedule's group either."""
    out = str(tmp_path / "onepass.s")
    subprocess.check_call([HIPCC, "--cuda-device-only", "-S"] + szo_build.COMMON + szo_build.DEVICE +
                          [os.path.join(szo_build.CSRC, "szo_onepass.hip"), "-o", out], stderr=subprocess.DEVNULL)
    text = open(out).read()
    kernels = re.findall(r"\.amdhsa_kernel (\S*onepass_\S*kernel\S*)", text)
    assert len(kernels) >= 11
    whole_schedules = 0
    for kernel in kernels:
        count = [(sum(i.startswith("v_mfma") for i in b), sum(i.startswith("ds_read_u16") for i in b)) for b in _blocks(text, kernel)]
        assert (8, 16) in count, (kernel, [c for c in count if c[0]])
        whole_schedules += any(m > 8 and g == 16 for m, g in count)
    assert 2 * whole_schedules >= len(kernels)


@pytest.mark.skipif(not HIPCC, reason="no hipcc")
def test_the_tiled_kernels_keep_their_main_loops_in_registers(tmp_path):
    """A register spilled in the main loop costs 8 to 15 % of a step.  The tiles with one dense product spill some words behind it, none
    before the end of its last products (stretches of 64 and more matrix instructions) and none among the sensitive products; the
    other grouped forms spill none at all."""
    out = str(tmp_path / "gemm.s")
    subprocess.check_call([HIPCC, "--cuda-device-only", "-S"] + szo_build.COMMON + szo_build.DEVICE +
                          [os.path.join(szo_build.CSRC, "szo_gemm.hip"), "-o", out], stderr=subprocess.DEVNULL)
    text = open(out).read()
    scratch = {name: int(size) for name, size in re.findall(r"\.name:\s+(\S*linear_fwd_table_kernel\S*)\s+\.private_segment_fixed_size: (\d+)", text)}
    shared = [name for name in scratch if re.search(r"Li16ELi[12]EEEv", name)]
    assert len(shared) == 4 and len(scratch) > 3
    assert all(size == 0 for name, size in scratch.items() if name not in shared), scratch
    for name in shared:
        blocks = _blocks(text, name)
        count = [(sum(i.startswith("v_mfma") for i in b), sum(i.startswith("scratch_") for i in b)) for b in blocks]
        main = [i for i, (products, _) in enumerate(count) if products >= 64]
        assert len(main) >= 2 and not any(spills for _, spills in count[:main[-1] + 1]), name
        assert any(0 < products < 64 for products, _ in count[main[-1] + 1:]) and not any(products and spills for products, spills in count), name
        assert scratch[name] <= 96, (name, scratch[name])
