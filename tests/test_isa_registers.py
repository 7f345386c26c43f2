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
