"""The 32 x 32 tile blend kernels of one workgroup per tile (16 wavefronts) fit
twice on a CU: at most 64 vector registers and half the LDS (CPU: the register
counts in the metadata of a gfx950 build of render.hip)."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_two_workgroups_of_32x32_tiles_per_cu(tmp_path):
    from paper_2403_04116_amd import build
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc not installed")
    asm = str(tmp_path / "render.s")
    subprocess.check_call([build.HIPCC, *build.CFLAGS, "--offload-device-only", "-S",
                           os.path.join(build.CSRC, "render.hip"), "-o", asm])
    text = open(asm).read()
    kernels = {}
    for block in re.split(r"\n  - \.agpr_count", text)[1:]:
        name = re.search(r"\.name:\s+(\S+)", block).group(1)
        kernels[name] = [int(re.search(rf"\.{key}:\s+(\d+)", block).group(1))
                         for key in ("vgpr_count", "group_segment_fixed_size")]
    # template arguments: tile, batch, then PERSIST where there is one
    plain = [n for n in kernels if re.search(r"k_render_(fwdILi32ELi\d+ELb[01]ELb0E|bwdILi32ELi\d+ELb0E|fwd_rgbILi32E)", n)]
    assert len(plain) == 3 * (3 + 2 + 1)   # batches x (plain, stored, counts; plain, stored; colours)
    for n in plain:
        vgpr, lds = kernels[n]
        assert vgpr <= 64 and lds <= 80 * 1024, (n, vgpr, lds)
