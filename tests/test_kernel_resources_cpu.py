"""Registers of the block-128 attention kernel, as the compiler reports them (no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_2510_21270_amd import build


@pytest.fixture(scope="module")
def wide_kernels(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "attn_wide.s")
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    subprocess.run(["hipcc"] + flags + ["-S", "--cuda-device-only", os.path.join(build.CSRC, "attn_wide.hip"), "-o", out],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    with open(out) as f:
        text = f.read()
    found = {}
    for name, body in re.findall(r"\.name:\s+(\S*attn_wide_kernel\S*)\n(.*?)\.wavefront_size", text, re.S):
        found[name] = {k: int(v) for k, v in re.findall(r"\.(\w+):\s+(\d+)\n", body)}
    return found


def test_a_row_s_loop_keeps_its_scalars_in_scalar_registers(wide_kernels):
    # Spilled scalar registers are lanes of a vector register: each costs an instruction in every block of a masked
    # sub-tile that needs it (24 .. 28 of 120, 5 % of short masked lists, when 162 were spilled).  The form that takes rows
    # from queues holds a few that are read between rows.
    assert len(wide_kernels) == 3
    queues = [k for k in wide_kernels if "ILi1ELb1E" in k]
    assert len(queues) == 1
    for name, info in wide_kernels.items():
        assert info["vgpr_spill_count"] == 0 and info["private_segment_fixed_size"] == 0, name
        assert info["sgpr_spill_count"] <= (16 if name in queues else 0), (name, info["sgpr_spill_count"])
