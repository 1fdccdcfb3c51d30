"""Registers of the attention kernels whose loops fill them, as the compiler reports them (no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_2510_21270_amd import build


def _kernels(directory, source, kernel):
    out = str(directory / "kernels.s")
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    subprocess.run(["hipcc"] + flags + ["-S", "--cuda-device-only", os.path.join(build.CSRC, source), "-o", out],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    with open(out) as f:
        text = f.read()
    found = {}
    for name, body in re.findall(r"\.name:\s+(\S*%s\S*)\n(.*?)\.wavefront_size" % kernel, text, re.S):
        found[name] = {k: int(v) for k, v in re.findall(r"\.(\w+):\s+(\d+)\n", body)}
    return found


@pytest.fixture(scope="module")
def wide_kernels(tmp_path_factory):
    return _kernels(tmp_path_factory.mktemp("asm"), "attn_wide.hip", "attn_wide_kernel")


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


def test_the_d64_loop_keeps_everything_in_registers(tmp_path):
    # two waves to a SIMD have 256 registers each, of which the loop takes 241 and 243
    kernels = _kernels(tmp_path, "attn_d64.hip", "attn_d64_kernel")
    assert len(kernels) == 2
    for name, info in kernels.items():
        assert info["vgpr_count"] <= 256, (name, info["vgpr_count"])
        assert info["vgpr_spill_count"] == info["sgpr_spill_count"] == info["private_segment_fixed_size"] == 0, name
